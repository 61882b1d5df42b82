// Prediction-quality diagnostics on the device (Sec. "Metrics" and the prediction-quality study):
// the top-k hit rate of the early pass against the actual routing, the mean per-token cosine
// similarity of two row-major matrices (hidden states h_{l-1} vs H_l, or early vs actual logits),
// and the fold of a count vector into rank loads under a placement (the realised balance of the
// actual routing under the old or the planned placement).
//
// Everything is deterministic: hits are an integer sum; cosines are summed per wave in a fixed
// order into a workspace and reduced by one workgroup in index order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fb_internal.h"

namespace fb {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kQThreads = 256;
constexpr int kQWaves = kQThreads / 64;

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// One token per thread: the predicted experts become a bit set, the actual ones are looked up.
// Bound by latency at the sizes of one layer.  The workgroups' sums meet in *hits, zeroed before the
// launch; where the rate is wanted they also count arrivals above bit kHitsBits (T * k < 2^48), so that
// the last one writes the sum and the rate with no launch of its own.  Ids are fetched four at a time,
// the first four of both lists before any is used; the unrolled code of eight at a time costs more in
// instruction fetches than it saves.  One by one / four / eight (both launches of a call, us): T = 8190,
// k = 6 5.6 / 5.1 / 5.4, k = 8 6.2 / 5.9 / 6.8, T = 1000, k = 2 4.4 / 4.3 / 5.1, k = 32 16.5 / 11.1 /
// 11.8, T = 300000, k = 8 23.9 / 21.5 / 19.9; the rate adds 0.2 to 0.7, as a launch of its own 1.5.
constexpr int kHitsBits = 48;
constexpr int kHitsBlocks = 1024;                // arrivals stay below 2^15
constexpr int kIds = 4;                          // ids fetched together
__global__ __launch_bounds__(kQThreads) void hits_kernel(const int32_t* __restrict__ pred,
                                                         const int32_t* __restrict__ act, int64_t T,
                                                         int32_t k, unsigned long long* __restrict__ hits,
                                                         double* __restrict__ rate) {
  __shared__ unsigned long long s_part[kQWaves];
  unsigned long long h = 0;
  for (int64_t t = blockIdx.x * (int64_t)kQThreads + threadIdx.x; t < T; t += (int64_t)gridDim.x * kQThreads) {
    const int32_t* p = pred + t * k;
    const int32_t* q = act + t * k;
    uint32_t bits[FB_MAX_EXPERTS / 32];
#pragma unroll
    for (int w = 0; w < FB_MAX_EXPERTS / 32; ++w) bits[w] = 0;
    uint32_t ip[kIds], iq[kIds];
    auto fetch = [&](uint32_t(&id)[kIds], const int32_t* from, int j0) {
#pragma unroll
      for (int j = 0; j < kIds; ++j) id[j] = j0 + j < k ? (uint32_t)from[j0 + j] : FB_MAX_EXPERTS;
    };
    fetch(ip, p, 0);
    fetch(iq, q, 0);
    for (int j0 = 0;;) {
#pragma unroll
      for (int j = 0; j < kIds; ++j)
#pragma unroll
        for (int w = 0; w < FB_MAX_EXPERTS / 32; ++w) bits[w] |= (w == (int)(ip[j] >> 5)) ? 1u << (ip[j] & 31) : 0u;
      j0 += kIds;
      if (j0 >= k) break;
      fetch(ip, p, j0);
    }
    for (int j0 = 0;;) {
#pragma unroll
      for (int j = 0; j < kIds; ++j) {
        uint32_t word = 0;
#pragma unroll
        for (int w = 0; w < FB_MAX_EXPERTS / 32; ++w) word = (w == (int)(iq[j] >> 5)) ? bits[w] : word;
        h += (word >> (iq[j] & 31)) & 1u;
      }
      j0 += kIds;
      if (j0 >= k) break;
      fetch(iq, q, j0);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) h += __shfl_xor(h, off);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = h;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long sum = 0;
    for (int w = 0; w < kQWaves; ++w) sum += s_part[w];
    if (rate == nullptr) {
      if (sum) atomicAdd(hits, sum);
      return;
    }
    const unsigned long long all = atomicAdd(hits, (1ull << kHitsBits) | sum) + sum;
    if ((all >> kHitsBits) == gridDim.x - 1) {
      const unsigned long long total = all & ((1ull << kHitsBits) - 1);
      atomicExch(hits, total);
      if (rate) *rate = T > 0 ? (double)total / (double)(T * k) : 1.0;
    }
  }
}

__global__ void zero_u64_kernel(unsigned long long* p) { *p = 0ull; }

// LPR lanes per row, 64 / LPR rows of a wave at a time; 16-byte loads; products and sums in double.
// Each wave writes the sum of the cosines of the rows it handled to partial[wave id].  Wide rows are
// bound by HBM (hidden states, 2048 columns of bf16: 4.9 TB/s of the card's 5.2 TB/s copy rate); rows
// of at most 32 chunks, such as logits, leave most of a 64-lane row's lanes idle and are bound by the
// reductions per row, so 16 lanes take one: 8190 x 64 float32 6.4
// -> 3.8 us.
template <bool BF16, int LPR>
__global__ __launch_bounds__(kQThreads) void cosine_kernel(const char* __restrict__ a,
                                                           const char* __restrict__ b, int64_t rows,
                                                           int32_t cols, int64_t lda_bytes,
                                                           int64_t ldb_bytes, double* __restrict__ partial) {
  constexpr int RPW = 64 / LPR;                // rows of a wave
  const int lane = threadIdx.x & 63;
  const int in_row = lane % LPR;
  const int64_t wave = (int64_t)blockIdx.x * kQWaves + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kQWaves;
  constexpr int kPer = BF16 ? 8 : 4;          // elements per 16-byte chunk
  const int chunks = cols / kPer;
  double acc = 0.0;
  for (int64_t r0 = wave * RPW; r0 < rows; r0 += nwaves * RPW) {
    const int64_t r = r0 + lane / LPR;
    double dot = 0.0, aa = 0.0, bb = 0.0;
    if (r < rows) {
      const u32x4* ra = reinterpret_cast<const u32x4*>(a + r * lda_bytes);
      const u32x4* rb = reinterpret_cast<const u32x4*>(b + r * ldb_bytes);
      for (int c = in_row; c < chunks; c += LPR) {
        const u32x4 va = __builtin_nontemporal_load(ra + c);
        const u32x4 vb = __builtin_nontemporal_load(rb + c);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (BF16) {
            const double x0 = (double)__uint_as_float(va[q] << 16), x1 = (double)__uint_as_float(va[q] & 0xFFFF0000u);
            const double y0 = (double)__uint_as_float(vb[q] << 16), y1 = (double)__uint_as_float(vb[q] & 0xFFFF0000u);
            dot = fma(x0, y0, dot); dot = fma(x1, y1, dot);
            aa = fma(x0, x0, aa); aa = fma(x1, x1, aa);
            bb = fma(y0, y0, bb); bb = fma(y1, y1, bb);
          } else {
            const double x = (double)__uint_as_float(va[q]), y = (double)__uint_as_float(vb[q]);
            dot = fma(x, y, dot); aa = fma(x, x, aa); bb = fma(y, y, bb);
          }
        }
      }
    }
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) {
      dot += __shfl_xor(dot, off);
      aa += __shfl_xor(aa, off);
      bb += __shfl_xor(bb, off);
    }
    if (r < rows) acc += dot / (sqrt(aa) * sqrt(bb));
  }
#pragma unroll
  for (int off = 32; off >= LPR; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) partial[wave] = acc;
}

// Sum of the per-wave partials in a fixed order (one workgroup), divided by the row count: a chain of
// latencies, so coalesced loads and wave sums rather than one thread adding 256 (4.9 -> 2.5 us).
__global__ __launch_bounds__(kQThreads) void mean_kernel(const double* __restrict__ partial, int64_t n,
                                                         int64_t rows, double* __restrict__ out) {
  __shared__ double s[kQWaves];
  double v = 0.0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < n; i += kQThreads) v += partial[i];
  v = wave_sum_f64(v);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double sum = 0.0;
    for (int w = 0; w < kQWaves; ++w) sum += s[w];
    *out = rows > 0 ? sum / (double)rows : 1.0;
  }
}

// Rank loads and max-to-mean of a count vector under a placement (one workgroup).
__global__ __launch_bounds__(kQThreads) void fold_kernel(const int32_t* __restrict__ counts, int32_t E,
                                                         const int32_t* __restrict__ e2r, int32_t R,
                                                         int32_t* __restrict__ rank_loads,
                                                         double* __restrict__ max_mean) {
  __shared__ int32_t rl[FB_MAX_RANKS];
  __shared__ int32_t s_bad;
  __shared__ long long s_mx[kQWaves], s_sum[kQWaves];
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  for (int r = tid; r < R; r += kQThreads) rl[r] = 0;
  __syncthreads();
  for (int e = tid; e < E; e += kQThreads) {
    const int r = e2r[e];
    if (r >= 0 && r < R) atomicAdd(&rl[r], counts[e]);
    else s_bad = 1;
  }
  __syncthreads();
  long long mx = 0, sum = 0;
  for (int r = tid; r < R; r += kQThreads) {
    const int v = rl[r];
    rank_loads[r] = v;
    mx = v > mx ? v : mx;
    sum += v;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const long long om = __shfl_xor(mx, off), os = __shfl_xor(sum, off);
    mx = om > mx ? om : mx;
    sum += os;
  }
  if ((tid & 63) == 0) { s_mx[tid >> 6] = mx; s_sum[tid >> 6] = sum; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kQWaves; ++w) { mx = s_mx[w] > mx ? s_mx[w] : mx; sum += s_sum[w]; }
    *max_mean = s_bad ? -1.0 : (sum == 0 ? 1.0 : (double)mx * (double)R / (double)sum);
  }
}

}  // namespace

size_t cosine_workspace_bytes() { return (size_t)kCosineBlocks * kQWaves * sizeof(double); }

int launch_hits(const int32_t* pred, const int32_t* act, int64_t T, int32_t k, int64_t* hits,
                double* rate, void* stream) {
  (void)hipGetLastError();
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto* h = reinterpret_cast<unsigned long long*>(hits);
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(1), 0, st, h);
  const int64_t blocks = (T + kQThreads - 1) / kQThreads;
  hipLaunchKernelGGL(hits_kernel, dim3((unsigned)(blocks < 1 ? 1 : blocks < kHitsBlocks ? blocks : kHitsBlocks)),
                     dim3(kQThreads), 0, st, pred, act, T, k, h, rate);
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

int launch_cosine(const void* a, const void* b, int64_t rows, int32_t cols, int64_t lda, int64_t ldb,
                  int32_t dtype, double* out, void* workspace, void* stream) {
  (void)hipGetLastError();
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int elem = dtype == FB_BF16 ? 2 : 4;
  double* partial = static_cast<double*>(workspace);
  // rows of at most 32 chunks of 16 bytes take 16 lanes each (see cosine_kernel)
  const bool narrow = (int64_t)cols * elem <= 32 * 16;
  const int64_t per_block = kQWaves * (narrow ? 4 : 1);
  const int64_t blocks64 = (rows + per_block - 1) / per_block;
  const int blocks = (int)(blocks64 < kCosineBlocks ? (blocks64 > 0 ? blocks64 : 1) : kCosineBlocks);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kQThreads), 0, st, static_cast<const char*>(a),
                       static_cast<const char*>(b), rows, cols, lda * elem, ldb * elem, partial);
  };
  if (dtype == FB_BF16) narrow ? go(cosine_kernel<true, 16>) : go(cosine_kernel<true, 64>);
  else narrow ? go(cosine_kernel<false, 16>) : go(cosine_kernel<false, 64>);
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(kQThreads), 0, st, partial, (int64_t)blocks * kQWaves,
                     rows, out);
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

// Rank loads of a replicated placement: slot value v = e + E * j is replica j of expert e, which
// carries floor(n_e / c_e) tokens plus one if j < n_e mod c_e (c_e = replicas of e).  One workgroup
// checks the placement rules (values in range, every expert present, the ordinals of every expert
// exactly 0 .. c_e - 1, no rank with two replicas of one expert, counts >= 0) and sums the shares per
// rank in LDS; a violated rule makes *max_mean = -1.  R * S <= FB_MAX_SLOTS_TOTAL and E <= R * S.
namespace {
__global__ __launch_bounds__(kQThreads) void slot_fold_kernel(
    const int32_t* __restrict__ counts, int32_t E, const int32_t* __restrict__ slots, int32_t R,
    int32_t S, int32_t* __restrict__ rank_loads, double* __restrict__ max_mean) {
  __shared__ int32_t reps[FB_MAX_SLOTS_TOTAL];   // replicas per expert
  __shared__ int32_t base[FB_MAX_SLOTS_TOTAL];   // exclusive prefix sum of reps
  __shared__ int32_t seen[FB_MAX_SLOTS_TOTAL];   // one flag per (expert, ordinal), at base[e] + j
  __shared__ int32_t sexp[FB_MAX_SLOTS_TOTAL];   // expert of every slot, -1 if empty or invalid
  __shared__ int32_t rl[FB_MAX_RANKS];
  __shared__ int32_t part[kQThreads];
  __shared__ int32_t s_bad;
  __shared__ long long s_mx[kQWaves], s_sum[kQWaves];
  const int tid = threadIdx.x;
  const int RS = R * S;
  if (tid == 0) s_bad = 0;
  for (int e = tid; e < E; e += kQThreads) reps[e] = 0;
  for (int c = tid; c < RS; c += kQThreads) seen[c] = 0;
  for (int r = tid; r < R; r += kQThreads) rl[r] = 0;
  __syncthreads();
  for (int c = tid; c < RS; c += kQThreads) {
    const int v = slots[c];
    int e = -1;
    if (v != -1) {
      if (v < 0 || v / E >= R) {
        s_bad = 1;
      } else {
        e = v % E;
        atomicAdd(&reps[e], 1);
      }
    }
    sexp[c] = e;
  }
  __syncthreads();
  // exclusive prefix sum of reps: each thread sums a contiguous chunk, thread 0 scans the chunks
  const int chunk = (E + kQThreads - 1) / kQThreads;
  const int e0 = tid * chunk, e1 = e0 + chunk < E ? e0 + chunk : E;
  int acc = 0;
  for (int e = e0; e < e1; ++e) acc += reps[e];
  part[tid] = acc;
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int t = 0; t < kQThreads; ++t) {
      const int x = part[t];
      part[t] = run;
      run += x;
    }
  }
  __syncthreads();
  acc = part[tid];
  for (int e = e0; e < e1; ++e) {
    base[e] = acc;
    acc += reps[e];
    if (reps[e] == 0 || counts[e] < 0) s_bad = 1;
  }
  __syncthreads();
  for (int c = tid; c < RS; c += kQThreads) {
    const int e = sexp[c];
    if (e < 0) continue;
    const int j = slots[c] / E;
    // base[e] + j stays below base[e] + reps[e] <= RS only when j < reps[e]
    if (j >= reps[e] || atomicAdd(&seen[base[e] + j], 1) != 0) {
      s_bad = 1;
      continue;
    }
    // no other slot of the same rank holds this expert
    const int r0 = (c / S) * S;
    for (int c2 = r0; c2 < c; ++c2)
      if (sexp[c2] == e) s_bad = 1;
    const int n = counts[e], k = reps[e];
    atomicAdd(&rl[c / S], n / k + (j < n % k ? 1 : 0));
  }
  __syncthreads();
  long long mx = 0, sum = 0;
  for (int r = tid; r < R; r += kQThreads) {
    const int v = rl[r];
    rank_loads[r] = v;
    mx = v > mx ? v : mx;
    sum += v;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const long long om = __shfl_xor(mx, off), os = __shfl_xor(sum, off);
    mx = om > mx ? om : mx;
    sum += os;
  }
  if ((tid & 63) == 0) { s_mx[tid >> 6] = mx; s_sum[tid >> 6] = sum; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kQWaves; ++w) { mx = s_mx[w] > mx ? s_mx[w] : mx; sum += s_sum[w]; }
    *max_mean = s_bad ? -1.0 : (sum == 0 ? 1.0 : (double)mx * (double)R / (double)sum);
  }
}
}  // namespace

int launch_fold(const int32_t* counts, int32_t E, const int32_t* e2r, int32_t R, int32_t* rank_loads,
                double* max_mean, void* stream) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(fold_kernel, dim3(1), dim3(kQThreads), 0, static_cast<hipStream_t>(stream), counts,
                     E, e2r, R, rank_loads, max_mean);
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

int launch_slot_fold(const int32_t* counts, int32_t E, const int32_t* slots, int32_t R, int32_t S,
                     int32_t* rank_loads, double* max_mean, void* stream) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(slot_fold_kernel, dim3(1), dim3(kQThreads), 0, static_cast<hipStream_t>(stream),
                     counts, E, slots, R, S, rank_loads, max_mean);
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

}  // namespace fb
