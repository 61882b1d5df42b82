// Fused residual workload predictor for gfx950 (MI355X).
//
// One kernel computes, for a tile of tokens, the early router logits (Sec. "Residual Workload
// Prediction", Eq. 2 with the linear router of Eq. 4), the routed model's scores and its
// (optionally group-limited) top-k selection, and the per-expert token histogram of Eq. 5.  The
// last workgroup to finish folds the histogram into per-rank loads under the expert-to-rank
// placement (Alg. 1, second step) and computes the max-to-mean ratio (Sec. "Metrics").
//
// Workgroup: 4 waves (256 threads), one per SIMD, one workgroup per CU.  A wave may then hold up to
// 512 registers, which the contraction spends on deep prefetching rather than on extra waves:
//   * Hidden rows go from HBM straight into LDS (buffer_load ... lds, 16 bytes per lane): no
//     register round trip and no LDS store instructions.  The k dimension runs in stages of 256
//     bytes of every row; a ring of NS stage buffers keeps up to NS - 1 stages in flight beyond the
//     one being read.  Each
//     workgroup-wide load instruction writes 4 rows x 256 bytes; inside a row the 16-byte chunks are
//     XOR-swizzled by the row index so the fragment reads below are free of bank conflicts.
//   * Each wave owns a slice of the experts (and, for small E, of the tokens).  Its router-weight
//     fragments come from the pre-packed weight (one contiguous 1 KB per load instruction,
//     L2-resident) straight into registers through a ring of 16 k-step slices, 15 k-steps ahead of
//     the MFMAs; the hidden fragments are read from LDS one k-step ahead.  The router weight is the
//     A operand (M = experts) and the hidden tile is B (N = tokens): v_mfma_f32_32x32x16_bf16 (or
//     v_mfma_f32_32x32x2_f32, or bf16 parts of the values, for f32), so each lane ends with groups of four
//     consecutive experts of one token.
//   * One workgroup barrier per stage, placed before the stage's last k-step: it publishes the next
//     stage (every wave waits for its own share of that stage's loads first) and frees the buffer
//     just read, which the next load batch then refills.  Waits are counted, never drained.
// The logits never leave the chip: scores go to an LDS tile, EPAD/32 lanes cooperate on one
// token, and the histogram is privatised in LDS with one global atomic per expert per workgroup.
//
// Selection is exact in float32 with ties to the lower expert index.  The fast path ranks 32-bit
// keys (top 24 bits of the order-preserving score encoding, then 255 - expert); its set equals the
// exact top-k whenever the k-th and (k+1)-th keys differ in their score bits, and tokens where they
// do not take an exact 64-bit path.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "fb_internal.h"
#include "fb_plan_wave.h"

namespace fb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kStepBytes = 32;                  // bytes of a row feeding one MFMA k-step
constexpr int kNStep = 8;                       // k-steps per stage
constexpr int kStageRowBytes = kStepBytes * kNStep;   // 256
constexpr int kRingW = 16;                      // router-weight k-step slices held per wave
constexpr int kMaxSplits = 16;                  // workgroups that share a tile's stages
constexpr int kMaxK = FB_MAX_TOPK;
constexpr int kMaxGroups = 32;
constexpr uint32_t kRsrcWord3 = 0x00020000u;    // raw buffer, 32-bit dwords
constexpr uint32_t kOobOffset = 0x80000000u;    // fails the buffer range check: load returns 0
#ifndef FB_SEL_CACHE
#define FB_SEL_CACHE 7
#endif
constexpr int kCache = FB_SEL_CACHE;            // per-lane cached keys in the top-k extraction

// Tile shapes: WE waves along experts x WT waves along tokens, BM tokens per workgroup; every wave
// tile is a whole number of 32 x 32 MFMA blocks.
template <int EPAD> struct TileCfg;
template <> struct TileCfg<256> { static constexpr int WE = 4, WT = 1, BM = 128; };
template <> struct TileCfg<128> { static constexpr int WE = 4, WT = 1, BM = 64; };
template <> struct TileCfg<64> { static constexpr int WE = 2, WT = 2, BM = 64; };
template <> struct TileCfg<32> { static constexpr int WE = 1, WT = 4, BM = 128; };

// Stages of the LDS ring for a tile height.  Each wave may have at most 63 vector-memory loads in
// flight; NS is the deepest ring whose counted waits stay below that (checked in the kernel).
constexpr int ring_stages(int BM) { return BM >= 128 ? 3 : 4; }

struct Params {
  const char* x;
  int64_t T;
  int32_t Hbytes;
  int32_t ldx_bytes;
  const char* wpack;   // packed router weight (see pack_kernel)
  int32_t E;
  const float* logit_bias;
  const float* select_bias;
  int32_t kind, k, n_group, topk_group, group_topn;
  const int32_t* e2r;
  int32_t R;
  int32_t* counts;
  int32_t* rank_loads;
  double* max_mean;
  int32_t* ws_acc;
  uint32_t* ws_ticket;
  uint32_t* ws_tile;   // split mode: arrival word per tile (kSplit)
  int32_t* topk_idx;
  float* logits;
  uint32_t tickets;    // workgroups that count (of both launches where a batch takes two)
  uint32_t full;       // split mode: tiles before the first split one, contracted whole by a launch before
  int32_t nstages;     // stages this workgroup contracts
  int32_t st_base;     // first of them
  int32_t st_total;    // stages of a whole row
  int32_t ks;          // splits of the stage range (split mode); 1 otherwise
  float* partial;      // split mode: partial logits, [tile][split][expert / 4][token][expert mod 4]
  int32_t plan_cpl;    // 0: no plan; 1 or 2: the one-wave planner's candidates per lane
  int32_t arrival_polls;   // kShare: looks at the arrival word before a slice is given up
  PlanDeviceLaunch plan;   // the swap plan of the counts, made by the last workgroup
};

// Workgroup barrier that orders LDS only; outstanding global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// 32-bit LDS address of a pointer into a __shared__ array.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// 16-byte LDS read as an instruction of its own; its completion is awaited with lgkm_wait.
__device__ __forceinline__ void ds_read_b128(u32x4& dst, uint32_t addr, int offset) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "i"(offset));
}
template <int N>
__device__ __forceinline__ void lgkm_wait() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N));
}
template <int N>
__device__ __forceinline__ void vm_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N));
}
// 16-byte buffer load into accumulation registers, as an instruction of its own; its completion is
// awaited with vm_wait.  rsrc: buffer descriptor (base, num_records bytes, raw 32-bit words).
__device__ __forceinline__ void buffer_load_b128_acc(u32x4& dst, const i32x4& rsrc, uint32_t voff,
                                                     uint32_t soff) {
  asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen" : "=a"(dst) : "v"(voff), "s"(rsrc), "s"(soff));
}
// After an explicit wait: the values below are (re)defined here, so nothing reads them earlier.
template <int N>
__device__ __forceinline__ void pin(u32x4 (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}
template <int N>
__device__ __forceinline__ void pin_acc(u32x4 (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+a"(v[i]));
}

// s_waitcnt immediate: at most `vm` vector-memory loads outstanding (6-bit count) and at most `lgkm`
// LDS/scalar operations (expcnt left free).
constexpr int waitcnt_imm(int vm, int lgkm) {
  return (vm & 15) | (((vm >> 4) & 3) << 14) | (7 << 4) | ((lgkm & 15) << 8);
}

// Order-preserving map of float bits to unsigned (for finite values; -0 is canonicalised first).
__device__ __forceinline__ uint32_t ord_bits(float s) {
  const uint32_t u = __float_as_uint(s);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// Inverse of ord_bits.
__device__ __forceinline__ float from_ord_bits(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

// Median of three (v_med3_u32): the middle value, used to maintain a sorted top-3.
__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// DPP patterns that stay inside aligned groups of 2, 4, 8 and 16 lanes.
constexpr int kXor1 = 0xB1;       // quad_perm [1,0,3,2]
constexpr int kXor2 = 0x4E;       // quad_perm [2,3,0,1]
constexpr int kXor3 = 0x1B;       // quad_perm [3,2,1,0]
constexpr int kHalfMirror = 0x141;
constexpr int kMirror = 0x140;

// Maximum of v over the aligned group of G lanes containing this lane.
template <int G>
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v) {
  if constexpr (G >= 2) v = max(v, dpp_u32<kXor1>(v));
  if constexpr (G >= 4) v = max(v, dpp_u32<kXor2>(v));
  if constexpr (G >= 8) v = max(v, dpp_u32<kHalfMirror>(v));
  if constexpr (G >= 16) v = max(v, dpp_u32<kMirror>(v));
  return v;
}

// Merge (m1 >= m2) pairs across the aligned group of g lanes (g a power of two <= 16).
template <int CTRL>
__device__ __forceinline__ void top2_merge_step(float& m1, float& m2) {
  const float o1 = dpp_f32<CTRL>(m1), o2 = dpp_f32<CTRL>(m2);
  const float hi = fmaxf(m1, o1), lo = fminf(m1, o1);
  m2 = fmaxf(lo, fmaxf(m2, o2));
  m1 = hi;
}
__device__ __forceinline__ void top2_group(float& m1, float& m2, int g) {
  if (g >= 2) top2_merge_step<kXor1>(m1, m2);
  if (g >= 4) top2_merge_step<kXor2>(m1, m2);
  if (g >= 8) top2_merge_step<kHalfMirror>(m1, m2);
  if (g >= 16) top2_merge_step<kMirror>(m1, m2);
}

// Rank of this lane's group among the groups of its token (score desc, lower group first), for
// groups that each cover lpg whole lanes of the token's G lanes (lane jl covers experts 32 jl ..
// 32 jl + 31; lanes at or past E hold no group).  Values of the other lanes of the aligned
// G-lane group come in by lane exchange: lanes jl ^ 1..3 through quad permutations, lanes
// jl ^ 4..7 through the half-row mirror (lane jl ^ 7) followed by the same permutations.
// Which lanes jl ^ x lead a group (lead[x]) and whose group comes before this lane's (lower[x]) does
// not depend on the token: computed once, as 0/1 integers kept in vector registers, so the rank is
// plain compare-and-select arithmetic with no branches.
template <int G>
struct RankLanes { int lead[G], lower[G]; };
template <int G>
__device__ __forceinline__ RankLanes<G> rank_lanes(int jl, int lpg, int E) {
  RankLanes<G> r;
  const int me = jl / lpg;
#pragma unroll
  for (int x = 0; x < G; ++x) {
    const int j = jl ^ x;
    r.lead[x] = (x != 0 && (j % lpg) == 0 && j * 32 < E) ? 1 : 0;
    r.lower[x] = (j / lpg < me) ? 1 : 0;
    asm volatile("" : "+v"(r.lead[x]), "+v"(r.lower[x]));
  }
  return r;
}
template <int G>
__device__ __forceinline__ int group_rank(float g, const RankLanes<G>& rl) {
  float v[8];
  v[0] = g;
  if constexpr (G >= 2) v[1] = dpp_f32<kXor1>(g);
  if constexpr (G >= 4) { v[2] = dpp_f32<kXor2>(g); v[3] = dpp_f32<kXor3>(g); }
  if constexpr (G >= 8) {
    const float m = dpp_f32<kHalfMirror>(g);   // lane jl ^ 7
    v[7] = m; v[6] = dpp_f32<kXor1>(m); v[5] = dpp_f32<kXor2>(m); v[4] = dpp_f32<kXor3>(m);
  }
  int rank = 0;
#pragma unroll
  for (int x = 1; x < G; ++x) {
    const float o = v[x];
    const int gt = o > g ? 1 : 0, eq = o == g ? 1 : 0;
    rank += rl.lead[x] & (gt | (eq & rl.lower[x]));
  }
  return rank;
}

// ---- packed router weight --------------------------------------------------------------------
// Stage st (kStageRowBytes of every row) occupies EPAD * kStageRowBytes contiguous bytes.  Inside
// it, the 1 KB chunk c = (we * kNStep + q) * FE + fe holds, for lane l, the 16 bytes of row
// e = we * EW + fe * 32 + (l & 31) at byte st * kStageRowBytes + q * 32 + (l >> 5) * 16 of that row:
// exactly the A-operand fragment wave `we` loads for expert block fe of k-step q.  Rows >= E and
// bytes past H are zero.
template <int EPAD>
__global__ void pack_kernel(const char* __restrict__ w, int32_t E, int32_t Hbytes, int32_t nstages,
                            u32x4* __restrict__ out) {
  using Cfg = TileCfg<EPAD>;
  constexpr int EW = EPAD / Cfg::WE, FE = EW / 32;
  constexpr int kUnitsPerStage = EPAD * (kStageRowBytes / 16);   // 16-byte units
  const int64_t units = (int64_t)nstages * kUnitsPerStage;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < units;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int st = (int)(idx / kUnitsPerStage);
    const int rem = (int)(idx % kUnitsPerStage);
    const int c = rem >> 6, l = rem & 63;
    const int fe = c % FE, q = (c / FE) % kNStep, we = c / (FE * kNStep);
    const int e = we * EW + fe * 32 + (l & 31);
    const int b = st * kStageRowBytes + q * kStepBytes + (l >> 5) * 16;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (e < E && b < Hbytes) v = *reinterpret_cast<const u32x4*>(w + (int64_t)e * Hbytes + b);
    out[idx] = v;
  }
}

// Whether float32 inputs are contracted in parts.  Float32 matrix instructions / parts (us per packed
// call): E = 8, H = 4096, T = 1000 20.9 / 21.9; E = 64, H = 2048, T = 1000 19.6 / 20.4, T = 30000 96.0 /
// 104.8; E = 128, H = 2048, T = 1000 27.2 / 26.0, T = 20000 150.5 / 132.2; E = 256, H = 7168, T = 64
// 43.7 / 35.1, T = 4096 with selections and logits 132 / 106, T = 20000 866 / 463.
constexpr bool parts_pay(int epad) { return epad >= 128; }

// ---- the contraction ---------------------------------------------------------------------------
// acc[fe][ft] += (router weight block fe) x (hidden block ft) over every stage of the tile; the NS
// stage buffers start at ring_lds.  MATH: bf16 inputs, float32 inputs in bf16 parts, or float32 inputs
// on the float32 matrix instructions.  kParts: *odd gets a non-zero lower half when some value is not
// the sum of its parts.
constexpr int kBf16 = 0, kParts = 1, kExact = 2;
template <int MATH, int EPAD, int FE, int FT, int NS, int BM, int TW>
__device__ __forceinline__ void contract(f32x16 (&acc)[FE][FT], const Params& p, int64_t row0,
                                         int wave, int we, int wt, int lane, char* ring_lds,
                                         uint32_t* odd) {
  constexpr int LPW = BM / 4 / kWaves;               // stage load instructions per wave (4 rows each)
  constexpr int UNROLL = kRingW / kNStep;            // one period of the weight ring per iteration
  constexpr int STAGE = BM * kStageRowBytes;         // LDS bytes of one stage buffer
  // counted waits (see the issue order below): loads issued after a stage's own batch by the time
  // the stage must be resident, and the most a wave ever has in flight
  constexpr int kWaitStage = 8 * FE * (NS - 1) + (NS - 2) * LPW;
  // the batch of stage t goes out at the end of stage t - NS, right before the weight slice of
  // k-step kLead + 8 t; the prologue keeps that order for stages 0 .. NS-1
  constexpr int kLead = kNStep - 1 + kRingW - 1 - kNStep * NS;
  static_assert(kLead < 0, "stage 0's batch precedes every weight slice");
  // Batches the prologue issues before any weight slice have fewer loads behind them than the
  // steady-state count assumes; the prologue waits for all of them (they went out together).
  constexpr int kEarly = (-kLead + kNStep - 1) / kNStep;          // stages t with kLead + 8 t < 0
  constexpr int kWaitFirst = (NS - kEarly) * LPW + (kRingW - 1) * FE;
  static_assert(kWaitStage <= 63 && (kRingW - 1) * FE + NS * LPW <= 63,
                "more loads in flight than a wave can count");
  static_assert(LPW >= 1 && BM % (4 * kWaves) == 0, "stage loads split evenly over the waves");
  static_assert(kRingW % kNStep == 0 && kNStep % 4 == 0, "the weight ring holds whole stages, a stage whole pairs of pairs of k-steps");
  const uint32_t lds0 = lds_addr(ring_lds);
  // wave-uniform; readfirstlane keeps them, and the offsets and the descriptor of the weight loads
  // derived from them, in scalar registers
  const int nst = __builtin_amdgcn_readfirstlane(p.nstages);
  const int st_base = __builtin_amdgcn_readfirstlane(p.st_base);
  const int Hb = p.Hbytes;
  const int64_t rows = (p.T - row0) < BM ? (p.T - row0) : BM;

  // hidden rows: rows past T are outside the buffer and read as zero
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(p.x + row0 * (int64_t)p.ldx_bytes), (short)0, (int)(rows * p.ldx_bytes), kRsrcWord3);
  // Load instruction j of this wave fills rows 4 (wave LPW + j) + (lane >> 4); lane l writes the
  // 16-byte slot (l & 15) of its row, which holds logical chunk (l & 15) ^ (row & 15).
  uint32_t voff[LPW];
  int cbyte[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int r = 4 * (wave * LPW + j) + (lane >> 4);
    const int c = (lane & 15) ^ (r & 15);
    voff[j] = (uint32_t)(r * p.ldx_bytes + c * 16);
    cbyte[j] = c * 16;
  }
  // a stage's batch; bytes at or past H (tail of the last stage) and stages past the end are not
  // fetched and land as zeros
  // The counted waits below assume each batch goes out whole, in program order with the weight
  // slices: the scheduling barriers keep other loads from moving into or across it.
  auto load_stage = [&](int bi, int st) {        // bi: stage buffer (wave-uniform)
    const bool live = st < nst;
    const int sb = live ? (st_base + st) * kStageRowBytes : 0;
    const int lim = live ? Hb - sb : 0;           // bytes of the stage inside the row (scalar)
    char* const dst = ring_lds + bi * STAGE + wave * LPW * 1024;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      const uint32_t off = cbyte[j] < lim ? voff[j] : kOobOffset;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr)(dst + j * 1024), 16, off, sb, 0, 2);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // router weight: stage st of the packed layout is EPAD * 256 bytes; this wave's fragment of
  // k-step q and expert block fe is the 1 KB chunk (we * kNStep + q) * FE + fe.  These loads are
  // instructions of their own (into accumulation registers, which the MFMAs read directly) with
  // counted waits: the issue order is fixed, so the count of loads issued after a k-step's slice is
  // known exactly, where the compiler's own tracking turns conservative at the loop head.
  constexpr int kPackStage = EPAD * kStageRowBytes;
  const uint64_t wbase_addr = reinterpret_cast<uint64_t>(p.wpack);
  const i32x4 wr = {__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)wbase_addr),
                    __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(wbase_addr >> 32)),
                    __builtin_amdgcn_readfirstlane(p.st_total * kPackStage), (int32_t)kRsrcWord3};
  const uint32_t wbase = (uint32_t)(we * kNStep * FE * 1024 + lane * 16);
  auto load_w = [&](u32x4(&dst)[FE], int st, int q) {
    const bool ok = st < nst;
#pragma unroll
    for (int fe = 0; fe < FE; ++fe)
      buffer_load_b128_acc(dst[fe], wr, ok ? wbase + (uint32_t)((q * FE + fe) * 1024) : kOobOffset,
                           ok ? (st_base + st) * kPackStage : 0);
  };
  // loads issued after the weight slice of k-step q (of any stage) by the time its MFMAs start: the
  // slices of the next kRingW - 1 k-steps, and the stage batches issued at k-step 7 of the stages
  // in between (two of them, except for q = 6, whose window holds one)
  auto wait_w = [&](int q) {
    if (q == kNStep - 2) vm_wait<(kRingW - 1) * FE + LPW>();
    else vm_wait<(kRingW - 1) * FE + 2 * LPW>();
  };
  static_assert(kRingW - 1 > kNStep && kRingW - 1 < 2 * kNStep, "two stage batches per weight window");

  // hidden fragment of k-step q: token wt TW + ft 32 + (lane & 31), logical chunk 2q + (lane >> 5).
  // These LDS reads are written as instructions of their own, with their waits counted below: the
  // compiler cannot tell a read of one ring buffer from the stage loads still filling another and
  // would otherwise wait for every load in flight before each read.
  uint32_t baddr[kNStep];
#pragma unroll
  for (int q = 0; q < kNStep; ++q)
    baddr[q] = lds0 + (uint32_t)((wt * TW + (lane & 31)) * kStageRowBytes +
                                 (((2 * q + (lane >> 5)) ^ (lane & 15)) * 16));
  auto load_b = [&](u32x4(&dst)[FT], int bi, int q) {
    const uint32_t a = baddr[q] + (uint32_t)(bi * STAGE);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) ds_read_b128(dst[ft], a, ft * 32 * kStageRowBytes);
  };

  // Where float32 inputs always come this way, every other k-pair goes to a second sum, added at the end,
  // so that each is rounded half as often.  Error of the logits against 64 bits, of their norm, one sum /
  // parts / two sums: E = 64, H = 2048 3.9e-7 / 2.4e-7 / 2.0e-7, E = 8, H = 4096 4.0e-7 / 2.3e-7 / 1.9e-7.
  // Time is the same (E = 64, T = 1000 19.6 / 19.7 us with one / two).
  constexpr bool kTwoSums = MATH == kExact && !parts_pay(EPAD);
  f32x16 odd_sum[FE][FT];
  if constexpr (kTwoSums) {
#pragma unroll
    for (int a = 0; a < FE; ++a)
#pragma unroll
      for (int b = 0; b < FT; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) odd_sum[a][b][r] = 0.f;
  }
  auto mma = [&](const u32x4(&a)[FE], const u32x4(&b)[FT]) {
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int fe = 0; fe < FE; ++fe) {
        if constexpr (MATH == kBf16) {
          acc[fe][ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, a[fe]), __builtin_bit_cast(bf16x8, b[ft]), acc[fe][ft], 0, 0, 0);
        } else {
          // four k-pairs per fragment; A and B take the same k for every lane
          const f32x4 av = __builtin_bit_cast(f32x4, a[fe]);
          const f32x4 bv = __builtin_bit_cast(f32x4, b[ft]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            f32x16& to = kTwoSums && (j & 1) ? odd_sum[fe][ft] : acc[fe][ft];
            to = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j], bv[j], to, 0, 0, 0);
          }
        }
      }
  };
  // float32 inputs in parts: every value is the sum of three bf16 parts (the value rounded to bf16, the
  // rest rounded to bf16, what is left), and the product keeps six of the nine part products, on bf16
  // MFMAs with float32 accumulation: the three left out are below 2^-24 of it.  Two k-steps (8 values of
  // a lane) make one fragment; the MFMAs of a pair of k-steps run among the splitting of the next pair,
  // half of them per k-step, so the vector ALU works beside the matrix cores.  The sum is exact unless a
  // value is too large to be rounded to bf16 or so small (below 2^-109) that what is left reaches past
  // bf16's exponents; `left` gathers the bits that the last part leaves out.
  // Bound by vector and matrix instructions in balance (E = 256: 104 and 12 per k-step and wave, 64
  // rows); the six products need 0.38 of the matrix time of v_mfma_f32_32x32x2_f32.  Where the parts
  // serve (see parts_pay), the error against 64 bits on dense rows is smaller (fewer accumulations):
  // 2.4e-7 instead of 2.9e-7 of the logits' norm at H = 512.  On rows with a single non-zero value it is
  // 3.5e-8 instead of 2.5e-8: the bf16 MFMA truncates as it accumulates, and keeping eight products
  // (3.45e-8) would cost 10 to 20% more time.
  struct Parts { u32x4 v[3]; };
  constexpr int kProducts = 6;
  constexpr int kSplitOps = (FE + FT) * 24 + FE * 4;   // vector instructions of a k-step's splitting
  Parts sa[2][FE], sb[2][FT];                    // [parity of the k-step pair]
  uint32_t left = 0;                             // bits of every value that its parts leave out
  if constexpr (MATH == kParts) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
      for (int fe = 0; fe < FE; ++fe) sa[1][fe].v[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) sb[1][ft].v[i] = u32x4{0u, 0u, 0u, 0u};
    }
  }
  // the parts of a lane's four values into dwords 2 half, 2 half + 1 of the fragments
  auto split4 = [&](Parts& out, const u32x4& x, int half) {
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const float a = __uint_as_float(x[2 * w]), b = __uint_as_float(x[2 * w + 1]);
      const uint32_t h = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
      const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xFFFF0000u);
      const uint32_t m = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)ra, (__bf16)rb});
      const uint32_t la = __float_as_uint(ra - __uint_as_float(m << 16));
      const uint32_t lb = __float_as_uint(rb - __uint_as_float(m & 0xFFFF0000u));
      out.v[0][2 * half + w] = h;
      out.v[1][2 * half + w] = m;
      out.v[2][2 * half + w] = __builtin_amdgcn_perm(lb, la, 0x07060302u);   // upper halves
      left = left | la | lb;
    }
  };
  // half of the part products of a pair of k-steps, smallest parts first
  auto mma_parts = [&](const Parts(&a)[FE], const Parts(&b)[FT], int half) {
    constexpr int kI[kProducts] = {2, 0, 1, 1, 0, 0}, kJ[kProducts] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int i = 0; i < kProducts / 2; ++i)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int fe = 0; fe < FE; ++fe)
          acc[fe][ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, a[fe].v[kI[kProducts / 2 * half + i]]),
              __builtin_bit_cast(bf16x8, b[ft].v[kJ[kProducts / 2 * half + i]]), acc[fe][ft], 0, 0, 0);
  };

  // ---- prologue: stages 0 .. NS-1 and k-steps 0 .. kRingW-2 in flight, then stage 0 published.
  // Loads go out in the steady state's order, so every wait at the loop head counts the same loads
  // on both paths into it.
  u32x4 ring[kRingW][FE];
  u32x4 bq[2][FT];
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (kLead + kNStep * t < 0) load_stage(t, t);
#pragma unroll
  for (int g = 0; g < kRingW - 1; ++g) {
#pragma unroll
    for (int t = 0; t < NS; ++t)
      if (kLead + kNStep * t == g) load_stage(t, t);
    load_w(ring[g], g / kNStep, g % kNStep);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (kLead + kNStep * t >= kRingW - 1) load_stage(t, t);
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(kWaitFirst, 0));
  asm volatile("s_barrier" ::: "memory");
  load_b(bq[0], 0, 0);
  __builtin_amdgcn_sched_barrier(0);

  // ---- steady state.  Issue order per stage: k-steps 0..6 each read the next hidden fragments
  // and one weight slice; k-step 7 waits for this wave's share of stage s+1, meets the other waves
  // (after which stage s is no longer read and stage s+1 is complete), refills stage s's buffer
  // with stage s+NS, reads stage s+1's first fragments, then its weight slice.
  int bi = 0;                                   // stage buffer of stage s (= s mod NS)
  for (int s0 = 0; s0 < nst; s0 += UNROLL) {
#pragma unroll
    for (int d = 0; d < UNROLL; ++d) {
      const int s = s0 + d;
      if (s >= nst) break;
      const int bn = bi + 1 == NS ? 0 : bi + 1;   // stage buffer of stage s + 1
#pragma unroll
      for (int q = 0; q < kNStep; ++q) {
        const int slot = (d * kNStep + q) % kRingW;
        if (q + 1 < kNStep) {
          load_b(bq[(q + 1) & 1], bi, q + 1);
        } else {
          // this wave's share of stage s + 1 has landed and its reads of stage s are done; after
          // the barrier every wave's are, so stage s + 1 is complete and stage s's buffer is free
          __builtin_amdgcn_s_waitcnt(waitcnt_imm(kWaitStage, 0));
          asm volatile("s_barrier" ::: "memory");
          load_stage(bi, s + NS);
          load_b(bq[0], bn, 0);
        }
        load_w(ring[(slot + kRingW - 1) % kRingW], s + (q + kRingW - 1) / kNStep, (q + kRingW - 1) % kNStep);
        lgkm_wait<FT>();                        // this k-step's fragments (the next k-step's may be in flight)
        wait_w(q);                              // this k-step's weight slice
        pin(bq[q & 1]);
        pin_acc(ring[slot]);
        if constexpr (MATH != kParts) {
          mma(ring[slot], bq[q & 1]);
        } else {
          const int par = (q >> 1) & 1;
#pragma unroll
          for (int fe = 0; fe < FE; ++fe) split4(sa[par][fe], ring[slot][fe], q & 1);
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) split4(sb[par][ft], bq[q & 1][ft], q & 1);
          mma_parts(sa[par ^ 1], sb[par ^ 1], q & 1);
#pragma unroll
          for (int i = 0; i < kProducts / 2 * FE * FT; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, kSplitOps / (kProducts / 2 * FE * FT), 0);   // its vector share
          }
        }
        // the bits left out are gathered in the k-step they come from, not kept apart until the end
        if constexpr (MATH == kParts) asm volatile("" : "+v"(left));
        // keep every load in the k-step it was written in: the prefetch distances are the design
        __builtin_amdgcn_sched_barrier(0);
      }
      bi = bn;
    }
  }
  // no stage load may still be writing LDS when the tile is reused below, and the fragments fetched past
  // the last stage keep their registers until they have landed
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
#pragma unroll
  for (int i = 0; i < kRingW; ++i) pin_acc(ring[i]);
  pin(bq[0]);
  pin(bq[1]);
  if constexpr (kTwoSums) {
#pragma unroll
    for (int a = 0; a < FE; ++a)
#pragma unroll
      for (int b = 0; b < FT; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] += odd_sum[a][b][r];
  }
  if constexpr (MATH == kParts) {                // the last pair of k-steps
    mma_parts(sa[1], sb[1], 0);
    mma_parts(sa[1], sb[1], 1);
    *odd = left;
  }
}

// Score of one logit without its bias lb (LBIAS: add it; padding experts hold -inf there and in sb).
template <bool SIG, bool LBIAS>
__device__ __forceinline__ float score_of(float logit, float lb, float sb) {
  const float z = LBIAS ? logit + lb : logit;
  if constexpr (SIG) return __builtin_amdgcn_rcpf(1.0f + __expf(-z)) + sb;
  return z + 0.0f;                               // -0 -> +0; padding experts stay -inf
}

// Tokens [slice_begin(i), slice_begin(i + 1)) of a tile are finished by its split i.
__device__ __forceinline__ int slice_begin(int i, int BM, int ks) { return i * BM / ks; }

// Device-scope 16-byte accesses of the partial logits (sc1: past this XCD's L2, so they meet at the
// point every XCD sees).  rsrc: raw buffer descriptor of the tile's partials.
constexpr int kDeviceScope = 16;
__device__ __forceinline__ void partial_store(const __amdgpu_buffer_rsrc_t& rsrc, const f32x4& v,
                                              uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, off, 0, kDeviceScope);
}
__device__ __forceinline__ f32x4 partial_load(const __amdgpu_buffer_rsrc_t& rsrc, uint32_t off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, kDeviceScope));
}

// Arrival word of a tile: arrivals in the low half, given-up slices (one bit per split) in the high.
constexpr uint32_t kArrivalMask = 0xFFFFu;
static_assert(kMaxSplits <= 16, "one given-up bit per split in the arrival word");

// The parts serve a workgroup whose values are all sums of their parts and whose logits are zero or at
// least 2^-100 (below, part products would underflow that a float32 product keeps) and finite.  Any
// other workgroup (infinities and values next to the largest among them, as both parts of such a value
// are infinite or NaN) contracts again on the float32 matrix instructions and has their results (E =
// 256, T = 4096: 116 us, 225 when every workgroup does).
// kLeastLogit: 2^-100, doubled, as bits, less one.
constexpr uint32_t kLeastLogit = (27u << 24) - 1u;

// BM_: tokens per workgroup (the configuration's own, or half of it when that fills the chip better)
// MODE: kFused contracts the whole row and finishes the tile.  Split mode (grid tiles x ks) contracts
// one of ks stage ranges and exchanges partial logits through memory: in kSplit the tile's last split
// to arrive adds them and finishes the tile, in kShare every split finishes its 1/ks of the tokens.
constexpr int kFused = 0, kSplit = 1, kShare = 2;
template <bool BF16, int EPAD, int BM_, int MODE>
__global__ __launch_bounds__(kThreads, 1) void predict_kernel(Params p) {
  using Cfg = TileCfg<EPAD>;
  constexpr int WE = Cfg::WE, WT = Cfg::WT, BM = BM_;
  constexpr int EW = EPAD / WE, TW = BM / WT;
  constexpr int FE = EW / 32, FT = TW / 32;
  constexpr int NS = ring_stages(BM);
  constexpr int STAGE = BM * kStageRowBytes;     // LDS bytes of one hidden stage
  constexpr int SROW = EPAD + 4;                 // score-tile row stride in floats
  constexpr int SCORE_BYTES = BM * SROW * 4;
  constexpr int SMEM = (NS * STAGE > SCORE_BYTES) ? NS * STAGE : SCORE_BYTES;
  constexpr bool SHARE = MODE == kShare;
  constexpr int LPT = EPAD / 32;                 // lanes per token in the selection phase
  constexpr int TPP = kThreads / LPT;            // token slots (lane groups) of the workgroup
  // tokens a lane group works on at once: 1 (interleaving two ran slower on MI355X)
  constexpr int NT = 1;
  constexpr int TPASS = TPP * NT;                // tokens per selection pass
  constexpr int NPASS = (BM + TPASS - 1) / TPASS;
  constexpr int GSC_TOK = TPASS < BM ? TPASS : BM;
  static_assert(WE * WT == kWaves, "every wave owns one tile slice");
  static_assert(EW % 32 == 0 && TW % 32 == 0, "wave tiles are whole 32 x 32 MFMA blocks");
  static_assert(BM % TPASS == 0 || (TPASS > BM && NT == 1 && BM % (64 / LPT) == 0),
                "every selection pass covers whole waves");

  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  __shared__ int32_t hist[EPAD];
  __shared__ __attribute__((aligned(16))) float s_lbias[EPAD];   // router bias (-inf past E)
  __shared__ __attribute__((aligned(16))) float s_sbias[EPAD];   // selection bias (-inf past E)
  // selected experts per token (ids < 256), with spare slots kMaxK .. kMaxK + LPT - 1
  __shared__ int16_t sel[BM][kMaxK + LPT];
  __shared__ uint8_t kmask[BM];                 // kept lanes of each token (second phase)
  __shared__ __attribute__((aligned(16))) float grp[BM][8];   // group scores (8 groups of 32)
  __shared__ __attribute__((aligned(16))) float gsc[GSC_TOK][kMaxGroups];
  __shared__ int32_t s_flag;
  __shared__ uint32_t s_marks;
  __shared__ int32_t s_stray;                     // an expert on a rank that does not exist
  __shared__ int32_t s_redo;                      // float32: the parts do not serve this workgroup's values

  const int tid0 = threadIdx.x;
  const int lane0 = tid0 & 63;
  // wave-uniform by construction; readfirstlane keeps it (and every buffer-load offset derived
  // from it) in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  const int we = wave % WE;
  const int wt = wave / WE;
  const int split_tile = MODE != kFused ? __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (uint32_t)p.ks)) : 0;
  const int tile = MODE != kFused ? (int)p.full + split_tile : (int)blockIdx.x;
  const int split = MODE != kFused ? (int)blockIdx.x - split_tile * p.ks : 0;
  // stages per split
  const int chunk = MODE != kFused ? __builtin_amdgcn_readfirstlane((p.st_total + p.ks - 1) / p.ks) : p.st_total;
  const int64_t row0 = (int64_t)tile * BM;
  const int E = p.E;
  const int polls = p.arrival_polls;               // (kShare)
  for (int i = tid0; i < EPAD; i += kThreads) {
    hist[i] = 0;
    // padding experts get -inf in both, so their score is -inf without a per-element test
    s_lbias[i] = i < E ? (p.logit_bias ? p.logit_bias[i] : 0.f) : -__builtin_inff();
    s_sbias[i] = i < E ? (p.select_bias ? p.select_bias[i] : 0.f) : -__builtin_inff();
  }

  f32x16 acc[FE][FT];
#pragma unroll
  for (int a = 0; a < FE; ++a)
#pragma unroll
    for (int b = 0; b < FT; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  {
    Params q = p;
    if constexpr (MODE != kFused) {
      q.st_base = split * chunk;
      q.nstages = p.st_total - q.st_base < chunk ? p.st_total - q.st_base : chunk;
    }
    const bool any = row0 < p.T && q.nstages > 0;
    if constexpr (BF16 || !parts_pay(EPAD)) {
      if (any)
        contract<BF16 ? kBf16 : kExact, EPAD, FE, FT, NS, BM, TW>(acc, q, row0, wave, we, wt, lane0, smem, nullptr);
    } else {
      if (tid0 == 0) s_redo = 0;
      if (any) {
        uint32_t odd = 0;
        contract<kParts, EPAD, FE, FT, NS, BM, TW>(acc, q, row0, wave, we, wt, lane0, smem, &odd);
        odd &= 0xFFFFu;
        uint32_t least = ~0u;                      // of 2 |logit| - 1 as bits: zeros do not count
        float finite = 0.f;                        // NaN with any logit that is not
#pragma unroll
        for (int a = 0; a < FE; ++a)
#pragma unroll
          for (int b = 0; b < FT; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              least = min(least, (__float_as_uint(acc[a][b][r]) << 1) - 1u);
              finite = fmaf(acc[a][b][r], 0.f, finite);
            }
        if (odd != 0 || least < kLeastLogit || finite != finite) s_redo = 1;
        lds_barrier();
        if (s_redo != 0) {
#pragma unroll
          for (int a = 0; a < FE; ++a)
#pragma unroll
            for (int b = 0; b < FT; ++b)
#pragma unroll
              for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
          contract<kExact, EPAD, FE, FT, NS, BM, TW>(acc, q, row0, wave, we, wt, lane0, smem, nullptr);
          lds_barrier();
        }
      } else {
        lds_barrier();
      }
    }
  }
  if constexpr (BF16 || !parts_pay(EPAD)) lds_barrier();   // (parts: behind the flag above)

  // The contraction of a 128-row tile takes every register.  In its sliced mode the thread's number, and
  // what follows from it, is made again here rather than kept across it (it went to scratch memory, 12
  // bytes per lane for bf16 and 20 for float32, which a first launch may have to set up).
  int fresh = lane0;
  if constexpr (SHARE && BM == 128) {
    fresh = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(fresh));
  }
  const int lane = fresh;
  const int tid = SHARE && BM == 128 ? wave * 64 + lane : tid0;

  float* S = reinterpret_cast<float*>(smem);
  // ---- split mode: exchange the partial logits ------------------------------------------------
  // Partials go to memory with device-scope stores; each thread waits for its own, and the barrier
  // orders them all before the arrival count.  Sums are taken in split order, so results repeat.
  __amdgpu_buffer_rsrc_t pr;
  constexpr int kBlockBytes = BM * EPAD * 4;       // partials of one split
  const int live = (p.st_total + chunk - 1) / chunk;   // splits that hold stages
  uint32_t taken = 1;                              // slices this workgroup finishes, one bit each
  if constexpr (MODE != kFused)
    pr = __builtin_amdgcn_make_buffer_rsrc((void*)(reinterpret_cast<char*>(p.partial) +
                                                   (size_t)split_tile * p.ks * kBlockBytes),
                                           (short)0, p.ks * kBlockBytes, kRsrcWord3);
  if constexpr (MODE == kSplit) {
    // The tile's last split to arrive adds the partials and finishes the whole tile.  16 bytes are four experts of one token, at unit
    // ((fe FT + ft) 4 + g) kThreads + thread; expert blocks past E are skipped.
    auto unit_off = [&](int j, int fe, int ft, int g) {
      return (uint32_t)(j * kBlockBytes + (((fe * FT + ft) * 4 + g) * kThreads + tid) * 16);
    };
    if (split < live) {
#pragma unroll
      for (int fe = 0; fe < FE; ++fe)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (we * EW + fe * 32 + g * 8 < E)
              partial_store(pr, f32x4{acc[fe][ft][g * 4], acc[fe][ft][g * 4 + 1], acc[fe][ft][g * 4 + 2],
                                      acc[fe][ft][g * 4 + 3]}, unit_off(split, fe, ft, g));
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    __syncthreads();
    if (tid == 0) s_flag = atomicAdd(&p.ws_tile[split_tile], 1u) == (uint32_t)p.ks - 1 ? 1 : 0;
    __syncthreads();
    if (s_flag != 1) return;
    taken = (1u << p.ks) - 1u;
    constexpr int kJ = 4;                          // splits whose loads are in flight together
#pragma unroll
    for (int fe = 0; fe < FE; ++fe)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[fe][ft][r] = 0.f;
        for (int j0 = 0; j0 < live; j0 += kJ) {
          f32x4 v[kJ][4];
#pragma unroll
          for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              v[j][g] = j0 + j < live && we * EW + fe * 32 + g * 8 < E
                            ? partial_load(pr, unit_off(j0 + j, fe, ft, g)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fe][ft][r] += v[j][r >> 2][r & 3];
        }
      }
  }
  if constexpr (SHARE) {
    // Every split finishes its own slice of the tile's tokens.  Its partials of that slice go to the
    // score tile in LDS, the others to memory (16 bytes, four experts of one token, at unit
    // (expert / 4) BM + token of its block).  Once every split of the tile has arrived, the slice's
    // partials are added and scored.
    // A workgroup that waits too long for the others (they may still be queued behind another
    // kernel's workgroups) stores its slice as well, marks it as given up and leaves; the tile's last
    // arrival reads the marks with its own count and finishes those slices too.  So no workgroup
    // depends on another one being resident, and the wait always ends.
    const int s0 = slice_begin(split, BM, p.ks), s1 = slice_begin(split + 1, BM, p.ks);
    const uint32_t pbase = (uint32_t)split * kBlockBytes;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const int tl = wt * TW + ft * 32 + (lane & 31);
      const bool own = tl >= s0 && tl < s1;
#pragma unroll
      for (int fe = 0; fe < FE; ++fe)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int e0 = we * EW + fe * 32 + g * 8 + (lane >> 5) * 4;
          const f32x4 v = {acc[fe][ft][g * 4], acc[fe][ft][g * 4 + 1], acc[fe][ft][g * 4 + 2],
                           acc[fe][ft][g * 4 + 3]};
          if (own) *reinterpret_cast<f32x4*>(S + (tl - s0) * SROW + e0) = v;
          else if (split < live && e0 < E)
            partial_store(pr, v, pbase + (uint32_t)((e0 / 4) * BM + tl) * 16u);
        }
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    __syncthreads();
    if (tid == 0) {
      const uint32_t old = atomicAdd(&p.ws_tile[split_tile], 1u);
      int state = 0;                               // 1: every split has arrived
      uint32_t marks = 0;
      if ((old & kArrivalMask) == (uint32_t)p.ks - 1) {
        state = 1;
        marks = old >> 16;
      }
      for (int i = 0; state == 0 && i < polls; ++i) {
        const uint32_t v = __hip_atomic_load(&p.ws_tile[split_tile], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        state = (v & kArrivalMask) == (uint32_t)p.ks ? 1 : 0;
        __builtin_amdgcn_s_sleep(1);
      }
      s_flag = state;
      s_marks = marks;
    }
    __syncthreads();
    if (s_flag == 0) {
      // give the slice up, unless the last split arrived in the meantime
      if (split < live)
        for (int i = tid; i < (s1 - s0) * (EPAD / 4); i += kThreads) {
          const int t = i / (EPAD / 4), c = i % (EPAD / 4);
          if (c * 4 < E)
            partial_store(pr, *reinterpret_cast<const f32x4*>(S + t * SROW + c * 4),
                          pbase + (uint32_t)(c * BM + s0 + t) * 16u);
        }
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
      __syncthreads();
      if (tid == 0)
        s_flag = (atomicOr(&p.ws_tile[split_tile], 0x10000u << split) & kArrivalMask) == (uint32_t)p.ks ? 1 : 0;
      __syncthreads();
      if (s_flag == 0) return;
    }
    taken = s_marks | 1u << split;
  }
  const int tickets = MODE != kFused ? __builtin_popcount(taken) : 1;   // slices finished here
  const int nslices = SHARE ? tickets : 1;         // a tile's one finisher takes it as a whole

  // Group-limited routing where the kept groups fill exactly half of a token's lanes (as with 8
  // groups of 32 keeping 4) finishes in a second selection phase on half the lanes (compact).
  // With exactly 8 groups of 32 the group scores come straight from the score computation
  // (early): each 32-expert block of a wave is one group, split over lanes l and l + 32.
  // (A split's slice is a pass or two of the first phase, so it skips the second.)
  const int ng = p.n_group;
  const int gsz = E / ng;
  const bool compact = !SHARE && NPASS % 2 == 0 && BM % TPASS == 0 && LPT >= 2 && ng > 1 && gsz >= 32 &&
                       p.topk_group * (gsz >> 5) * 2 == LPT;
  const bool early = compact && LPT == 8 && gsz == 32 && ng == 8 && p.kind == FB_SIGMOID &&
                     p.logit_bias == nullptr;

  // ---- logits and scores into an LDS tile S[token][expert] ------------------------
  // Lane l of a 32 x 32 block holds token (l & 31) and experts g * 8 + (l >> 5) * 4 + r in
  // register g * 4 + r.
  // the early logits of four experts of token t; 16 bytes at once where every such group is aligned
  const bool logits16 = (E & 3) == 0 && (reinterpret_cast<uintptr_t>(p.logits) & 15u) == 0;
  auto store_logits = [&](int64_t t, int e0, const f32x4& v) __attribute__((always_inline)) {
    float* to = p.logits + t * E + e0;
    if (logits16) {
      if (e0 < E) *reinterpret_cast<f32x4*>(to) = v;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (e0 + r < E) to[r] = v[r];
    }
  };
  if (!SHARE && row0 < p.T) {
    if (p.logits) {                              // debug output of the early logits
#pragma unroll
      for (int fe = 0; fe < FE; ++fe)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int e0 = we * EW + fe * 32 + g * 8 + (lane >> 5) * 4;
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) {
            const int64_t t = row0 + wt * TW + ft * 32 + (lane & 31);
            if (t < p.T) {
              const f32x4 v = {acc[fe][ft][g * 4], acc[fe][ft][g * 4 + 1], acc[fe][ft][g * 4 + 2],
                               acc[fe][ft][g * 4 + 3]};
              store_logits(t, e0, v + *reinterpret_cast<const f32x4*>(s_lbias + e0));
            }
          }
        }
    }
    // The common case (sigmoid, no logit bias) is its own instantiation: the exponential and
    // the reciprocal dominate this phase, and it then needs only three other operations per
    // score.  A sigmoid score is never -0 (the reciprocal is positive, and +0 + -0 = +0), so only
    // the logits need the -0 -> +0 canonicalisation of the order-preserving key.
    auto emit = [&](auto sig_c, auto lbias_c, auto groups_c) __attribute__((always_inline)) {
      constexpr bool SIG = decltype(sig_c)::value, LBIAS = decltype(lbias_c)::value;
      constexpr bool GROUPS = decltype(groups_c)::value;
      // top two scores of each (expert block, token block) over this lane's 16 of its 32 experts
      float t1[FE][FT], t2[FE][FT];
#pragma unroll
      for (int fe = 0; fe < FE; ++fe)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) { t1[fe][ft] = -__builtin_inff(); t2[fe][ft] = -__builtin_inff(); }
#pragma unroll
      for (int fe = 0; fe < FE; ++fe) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int e0 = we * EW + fe * 32 + g * 8 + (lane >> 5) * 4;
          const f32x4 lb = *reinterpret_cast<const f32x4*>(s_lbias + e0);
          const f32x4 sb = *reinterpret_cast<const f32x4*>(s_sbias + e0);
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) {
            const int tl = wt * TW + ft * 32 + (lane & 31);
            f32x4 sv;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              sv[r] = score_of<SIG, LBIAS>(acc[fe][ft][g * 4 + r], lb[r], sb[r]);
              if constexpr (GROUPS) {
                t2[fe][ft] = __builtin_amdgcn_fmed3f(t1[fe][ft], t2[fe][ft], sv[r]);
                t1[fe][ft] = fmaxf(t1[fe][ft], sv[r]);
              }
            }
            *reinterpret_cast<f32x4*>(S + tl * SROW + e0) = sv;
          }
        }
      }
      if constexpr (GROUPS) {
        // merge with lane l + 32, which holds the block's other 16 experts of the same token: the
        // lane-half swap hands lanes 0..31 the values of lanes 32..63 (the upper half's result is
        // not used)
#pragma unroll
        for (int fe = 0; fe < FE; ++fe)
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) {
            const uint32_t u1 = __float_as_uint(t1[fe][ft]), u2 = __float_as_uint(t2[fe][ft]);
            const float o1 = __uint_as_float(__builtin_amdgcn_permlane32_swap(u1, u1, false, false)[1]);
            const float o2 = __uint_as_float(__builtin_amdgcn_permlane32_swap(u2, u2, false, false)[1]);
            const float m1 = fmaxf(t1[fe][ft], o1);
            const float m2 = fmaxf(fminf(t1[fe][ft], o1), fmaxf(t2[fe][ft], o2));
            if (lane < 32)
              grp[wt * TW + ft * 32 + lane][we * FE + fe] = p.group_topn == 2 ? m1 + m2 : m1;
          }
      }
    };
    using T1 = std::integral_constant<bool, true>;
    using F0 = std::integral_constant<bool, false>;
    if (p.kind == FB_SIGMOID) {
      if (p.logit_bias) emit(T1{}, T1{}, F0{});
      else if (early) emit(T1{}, F0{}, T1{});
      else emit(T1{}, F0{}, F0{});
    } else {
      emit(F0{}, T1{}, F0{});
    }
  }
  lds_barrier();

  // ---- selection: LPT lanes per token, 32 contiguous experts per lane ------------------------
  // Lane jl reads its eight 4-expert chunks starting at chunk jl, which keeps the 16 lanes of a
  // DPP row (two tokens) on distinct LDS banks; element 4q + j of the lane is expert
  // 32 jl + 4 ((q + jl) mod 8) + j.  Tokens past T take part with no selectable expert.  With one
  // wave per SIMD nothing hides latency between waves, so each lane group works on NT tokens at
  // once as independent instruction chains.
  const int k = p.k;
  const int jl = tid % LPT;      // lane within the token group
  const int gslot = tid / LPT;   // token slot within a pass
  const int gshift = __builtin_ctz((unsigned)gsz);   // group sizes below 32 are powers of two
  auto local_of = [&](int i) { return ((((i >> 2) + jl) & 7) << 2) | (i & 3); };  // expert - 32 jl
  const int idx_base = 255 - jl * 32;        // key index bits of element i: idx_base - local_of(i)
  auto read_scores = [&](float(&dst)[32], int tlr) {
    const float* row = S + tlr * SROW + jl * 32;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(row + ((q + jl) & 7) * 4);
      dst[q * 4 + 0] = v[0]; dst[q * 4 + 1] = v[1]; dst[q * 4 + 2] = v[2]; dst[q * 4 + 3] = v[3];
    }
  };
  uint32_t idxb[32];                         // key index bits of each element
#pragma unroll
  for (int i = 0; i < 32; ++i) idxb[i] = (uint32_t)(idx_base - local_of(i));
  const RankLanes<LPT> rlanes = rank_lanes<LPT>(jl, gsz >= 32 ? gsz >> 5 : 1, E);
  // ---- finishing a token: per-lane key caches, k extraction rounds, boundary ties, histogram --
  // G lanes per token; lane jg holds 32 keys; element i of the lane is expert
  // 32 L + 4 ((i / 4 + L) mod 8) + i mod 4 (L = the lane's 32-expert slice).
  auto finish = [&](auto g_c, int jg, int tlu, bool tv, int64_t ttu, const uint32_t(&key)[32],
                    const float(&sv)[32], int L) __attribute__((always_inline)) {
    constexpr int G = decltype(g_c)::value;
    // per-lane cache of the kCache largest keys (descending), refilled by a rescan below the last
    // popped key when it runs dry
    uint32_t c[kCache];
#pragma unroll
    for (int d = 0; d < kCache; ++d) c[d] = 0;
    auto insert = [&](uint32_t v) {
#pragma unroll
      for (int d = kCache - 1; d >= 1; --d) c[d] = umed3(c[d - 1], c[d], v);
      c[0] = max(c[0], v);
    };
#pragma unroll
    for (int i = 0; i < 32; ++i) insert(key[i]);
    uint32_t last = 0xFFFFFFFFu, kth = 0, next = 0;
    // k rounds, each popping the token's largest remaining key.  Rounds are branch-free per lane:
    // the popping lane records the expert in slot r, every other lane writes its own spare slot
    // past kMaxK; a refill runs only when some lane of the wave ran dry, and lanes that did not
    // insert zeros (which leave a sorted cache unchanged).
    for (int r = 0; r < k; ++r) {
      const uint32_t h = c[0];
      const uint32_t m = group_max_u32<G>(h);
      kth = m;
      // m is never 0 here: every lane holds 32 keys and only experts >= 255 can have key 0, so
      // each of the first k <= 32 maxima is a real key with exactly one owner
      const bool mine = h == m;
      sel[tlu][mine ? r : kMaxK + jg] = (int16_t)(255 - (int)(m & 0xFFu));
#pragma unroll
      for (int d = 0; d < kCache - 1; ++d) c[d] = mine ? c[d + 1] : c[d];
      c[kCache - 1] = mine ? 0u : c[kCache - 1];
      last = mine ? m : last;
      // refill below last; a lane with nothing left below it inserts only zeros
      const bool dry = mine && c[0] == 0;
      if (__builtin_amdgcn_ballot_w64(dry) != 0) {   // rare
#pragma unroll
        for (int i = 0; i < 32; ++i) insert(dry && key[i] < last ? key[i] : 0u);
      }
    }
    // the (k+1)-th key, for the boundary test below: nothing is popped
    next = group_max_u32<G>(c[0]);
    const uint32_t tb = kth >> 8;              // score bits of the k-th key
    const bool tie = tv && (next >> 8) != 0 && (next >> 8) == tb;
    if (tie) {
      // Exact path for the boundary only.  Every key whose score bits exceed tb is selected and
      // already in place (the keys were popped in descending order); the remaining slots go to
      // the experts whose score bits equal tb, ranked by the full 64-bit key (all score bits,
      // then the inverted index), which is the exact order.
      int above = 0;
#pragma unroll
      for (int i = 0; i < 32; ++i) above += (key[i] >> 8) > tb;
#pragma unroll
      for (int off = 1; off < G; off <<= 1) above += __shfl_xor(above, off, G);
      uint64_t lastk = ~0ull;
      for (int r = above; r < k; ++r) {
        uint64_t best = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          const uint32_t e = (uint32_t)(L * 32 + (((((i >> 2) + L) & 7) << 2) | (i & 3)));
          const uint64_t kk = ((uint64_t)ord_bits(sv[i] + 0.0f) << 32) | (uint64_t)(0xFFFFFFFFu - e);
          const bool ok = (key[i] >> 8) == tb && kk < lastk && kk > best;
          best = ok ? kk : best;
        }
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {
          const uint64_t o = __shfl_xor(best, off, G);
          best = o > best ? o : best;
        }
        if (best == 0) break;                  // cannot happen: at least two keys share tb
        lastk = best;
        if (jg == 0) sel[tlu][r] = (int16_t)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFu));
      }
    }
    wave_lds_sync();
    if (tv) {
      for (int r = jg; r < k; r += G) {
        const int e = sel[tlu][r];
        if ((unsigned)e < (unsigned)E) atomicAdd(&hist[e], 1);
      }
    }
    // The selections in exact descending score order.  With several lanes per token each places its
    // share of the entries by counting the ones that come before; one lane alone sorts by insertion,
    // which is a chain of LDS reads, k steps of about 0.1 us.  With the
    // logits in 16-byte stores: E = 256, T = 16384, k = 8 92.5 -> 82.5 us with both outputs, E = 128, T
    // = 16000 31.2 -> 28.0.
    // Counting places every entry once only if the scores are ordered: a NaN compares false with every
    // score and would leave slots unwritten, so a token whose entries hold one is sorted by insertion,
    // which permutes whatever it is given.  Every lane that counts sees all k scores.
    bool ordered = G > 1;
    if (p.topk_idx && G > 1 && tv) {
      const int16_t* list = sel[tlu];
      for (int r = jg; r < k; r += G) {
        const int e = list[r];
        const float se = (unsigned)e < (unsigned)E ? S[tlu * SROW + e] : -__builtin_inff();
        int rank = 0;
#pragma unroll 4
        for (int q = 0; q < k; ++q) {
          const int eo = list[q];
          const float so = (unsigned)eo < (unsigned)E ? S[tlu * SROW + eo] : -__builtin_inff();
          rank += (int)(so > se) | ((int)(so == se) & (int)(eo < e));
          ordered &= so == so;
        }
        if (ordered) p.topk_idx[ttu * k + rank] = e;
      }
    }
    if (p.topk_idx && (G == 1 || __builtin_expect(!ordered, 0)) && jg == 0 && tv) {
      int16_t* list = sel[tlu];
#pragma unroll 1
      for (int r = 1; r < k; ++r) {
        const int e = list[r];
        const float se = (unsigned)e < (unsigned)E ? S[tlu * SROW + e] : -__builtin_inff();
        int q = r;
#pragma unroll 1
        while (q > 0) {
          const int eo = list[q - 1];
          const float so = (unsigned)eo < (unsigned)E ? S[tlu * SROW + eo] : -__builtin_inff();
          if (so > se || (so == se && eo < e)) break;
          list[q] = (int16_t)eo;
          --q;
        }
        list[q] = (int16_t)e;
      }
#pragma unroll 1
      for (int r = 0; r < k; ++r) p.topk_idx[ttu * k + r] = list[r];
    }
  };
  // split mode: the sum of the partials of tokens [t0, t0 + nt) and their scores, into rows 0 .. nt - 1
  // of the score tile.  own: the split whose partials those rows already hold, -1 for none.
  auto sum_slice = [&](auto sig_c, auto lbias_c, auto units_c, int t0, int nt, int own) __attribute__((always_inline)) {
    constexpr bool SIG = decltype(sig_c)::value, LBIAS = decltype(lbias_c)::value;
    constexpr int kU = decltype(units_c)::value;   // units per thread and splits per batch of loads
    constexpr int kJ = 16 / kU;
    const int units = nt * (EPAD / 4);
    const float inv_nt = 1.0f / (float)nt;
    for (int i0 = tid; i0 < units; i0 += kU * kThreads) {
      f32x4 sum[kU];
      int t[kU], c[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int i = i0 + u * kThreads;
        c[u] = (int)(((float)i + 0.5f) * inv_nt);  // i / nt: i < 2^14, so the product is exact enough
        t[u] = i - c[u] * nt;
        sum[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      for (int j0 = 0; j0 < live; j0 += kJ) {
        f32x4 v[kU][kJ];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
          for (int j = 0; j < kJ; ++j)
            v[u][j] = partial_load(pr, i0 + u * kThreads < units && c[u] * 4 < E && j0 + j < live && j0 + j != own
                                           ? (uint32_t)((j0 + j) * kBlockBytes) + (uint32_t)(c[u] * BM + t0 + t[u]) * 16u
                                           : kOobOffset);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          f32x4 mine = {0.f, 0.f, 0.f, 0.f};
          if (own >= j0 && own < j0 + kJ && i0 + u * kThreads < units)
            mine = *reinterpret_cast<const f32x4*>(S + t[u] * SROW + c[u] * 4);
#pragma unroll
          for (int j = 0; j < kJ; ++j) sum[u] += j0 + j == own ? mine : v[u][j];
        }
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        if (i0 + u * kThreads >= units) continue;
        const int e0 = c[u] * 4;
        const f32x4 lb = *reinterpret_cast<const f32x4*>(s_lbias + e0);
        const f32x4 sb = *reinterpret_cast<const f32x4*>(s_sbias + e0);
        const int64_t tt = row0 + t0 + t[u];
        if (p.logits && tt < p.T) store_logits(tt, e0, sum[u] + lb);
        f32x4 sv;
#pragma unroll
        for (int r = 0; r < 4; ++r) sv[r] = score_of<SIG, LBIAS>(sum[u][r], lb[r], sb[r]);
        *reinterpret_cast<f32x4*>(S + t[u] * SROW + e0) = sv;
      }
    }
  };
  for (int si = 0; si < nslices; ++si) {
  int t0 = 0, nt = BM;                             // tokens of the tile in rows 0 .. nt - 1 of S
  if constexpr (SHARE) {
    const int own = si == 0 ? split : -1;
    const int sl = si == 0 ? split : __builtin_ctz(taken);
    taken &= ~(1u << sl);
    t0 = slice_begin(sl, BM, p.ks);
    nt = slice_begin(sl + 1, BM, p.ks) - t0;
    using T1 = std::integral_constant<bool, true>;
    using F0 = std::integral_constant<bool, false>;
    // the smaller the slice, the more splits share the tile: all of them in one or two batches of loads
    using U4 = std::integral_constant<int, 4>;
    using U2 = std::integral_constant<int, 2>;
    using U1 = std::integral_constant<int, 1>;
    auto sum_by = [&](auto sig_c, auto lbias_c) __attribute__((always_inline)) {
      if (nt * (EPAD / 4) <= kThreads) sum_slice(sig_c, lbias_c, U1{}, t0, nt, own);
      else if (nt * (EPAD / 4) <= 2 * kThreads) sum_slice(sig_c, lbias_c, U2{}, t0, nt, own);
      else sum_slice(sig_c, lbias_c, U4{}, t0, nt, own);
    };
    if (p.kind == FB_SIGMOID) {
      if (p.logit_bias) sum_by(T1{}, T1{});
      else sum_by(T1{}, F0{});
    } else {
      sum_by(F0{}, T1{});
    }
    lds_barrier();
  }
  const int npass = SHARE ? (nt + TPASS - 1) / TPASS : NPASS;
  // each pass's scores are read while the previous pass is processed
  float snext[NT][32];
  if (!early) {
#pragma unroll
  for (int u = 0; u < NT; ++u)
    if (u * TPP + gslot < BM) read_scores(snext[u], u * TPP + gslot);
#pragma unroll 1
  for (int pass = 0; pass < npass; ++pass) {
    if (pass * TPASS + (gslot & ~(64 / LPT - 1)) >= nt) continue;  // whole waves
    int tl[NT];
    int64_t tt[NT];
    bool tvalid[NT];
    float s[NT][32];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      tl[u] = pass * TPASS + u * TPP + gslot;
      tt[u] = row0 + t0 + tl[u];
      tvalid[u] = tt[u] < p.T && (!SHARE || tl[u] < nt);
#pragma unroll
      for (int i = 0; i < 32; ++i) s[u][i] = snext[u][i];
      if (tl[u] + TPASS < BM) read_scores(snext[u], tl[u] + TPASS);
    }
    uint32_t ob[NT][32];                       // order-preserving bits of the scores
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int i = 0; i < 32; ++i) ob[u][i] = ord_bits(s[u][i]);
    uint32_t keep[NT];                         // bit i: element i survives the group limit
#pragma unroll
    for (int u = 0; u < NT; ++u) keep[u] = 0xFFFFFFFFu;
    if (ng > 1) {
      // group scores: sum of the group's group_topn best scores, largest first
      if (gsz >= 32) {
        // whole lanes per group: group scores and ranks stay in registers (lane exchanges inside
        // the token's LPT lanes); the else branch handles groups smaller than a lane's slice
        const int lpg = gsz >> 5;
        const bool real = jl * 32 < E;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          // top two of the lane's scores, compared as order-preserving integers (no NaN handling
          // needed: scores are finite or -inf), then merged over the group's lanes
          uint32_t k1 = 0, k2 = 0;
#pragma unroll
          for (int i = 0; i < 32; ++i) {
            k2 = umed3(k1, k2, ob[u][i]);
            k1 = max(k1, ob[u][i]);
          }
          float m1 = from_ord_bits(k1), m2 = from_ord_bits(k2);
          if (lpg > 1) top2_group(m1, m2, lpg);
          const float g = p.group_topn == 2 ? m1 + m2 : m1;
          const int rank = group_rank<LPT>(g, rlanes);
          keep[u] = (real && rank < p.topk_group) ? 0xFFFFFFFFu : 0u;
        }
      } else {
        const int gpl = 32 >> gshift;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          float* gs = gsc[u * TPP + gslot];
          for (int v = 0; v < gpl; ++v) {
            float m1 = -__builtin_inff(), m2 = -__builtin_inff();
#pragma unroll
            for (int i = 0; i < 32; ++i) {
              const bool in = (local_of(i) >> gshift) == v;
              m2 = in ? __builtin_amdgcn_fmed3f(m1, m2, s[u][i]) : m2;
              m1 = in ? fmaxf(m1, s[u][i]) : m1;
            }
            if (jl * 32 + v * gsz < E) gs[jl * gpl + v] = p.group_topn == 2 ? m1 + m2 : m1;
          }
        }
        wave_lds_sync();
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          const float* gs = gsc[u * TPP + gslot];
          // rank of a group among all groups (score desc, lower index first), four scores per read
          // (rows hold kMaxGroups entries, so the reads stay in bounds)
          auto kept = [&](int g) -> bool {
            const float mine = gs[g];
            int rank = 0;
#pragma unroll 1
            for (int h4 = 0; h4 < ng; h4 += 4) {
              const f32x4 o = *reinterpret_cast<const f32x4*>(gs + h4);
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const int h = h4 + j;
                rank += (h < ng) & ((o[j] > mine) | ((o[j] == mine) & (h < g)));
              }
            }
            return rank < p.topk_group;
          };
          keep[u] = 0;
          for (int v = 0; v < gpl; ++v) {
            if (jl * 32 + v * gsz < E && kept(jl * gpl + v)) {
#pragma unroll
              for (int i = 0; i < 32; ++i) keep[u] |= (uint32_t)((local_of(i) >> gshift) == v) << i;
            }
          }
        }
      }
    }
    // 32-bit keys: the top 24 bits of the order-preserving score encoding, then 255 - expert.
    // Experts outside the kept groups (and every expert of a token past T) keep only their index
    // bits, which ranks them below every selectable expert; padding experts score -inf.
    if (compact) {
      // Only the kept groups matter from here on, and they fill exactly half of the token's lanes:
      // record which lanes they are and finish the token in the second phase below, two tokens
      // per lane group.
      const uint64_t b = __builtin_amdgcn_ballot_w64(keep[0] != 0);
      if (jl == 0) kmask[tl[0]] = (uint8_t)((b >> (lane & (64 - LPT))) & ((1u << LPT) - 1u));
      continue;
    }
    uint32_t key[32];
    if (ng == 1 || gsz >= 32) {                // the lane's experts are kept or dropped together
      const uint32_t m = tvalid[0] && keep[0] ? 0xFFFFFF00u : 0u;
#pragma unroll
      for (int i = 0; i < 32; ++i) key[i] = (ob[0][i] & m) | idxb[i];
    } else {
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const uint32_t m = tvalid[0] && ((keep[0] >> i) & 1u) ? 0xFFFFFF00u : 0u;
        key[i] = (ob[0][i] & m) | idxb[i];
      }
    }
    finish(std::integral_constant<int, LPT>{}, jl, tl[0], tvalid[0], tt[0], key, s[0], jl);
  }
  }
  if (compact) {
    // Second phase: the lane group of a token slot takes two tokens of this wave, half of its
    // lanes each; lane jb of a half reads the jb-th kept group's 32 scores back from the tile.
    constexpr int G2 = LPT / 2;
    wave_lds_sync();
    const int half = jl / G2, jb = jl % G2;
#pragma unroll 1
    for (int pb = 0; pb < NPASS / 2; ++pb) {
      const int tlc = (2 * pb + half) * TPASS + gslot;
      const int64_t ttc = row0 + tlc;
      const bool tvc = ttc < p.T;
      // the jb-th set bit of the token's kept-lane mask
      uint32_t km;
      if (early) {
        // rank groups jb and jb + 4 of the token's 8 (score desc, lower group first), then
        // gather the kept set over the half's four lanes
        const f32x4 ga = *reinterpret_cast<const f32x4*>(&grp[tlc][0]);
        const f32x4 gb = *reinterpret_cast<const f32x4*>(&grp[tlc][4]);
        const float gv[8] = {ga[0], ga[1], ga[2], ga[3], gb[0], gb[1], gb[2], gb[3]};
        uint32_t kb = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int gi = jb + 4 * h;
          const float mine = h ? gv[jb + 4] : gv[jb];
          int rank = 0;
#pragma unroll
          for (int x = 0; x < 8; ++x)
            rank += (int)(gv[x] > mine) | ((int)(gv[x] == mine) & (int)(x < gi));
          kb |= (uint32_t)(rank < p.topk_group) << gi;
        }
        kb |= (uint32_t)__shfl_xor((int)kb, 1, G2);
        kb |= (uint32_t)__shfl_xor((int)kb, 2, G2);
        km = kb;
      } else {
        km = kmask[tlc];
      }
      int L = 0, seen = 0;
#pragma unroll
      for (int b = 0; b < LPT; ++b) {
        const int on = (km >> b) & 1;
        L = (on && seen == jb) ? b : L;
        seen += on;
      }
      float sc[32];
      const float* row = S + tlc * SROW + L * 32;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + ((q + L) & 7) * 4);
        sc[q * 4 + 0] = v[0]; sc[q * 4 + 1] = v[1]; sc[q * 4 + 2] = v[2]; sc[q * 4 + 3] = v[3];
      }
      const uint32_t m = tvc ? 0xFFFFFF00u : 0u;
      uint32_t key[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const int loc = ((((i >> 2) + L) & 7) << 2) | (i & 3);
        key[i] = (ord_bits(sc[i]) & m) | (uint32_t)(255 - (L * 32 + loc));
      }
      finish(std::integral_constant<int, G2>{}, jb, tlc, tvc, ttc, key, sc, L);
    }
  }
  lds_barrier();
  }

  // ---- one global atomic per expert per workgroup, then the completion ticket ----------------
  // Workgroups exchange data only through device-scope atomics, which are coherent across the
  // XCDs' L2 caches without a fence.  Each thread waits for the pre-op values of its counter
  // updates (so they have been performed) before the barrier; only then does thread 0 take the
  // ticket.  The workgroup that takes the last ticket therefore reads complete counters with its
  // own atomics.  This avoids an agent-scope fence per workgroup, which on gfx950 writes back and
  // invalidates the whole L2 and serialises across the workgroups.
  // The tables that the last workgroup needs do not depend on the counts: every workgroup fetches
  // them here, under the latency of its counter updates (E <= 256: thread e has expert e).
  static_assert(EPAD <= kThreads, "one expert per thread");
  constexpr int kPre = (wave_cap(1, 2) + kThreads - 1) / kThreads;   // R * S <= 704
  const bool has_plan = p.plan_cpl != 0;
  const int rs_plan = has_plan ? p.plan.R * p.plan.S : 0;
  const bool timed = has_plan && p.plan.timed;
  int32_t pre[kPre];
#pragma unroll
  for (int i = 0; i < kPre; ++i) {
    const int c = tid + i * kThreads;
    pre[i] = c < rs_plan ? p.plan.slot_expert[c] : -1;
  }
  const int my_rank = tid < E ? p.e2r[tid] : 0;
  const int64_t my_bytes = timed && tid < E ? p.plan.expert_bytes[tid] : 0;
  const int32_t my_node = timed && tid < p.plan.R ? p.plan.rank_node[tid] : 0;
  int done = 0;
  if (tid < E) {
    const int v = hist[tid];
    if (v) done = atomicAdd(&p.ws_acc[tid], v);
  }
  if (done < 0) s_flag = -1;                   // never true (counters stay below 2^31); uses the values
  __syncthreads();
  if (tid == 0) s_flag = (atomicAdd(p.ws_ticket, (uint32_t)tickets) == p.tickets - (uint32_t)tickets) ? 1 : 0;
  __syncthreads();
  if (s_flag != 1) return;

  // ---- last workgroup: counts, rank fold, max/mean; leaves the workspace zeroed -------------
  // A chain of latencies on the critical path of every pass, so nothing waits that need not: the
  // planner's tables are checked and laid out while the counters are on their way, the barrier that
  // publishes the counts starts the planner in wave 0, and wave 1 writes the fold beside it.
  const int total = tid < E ? atomicExch(&p.ws_acc[tid], 0) : 0;
  if (tid == 0) atomicExch(p.ws_ticket, 0u);
  // every workgroup is past its wait once the last ticket is taken: the arrival words go back to zero
  if constexpr (MODE != kFused) {
    uint32_t per_tile = (uint32_t)p.ks;
    if constexpr (SHARE && BM == 128) asm volatile("" : "+s"(per_tile));   // (its reciprocal was kept, too)
    for (int i = tid; i < (int)((p.tickets - p.full) / per_tile); i += kThreads) atomicExch(&p.ws_tile[i], 0u);
  }
  constexpr size_t kPlanLds = (plan_wave_lds_bytes(wave_cap(1, 2), 1) + 15) / 16 * 16;
  static_assert(SMEM >= kPlanLds + FB_MAX_RANKS * 4, "the planner's tables and the rank loads fit");
  const PlanWaveLds pl = plan_wave_lds(smem, wave_cap(1, 2), 1);
  int32_t* rl = reinterpret_cast<int32_t*>(smem + kPlanLds);
  for (int r = tid; r < p.R; r += kThreads) rl[r] = 0;
  if (tid == 0) { s_stray = 0; *pl.state = 0; }
  if (has_plan) {
    if (tid < E) pl.reps[tid] = 0;
    if (tid < 64) { pl.load[tid] = 0; pl.part[tid] = 0; }
  }
  lds_barrier();
  if (has_plan) {
    // a plain placement holds every expert once; a replica (a value >= E) leaves the table to the
    // planner's full check
    int state = 0;
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
      const int c = tid + i * kThreads;
      if (c >= rs_plan) break;
      const int v = pre[i];
      pl.vals[c] = v;
      if (v < -1) state |= kPlanBad;
      else if (v >= E) state |= kPlanReplicas;
      else if (v >= 0) { atomicAdd(&pl.reps[v], 1); pl.base[v] = c; }
      else pl.slot[c] = make_uint2((uint32_t)(E + c), 0u);
    }
    if (timed && tid < E) {
      pl.ebytes[tid] = my_bytes;
      if (my_bytes < 0 || my_bytes > kCostLimit) state |= kPlanBad;
    }
    lds_barrier();
    if (tid < E) {
      pl.cnt[tid] = total;
      if (pl.reps[tid] != 1) state |= kPlanNotOnce;
      else {                                   // base holds a slot of the table, whatever else is wrong
        const int c = pl.base[tid];
        pl.slot[c] = make_uint2((uint32_t)tid, (uint32_t)total);
        atomicAdd(&pl.load[c / p.plan.S], (unsigned long long)(int64_t)total);
      }
      if (total < 0) state |= kPlanBad;
    }
    if (state) atomicOr(pl.state, state);
  }
  if (tid < E) {
    p.counts[tid] = total;
    if (my_rank >= 0 && my_rank < p.R) atomicAdd(&rl[my_rank], total);
    else s_stray = 1;
  }
  lds_barrier();
  if (wave == 1) {
    int64_t mx = 0, sum = 0;
    for (int r = lane; r < p.R; r += 64) {
      const int v = rl[r];
      p.rank_loads[r] = v;
      mx = v > mx ? v : mx;
      sum += v;
    }
    for (int off = 32; off > 0; off >>= 1) {
      const int64_t om = __shfl_xor(mx, off), os = __shfl_xor(sum, off);
      mx = om > mx ? om : mx;
      sum += os;
    }
    if (lane == 0) {
      const double ratio = sum == 0 ? 1.0 : (double)mx * (double)p.R / (double)sum;
      *p.max_mean = s_stray ? -1.0 : ratio;
    }
  }
  if (has_plan && wave == 0) {
    // The swap plan of the counts (Alg. 1, frontier mode): the one-wave planner in this workgroup's
    // first wave, in LDS the selection no longer needs, with its tables already there.
    if (p.plan_cpl == 1) plan_wave_body<1, 1, true>(lane, p.plan, pl, my_node);
    else plan_wave_body<1, 2, true>(lane, p.plan, pl, my_node);
  }
}

__global__ void zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

int epad_of(int32_t E) {
  return E <= 32 ? 32 : E <= 64 ? 64 : E <= 128 ? 128 : 256;
}

// Split mode: when `tiles` workgroups would occupy at most half of the CUs, the stage range of every
// tile is split over several workgroups, so that more CUs stream the hidden rows and each streams a
// share of the router weight.  `room`: bytes for the partials.
//   * At least four stages per split (two where 16 splits are allowed): below that the first loads'
//     latency is most of a split's time (E = 128, H = 2048, T = 1000: 19.8 us with 2 splits of 4
//     stages, 23.0 us with 4 of 2).
//   * Up to 8 splits, 16 for at most four 256-expert tiles.  E = 256, H = 7168, per pass with its
//     plan, 4 / 8 / 16 splits: T = 64 39.1 / 33.5 / 31.7 us, T = 192 38.6 / 34.0 / 32.4, T = 500
//     38.5 / 34.4 / 35.5.
//   * bf16 256-expert tiles of 64 tokens take more than 4 splits only with 32 stages or more and at most
//     0.4 tiles per stage: the more workgroups there are, each writing and reading 64 KB of partials at
//     the same time, the more the exchange costs, and the fewer stages, the less a shorter contraction
//     saves.  Without a plan, 4 splits / as many as the CUs take (us): H = 7168 (56 stages), T = 1344 (21
//     tiles) 30.7 / 30.3, T = 1600 (25) 31.1 / 32.2, T = 2048 (32) 32.2 / 37.5, T = 3200 (50) 35.9 /
//     39.4; H = 4096 (32), T = 704 (11) 24.3 / 22.8, T = 1088 (17) 24.9 / 25.7, T = 2048 27.5 / 34.0; H =
//     3072 (24), T = 300 (5) 21.4 / 22.2.  float32 contracts longer: H = 7168, T = 2048 89.2 / 69.3.
int split_count(int64_t tiles, int BM, int epad, bool bf16, int st_total, int num_cus, size_t room) {
  // at most half of the CUs hold tiles, and each tile has an arrival word
  if (tiles <= 0 || tiles * 2 > num_cus || tiles > kMaxSplitTiles) return 1;
  const bool few = epad == 256 && tiles <= 4 && st_total >= 2 * kMaxSplits;
  int64_t ks = num_cus / tiles;
  const bool crowded = epad == 256 && bf16 && BM < kMaxTileRows && (st_total < 32 || tiles * 5 > st_total * 2);
  const int cap = crowded ? 4 : 8;
  const int64_t most = few ? kMaxSplits : st_total / 4 < cap ? st_total / 4 : cap;
  if (ks > most) ks = most;
  const size_t per_split = (size_t)tiles * BM * epad * sizeof(float);
  if ((size_t)ks * per_split > room) ks = (int64_t)(room / per_split);
  return ks > 1 ? (int)ks : 1;
}

// Whether every split finishes a slice of its tile.  Worth it where the tile's selection and outputs
// take longer than the exchange: 256 experts in at least four slices.  The last split finishing the
// whole tile instead / slices (us per pass with its plan): E = 256, H = 7168, T = 4096 in 4 splits
// 46.9 / 46.5 (float32 with selections and logits written 142 / 133), T = 6000 in 2 splits 55.8 /
// 57.4; E = 128, H = 2048, T = 4000 in 2 splits 24.2 / 28.2; E = 64, T = 3000 19.1 / 23.6.  Nor for many
// bf16 tiles of few stages without debug outputs, where the exchange is most of what is left (no plan,
// us): H = 4096 (32 stages), T = 2500 (40 tiles) 28.3 / 28.0, T = 3500 (55) 29.3 / 30.8, T = 4096 (64)
// 30.1 / 32.8, with both outputs 34.9 / 34.5; H = 7168 (56), T = 3500 36.6 / 36.4.
constexpr bool can_share(int epad) { return epad == 256; }
bool shares(int epad, int ks, int64_t tiles, int st_total, bool bf16, bool outputs) {
  return can_share(epad) && ks >= 4 && (outputs || !bf16 || tiles <= 48 || st_total >= 48);
}

// Tiles of a batch: tile height, tiles, how many of them are contracted whole, and the splits of the
// ones after those (1: there are none).
struct BatchShape {
  int bm;
  int64_t tiles, full;
  int ks;
};

BatchShape shape_with(int bm, int epad, bool bf16, int64_t T, int st_total, int num_cus, size_t room) {
  BatchShape s{bm, (T + bm - 1) / bm, 0, 1};
  if (s.tiles <= num_cus) {
    s.ks = split_count(s.tiles, bm, epad, bf16, st_total, num_cus, room);
  } else if (can_share(epad)) {
    // A 256-expert tile takes a CU (LDS and registers), so the tiles past a whole number of rounds
    // would be a round of their own on a few CUs: they follow as a launch in split mode instead, and
    // both launches add to the same counters and tickets.  E = 256, H = 7168, with the plan, round of
    // their own / split launch: T = 33000 214 / 154 us, T = 36000 220 / 167, T = 40000 223 / 181, T =
    // 48000 (two splits) 229 / 210.  One kernel with both kinds of workgroups saved the second launch
    // but ran its whole tiles 8% slower (117 instead of 108 us to the end of the contraction).
    s.ks = split_count(s.tiles % num_cus, bm, epad, bf16, st_total, num_cus, room);
    s.full = s.tiles - s.tiles % num_cus;
  }
  if (s.ks == 1) s.full = s.tiles;
  return s;
}

// Shape of a batch of T tokens with rows of st_total stages and `room` bytes for partials.
template <int EPAD>
BatchShape batch_shape(int64_t T, bool bf16, int st_total, int num_cus, size_t room) {
  constexpr int BM = TileCfg<EPAD>::BM;
  static_assert(BM <= kMaxTileRows && EPAD <= FB_MAX_EXPERTS, "a split's partials stay within the bound of the scratch");
  if constexpr (EPAD == 256) {
    // Half-height tiles when the full-height grid would leave CUs idle and the half-height one still
    // fits in a single round of workgroups: every CU then streams the weight for fewer tokens.
    const BatchShape h = shape_with(BM / 2, EPAD, bf16, T, st_total, num_cus, room);
    if (T > 0 && h.tiles <= num_cus) return h;
  }
  return shape_with(BM, EPAD, bf16, T, st_total, num_cus, room);
}

template <int EPAD>
size_t split_bytes_cfg(int64_t T, int32_t H, int32_t dtype, int num_cus) {
  const int st_total = (H * (dtype == FB_BF16 ? 2 : 4) + kStageRowBytes - 1) / kStageRowBytes;
  const BatchShape s = batch_shape<EPAD>(T, dtype == FB_BF16, st_total, num_cus, SIZE_MAX);
  return (size_t)(s.tiles - s.full) * s.ks * s.bm * EPAD * sizeof(float);
}

template <int EPAD>
int launch_pack_cfg(const void* w, int32_t E, int32_t Hbytes, void* out, void* stream) {
  const int32_t nst = (Hbytes + kStageRowBytes - 1) / kStageRowBytes;
  const int64_t units = (int64_t)nst * EPAD * (kStageRowBytes / 16);
  const int64_t blocks64 = (units + 255) / 256;
  const int blocks = (int)(blocks64 < 4096 ? (blocks64 > 0 ? blocks64 : 1) : 4096);
  hipLaunchKernelGGL((pack_kernel<EPAD>), dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<const char*>(w), E, Hbytes, nst, static_cast<u32x4*>(out));
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

template <bool BF16, int EPAD, int BM>
int launch_cfg_bm(const PredictLaunch& a, const BatchShape& shape) {
  const int elem = BF16 ? 2 : 4;
  Params p;
  p.x = static_cast<const char*>(a.hidden);
  p.T = a.T;
  p.Hbytes = a.H * elem;
  p.ldx_bytes = (int32_t)(a.ld_hidden * elem);
  p.wpack = static_cast<const char*>(a.router_packed);
  p.E = a.E;
  p.logit_bias = a.logit_bias;
  p.select_bias = a.select_bias;
  p.kind = a.scoring.kind;
  p.k = a.scoring.k;
  p.n_group = a.scoring.n_group;
  p.topk_group = a.scoring.topk_group;
  p.group_topn = a.scoring.group_topn;
  p.e2r = a.expert_to_rank;
  p.R = a.R;
  p.counts = a.counts;
  p.rank_loads = a.rank_loads;
  p.max_mean = a.max_mean;
  p.ws_acc = reinterpret_cast<int32_t*>(static_cast<char*>(a.workspace) + kWsAccOffset);
  p.ws_ticket = reinterpret_cast<uint32_t*>(static_cast<char*>(a.workspace) + kWsTicketOffset);
  p.ws_tile = reinterpret_cast<uint32_t*>(static_cast<char*>(a.workspace) + kWsTileTicketOffset);
  p.topk_idx = a.topk_idx;
  p.logits = a.logits;
  const int64_t split_blocks = (shape.tiles - shape.full) * shape.ks;
  const int64_t full_blocks = shape.tiles > 0 ? shape.full : 1;
  p.full = (uint32_t)shape.full;
  p.tickets = (uint32_t)(full_blocks + split_blocks);
  p.st_total = (p.Hbytes + kStageRowBytes - 1) / kStageRowBytes;
  p.nstages = p.st_total;
  p.st_base = 0;
  p.ks = shape.ks;
  p.arrival_polls = a.arrival_polls;
  p.partial = a.partial;
  p.plan_cpl = 0;
  if (a.plan != nullptr) {
    p.plan = *a.plan;
    p.plan_cpl = (int64_t)a.plan->S * a.plan->S <= 64 ? 1 : 2;
  }
  hipStream_t st = static_cast<hipStream_t>(a.stream);
  const dim3 block(kThreads), split_grid((unsigned)split_blocks);
  const bool share = shares(EPAD, p.ks, shape.tiles, p.st_total, BF16, p.topk_idx != nullptr || p.logits != nullptr);
  if (full_blocks > 0)
    hipLaunchKernelGGL((predict_kernel<BF16, EPAD, BM, kFused>), dim3((unsigned)full_blocks), block, 0, st, p);
  if (split_blocks > 0) {
    if constexpr (can_share(EPAD)) {
      // (full-height tiles split only past whole rounds)
      if (share || BM == TileCfg<EPAD>::BM)
        hipLaunchKernelGGL((predict_kernel<BF16, EPAD, BM, kShare>), split_grid, block, 0, st, p);
    }
    if constexpr (!can_share(EPAD) || BM != TileCfg<EPAD>::BM) {
      if (!share)
        hipLaunchKernelGGL((predict_kernel<BF16, EPAD, BM, kSplit>), split_grid, block, 0, st, p);
    }
  }
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

template <bool BF16, int EPAD>
int launch_cfg(const PredictLaunch& a) {
  constexpr int BM = TileCfg<EPAD>::BM;
  const int st_total = (a.H * (BF16 ? 2 : 4) + kStageRowBytes - 1) / kStageRowBytes;
  const BatchShape s = batch_shape<EPAD>(a.T, BF16, st_total, a.num_cus, a.partial != nullptr ? a.partial_bytes : 0);
  if constexpr (EPAD == 256) {
    if (s.bm == BM / 2) return launch_cfg_bm<BF16, EPAD, BM / 2>(a, s);
  }
  return launch_cfg_bm<BF16, EPAD, BM>(a, s);
}

template <bool BF16>
int launch_dtype(const PredictLaunch& a) {
  switch (epad_of(a.E)) {
    case 32: return launch_cfg<BF16, 32>(a);
    case 64: return launch_cfg<BF16, 64>(a);
    case 128: return launch_cfg<BF16, 128>(a);
    default: return launch_cfg<BF16, 256>(a);
  }
}

}  // namespace

size_t router_packed_bytes(int32_t E, int32_t H, int32_t dtype) {
  const int64_t Hbytes = (int64_t)H * (dtype == FB_BF16 ? 2 : 4);
  const int64_t nst = (Hbytes + kStageRowBytes - 1) / kStageRowBytes;
  return (size_t)(nst * epad_of(E) * kStageRowBytes);
}

int launch_pack(const void* router_w, int32_t E, int32_t H, int32_t dtype, void* packed, void* stream) {
  (void)hipGetLastError();
  const int32_t Hbytes = H * (dtype == FB_BF16 ? 2 : 4);
  switch (epad_of(E)) {
    case 32: return launch_pack_cfg<32>(router_w, E, Hbytes, packed, stream);
    case 64: return launch_pack_cfg<64>(router_w, E, Hbytes, packed, stream);
    case 128: return launch_pack_cfg<128>(router_w, E, Hbytes, packed, stream);
    default: return launch_pack_cfg<256>(router_w, E, Hbytes, packed, stream);
  }
}

size_t split_workspace_bytes(int64_t T, int32_t E, int32_t H, int32_t dtype, int num_cus) {
  switch (epad_of(E)) {
    case 32: return split_bytes_cfg<32>(T, H, dtype, num_cus);
    case 64: return split_bytes_cfg<64>(T, H, dtype, num_cus);
    case 128: return split_bytes_cfg<128>(T, H, dtype, num_cus);
    default: return split_bytes_cfg<256>(T, H, dtype, num_cus);
  }
}

int launch_predict(const PredictLaunch& a) {
  (void)hipGetLastError();
  return a.dtype == FB_BF16 ? launch_dtype<true>(a) : launch_dtype<false>(a);
}

int launch_workspace_zero(void* workspace, size_t bytes, void* stream) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<uint32_t*>(workspace), bytes / 4);
  return hipGetLastError() == hipSuccess ? FB_OK : FB_EDEVICE;
}

// ---- scratch of the no-allocation entry point ----------------------------------------------------
// fb_predict_load_packed_noalloc runs the kernels above with this array as its workspace.  In host
// code its name is not a device address: the address of each device's copy comes from
// hipGetSymbolAddress and is kept per device.
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxScratchDevices];
}  // namespace

int noalloc_scratch(void** ptr, void* stream) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
    (void)hipGetLastError();
    return FB_EDEVICE;
  }
  if (dev >= kMaxScratchDevices) return FB_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_addr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return FB_EDEVICE;
    }
    // The header (accumulators and ticket) must start at zero; every completed call leaves it
    // zeroed again.  A fill kernel rather than a memset node, so a first call made under graph
    // capture stays valid on every replay.
    const int zc = launch_workspace_zero(p, kWsBytes, stream);
    if (zc != FB_OK) return zc;
    g_scratch_addr[dev] = p;
  }
  *ptr = g_scratch_addr[dev];
  return FB_OK;
}

}  // namespace fb
