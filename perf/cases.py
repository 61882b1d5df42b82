"""The work that users of this library have it do, as measurable cases.

Every case goes through the public Python entry points.  Three kinds of work:

  pass     the early pass of one MoE layer: Predictor.predict_plan on a batch of hidden states with a
           router packed at load time (prediction, histogram, fold and swap plan in one call), under a
           swap-count or a time budget; or Predictor.predict_load with its selections and logits, as a
           program does that reuses the early routing.
  study    the prediction-quality study of one layer: the predicted pass on h and the actual pass on
           the target layer's input with the plain router weight, then prediction_quality.
  replan   the planner alone on counts that are already on the device (re-planning from history).

Shapes are the benchmark's workloads (tiny, Mixtral-, Qwen3- and DeepSeek-V3-shaped, the skew sweep),
the 64-expert shape of Moonlight, and token counts from a decode batch to the largest prefill batch.
"""
import math

import torch

import paper_2608_14205_amd as fb

# hidden size, experts, routing rule, placement (ranks x slots) and swap budget of each router
MODELS = {
    "tiny": dict(H=1024, E=16, kind="softmax", k=2, ng=1, kg=1, topn=1, R=8, S=2, B=2),
    "mixtral": dict(H=4096, E=8, kind="softmax", k=2, ng=1, kg=1, topn=1, R=8, S=2, B=1),
    "moonlight": dict(H=2048, E=64, kind="sigmoid", k=6, ng=1, kg=1, topn=1, R=8, S=8, B=4),
    "qwen3": dict(H=2048, E=128, kind="softmax", k=8, ng=1, kg=1, topn=1, R=32, S=4, B=6),
    "dsv3": dict(H=7168, E=256, kind="sigmoid", k=8, ng=8, kg=4, topn=2, R=32, S=8, B=8),
}


def listed():
    return [
        # the smallest call: the float32 Tiny workload
        dict(name="tiny_f32", job="pass", model="tiny", T=512, dtype="f32", timed=False, full=False),
        # a decode step's batch: one tile or two, all of the router weight
        dict(name="dsv3_decode", job="pass", model="dsv3", T=192, dtype="bf16", timed=False, full=False),
        # a ragged chunk of a chunked prefill, planned under the profiled attention time
        dict(name="dsv3_chunk_timed", job="pass", model="dsv3", T=1237, dtype="bf16", timed=True, full=False),
        # the named prefill workloads, each layer's pass as the serving loop calls it
        dict(name="mixtral", job="pass", model="mixtral", T=8192, dtype="bf16", timed=False, full=False),
        dict(name="qwen3", job="pass", model="qwen3", T=16384, dtype="bf16", timed=False, full=False),
        dict(name="dsv3_4096", job="pass", model="dsv3", T=4096, dtype="bf16", timed=False, full=False),
        dict(name="dsv3_16384", job="pass", model="dsv3", T=16384, dtype="bf16", timed=False, full=False),
        dict(name="dsv3_32768", job="pass", model="dsv3", T=32768, dtype="bf16", timed=False, full=False),
        # the largest batch of the skew sweep
        dict(name="dsv3_65536", job="pass", model="dsv3", T=65536, dtype="bf16", timed=False, full=False),
        # a router kept in float32, its early selections and logits handed on
        dict(name="dsv3_gate_f32", job="pass", model="dsv3", T=4096, dtype="f32", timed=False, full=True),
        # the prediction-quality study of one layer, a ragged batch, router not packed beforehand
        dict(name="moonlight_study", job="study", model="moonlight", T=8190, dtype="bf16"),
        # every rank pair considered: the planner's full mode on predicted DeepSeek-V3-shaped counts
        dict(name="replan_full", job="replan", R=32, S=8, B=16, T=16384, mode="full", timed=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pass", "pass", "pass", "pass", "f32", "study", "replan"])
    if kind == "pass":
        model = rng.choice(["mixtral", "moonlight", "qwen3", "dsv3", "dsv3"])
        most = {"mixtral": 32768, "moonlight": 32768, "qwen3": 32768, "dsv3": 49152}[model]
        return dict(job="pass", model=model, T=_log_int(rng, 64, most), dtype="bf16",
                    timed=rng.random() < 0.25, full=False)
    if kind == "f32":
        model = rng.choice(["tiny", "moonlight", "dsv3"])
        return dict(job="pass", model=model, T=_log_int(rng, 100, 4096), dtype="f32",
                    timed=False, full=rng.random() < 0.5)
    if kind == "study":
        return dict(job="study", model=rng.choice(["moonlight", "qwen3"]), T=_log_int(rng, 500, 12000),
                    dtype=rng.choice(["bf16", "bf16", "f32"]))
    S = rng.choice([2, 4, 8, 8, 9])
    R = rng.choice([8, 16, 32, 48])
    return dict(job="replan", R=R, S=S, B=rng.choice([4, 8, 16]), T=_log_int(rng, 1000, 65536),
                mode=rng.choice(["full", "full", "frontier"]), timed=rng.random() < 0.4)


# ---- inputs --------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _zipf(n, s):
    p = torch.arange(1, n + 1, dtype=torch.float64, device="cuda").pow(-s)
    return p / p.sum()


def _router_inputs(m, T, dtype, g):
    """Router weight N(0, 0.02), hidden states 3 w[z] + N(0, 1) with Zipf(1.1) clusters z over the
    experts (in a random order), and the selection bias N(0, 0.01) of sigmoid routing."""
    E, H = m["E"], m["H"]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    w = (torch.randn(E, H, generator=g, device="cuda") * 0.02).to(dt)
    perm = torch.randperm(E, generator=g, device="cuda")
    z = perm[torch.multinomial(_zipf(E, 1.1), T, replacement=True, generator=g)]
    x = torch.empty(T, H, dtype=dt, device="cuda")
    for t in range(0, T, 8192):
        n = min(8192, T - t)
        x[t:t + n] = 3.0 * w[z[t:t + n]].float() + torch.randn(n, H, generator=g, device="cuda")
    bias = 0.01 * torch.randn(E, generator=g, device="cuda") if m["kind"] == "sigmoid" else None
    return x, w, bias


def _slots(R, S, E):
    """Contiguous placement: expert e on rank e / (E / R); slots past the experts of a rank empty."""
    per = E // R
    t = torch.full((R, S), -1, dtype=torch.int32)
    e2r = torch.empty(E, dtype=torch.int32)
    for e in range(E):
        t[e // per, e % per] = e
        e2r[e] = e // per
    return t.cuda(), e2r.cuda()


def _cost(R, E):
    """Ranks on nodes of 8, 88 MB experts, 8 ms of attention: the benchmark's cost model."""
    node = torch.arange(R, dtype=torch.int32, device="cuda") // 8
    size = torch.full((E,), 3 * 7168 * 2048 * 2, dtype=torch.int64, device="cuda")
    return fb.CostModel(node, size, (20_000, 50_000), (100_000, 25_000), 8_000_000)


def _carve(parts):
    """Views of one zeroed byte buffer, each 16-byte aligned: everything a pass reports, so that the
    program brings it to the host with one copy.  parts: (shape, dtype) or None."""
    size = {torch.int32: 4, torch.int64: 8, torch.float64: 8, torch.uint8: 1}
    at, spans = 0, []
    for p in parts:
        if p is None:
            spans.append(None)
            continue
        n = math.prod(p[0]) * size[p[1]]
        spans.append((at, n))
        at += (n + 15) // 16 * 16
    buf = torch.zeros(at, dtype=torch.uint8, device="cuda")
    return buf, [None if s is None else buf[s[0]:s[0] + s[1]].view(p[1]).view(p[0])
                 for s, p in zip(spans, parts)]


def _plan_parts(R, S, E, B, timed):
    return [((max(B, 1) * 32,), torch.uint8), ((1,), torch.int32), ((R, S), torch.int32),
            ((E,), torch.int32), ((R,), torch.int64), ((1,), torch.int32),
            ((max(B, 1),), torch.int64) if timed else None]


def _pred_parts(E, R, T, k, topk):
    return [((E,), torch.int32), ((R,), torch.int32), ((1,), torch.float64),
            ((T, k), torch.int32) if topk else None]


def _counts(R, S, T, g):
    """Predicted workload of a top-8 router over R * S experts: half of it skewed by Zipf(1.1)."""
    E = R * S
    p = 0.5 * _zipf(E, 1.1)[torch.randperm(E, generator=g, device="cuda")] + 0.5 / E
    c = torch.multinomial(p, T * 8, replacement=True, generator=g)
    return torch.bincount(c, minlength=E).to(torch.int32)


def prepare(case, seed):
    g = _gen(seed)
    if case["job"] == "replan":
        R, S, B = case["R"], case["S"], case["B"]
        E = R * S
        buf, p = _carve(_plan_parts(R, S, E, B, case["timed"]))
        return dict(case=case, counts=_counts(R, S, case["T"], g), slots=_slots(R, S, E)[0],
                    budget=fb.Budget(B, mode=case["mode"]), buf=buf, plan=fb.DevicePlan(*p),
                    cost=_cost(R, E) if case["timed"] else None)
    m, T = MODELS[case["model"]], case["T"]
    x, w, bias = _router_inputs(m, T, case["dtype"], g)
    slots, e2r = _slots(m["R"], m["S"], m["E"])
    st = dict(case=case, m=m, x=x, bias=bias, slots=slots, e2r=e2r, predictor=fb.Predictor("cuda"),
              scoring=fb.Scoring(m["kind"], m["k"], m["ng"], m["kg"], m["topn"]))
    if case["job"] == "study":
        # the target layer's router input: h plus a residual update N(0, 0.2)
        st["target"] = torch.empty_like(x)
        for t in range(0, T, 8192):
            n = min(8192, T - t)
            st["target"][t:t + n] = x[t:t + n].float() + 0.2 * torch.randn(n, m["H"], generator=g, device="cuda")
        st["w"] = w
        st["buf"], p = _carve(2 * _pred_parts(m["E"], m["R"], T, m["k"], True))
        st["logits"] = [torch.zeros(T, m["E"], device="cuda") for _ in range(2)]
        st["pred"] = [fb.Prediction(*p[4 * i:4 * i + 4], st["logits"][i]) for i in range(2)]
        return st
    st["router"] = fb.pack_router_weight(w)
    pred = _pred_parts(m["E"], m["R"], T, m["k"], case["full"])
    plan = [] if case["full"] else _plan_parts(m["R"], m["S"], m["E"], m["B"], case["timed"])
    st["buf"], p = _carve(pred + plan)
    st["logits"] = torch.zeros(T, m["E"], device="cuda") if case["full"] else None
    st["pred"] = fb.Prediction(*p[:4], st["logits"])
    st["plan"] = None if case["full"] else fb.DevicePlan(*p[4:])
    st["budget"] = fb.Budget(m["B"])
    st["cost"] = _cost(m["R"], m["E"]) if case["timed"] else None
    return st


def run(st):
    case = st["case"]
    if case["job"] == "replan":
        if st["cost"] is not None:
            fb.plan_swaps_timed_device(st["counts"], st["slots"], st["budget"], st["cost"], out=st["plan"])
        else:
            fb.plan_swaps_device(st["counts"], st["slots"], st["budget"], out=st["plan"])
        return st["buf"]
    m, pr = st["m"], st["predictor"]
    if case["job"] == "study":
        for x, out in zip((st["x"], st["target"]), st["pred"]):
            pr.predict_load(x, st["w"], st["scoring"], st["e2r"], m["R"], select_bias=st["bias"],
                            out=out, return_topk=True, return_logits=True)
        q = fb.prediction_quality(st["pred"][0], st["pred"][1], st["x"], st["target"])
        # the hit count is hit_rate * T * k
        return dict(block=st["buf"], logits=st["logits"], hit_rate=q.hit_rate,
                    logit_cosine=q.logit_cosine, hidden_cosine=q.hidden_cosine)
    if case["full"]:
        pr.predict_load(st["x"], st["router"], st["scoring"], st["e2r"], m["R"], select_bias=st["bias"],
                        out=st["pred"], return_topk=True, return_logits=True)
        return dict(block=st["buf"], logits=st["logits"])
    pr.predict_plan(st["x"], st["router"], st["scoring"], st["e2r"], st["slots"], st["budget"],
                    select_bias=st["bias"], out=st["pred"], plan=st["plan"], cost=st["cost"])
    return dict(block=st["buf"])


# ---- what a pass cannot do without, and how far two correct passes may differ -------------------------

def work(case):
    if case["job"] == "replan":
        R, S, B = case["R"], case["S"], case["B"]
        E = R * S
        # counts and table in, table, expert ranks, loads and swaps out; one look at every candidate
        # pair of items per round
        pairs = S * S * (R * (R - 1) // 2 if case["mode"] == "full" else 1)
        return {"bytes": 4 * E + 4 * R * S + 4 * R * S + 4 * E + 8 * R + 40 * B, "flops": 6 * pairs * B}
    m, T = MODELS[case["model"]], case["T"]
    b = 2 if case["dtype"] == "bf16" else 4
    E, H, R, k = m["E"], m["H"], m["R"], m["k"]
    once = T * H * b + E * H * b + 12 * E + 4 * R + 8
    if case["job"] == "study":
        # both passes share the weight; their selections and logits are written; the cosines and hits
        # need no further reading
        return {"bytes": 2 * once - E * H * b + 2 * (4 * T * k + 4 * T * E), "flops": 4 * T * H * E + 6 * T * (H + E)}
    if case["full"]:
        return {"bytes": once + 4 * T * k + 4 * T * E, "flops": 2 * T * H * E}
    return {"bytes": once + 12 * R * m["S"] + 8 * R, "flops": 2 * T * H * E}


def tolerance(case):
    if case["job"] == "replan":
        return "exact"
    # Measured by running each case again with the hidden dimension permuted, which is another order
    # of the same float32 sums: logits differ by 1e-6 of their norm and at most 7e-6 of a value.  The
    # block of whole numbers moves only with tokens whose k-th and (k + 1)-th scores are closer than
    # that (about 1 token in 40,000); one such token changes about 6 of the block's bytes, 0.3% of the
    # smallest block of a many-expert router.
    return {"rel": 4e-6, "max": 3e-5, "differ": 0.01}


def exact(case, seed):
    """64-bit logits, and for the study the 64-bit cosines.  None for the rest: the blocks are whole
    numbers (and a ratio of two), as is the hit rate."""
    if case["job"] == "replan" or (case["job"] == "pass" and not case["full"]):
        return None
    g = _gen(seed)
    m, T = MODELS[case["model"]], case["T"]
    if case["job"] == "pass":
        x, w, _ = _router_inputs(m, T, case["dtype"], g)
        return dict(block=None, logits=x.double() @ w.double().t())
    st = prepare(case, seed)
    x, y, w = st["x"].double(), st["target"].double(), st["w"].double()
    zx, zy = x @ w.t(), y @ w.t()

    def cosine(a, b):
        return float(((a * b).sum(1) / (a.norm(dim=1) * b.norm(dim=1))).mean())

    return dict(block=None, logits=[zx, zy], hit_rate=None, logit_cosine=cosine(zx, zy),
                hidden_cosine=cosine(x, y))
