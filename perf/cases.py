"""What is timed when this library's speed is looked at: decode steps of DIP / DIP-CA SwiGLU
layers through the public calls of paper_2412_01380_amd, over the range they are used in.

A case is a dict of plain values:
  kind    "layers"   one dip_swiglu_mlp_forward per layer, as a model calls it with its attention
                     in between
          "stack"    one dip_swiglu_mlp_forward_stack for all layers of a token
          "batched"  one dip_swiglu_mlp_forward_batched per layer (a small decode batch)
          "bstack"   one dip_swiglu_mlp_forward_batched_stack for all layers of a step
          "scheme"   GLU, Gate or Up pruning of Sec. 3.2, one call per layer
          "ops"      the single steps by hand: scores, top-K, gathered product, cache update
          "tiered"   weights in pinned host memory behind an HBM slot cache, one call per layer
  d, f    d_model and d_ff;   L  layers;   B  rows per step;   fmt  weight format
  r       keep ratio at both pruning points
  frac    share of the columns the residency caches hold (0: plain DIP, no caches)
  policy  "lru" or "lfu";   gamma  the penalty of Eq. 10;   x  the input distribution

One pass is one decode step (one token, or B rows) through all L layers.  A state holds the
weights, the caches and a short stream of tokens; successive passes take successive tokens, as
a decode loop does, and the caches evolve.
"""
import math

import torch

import paper_2412_01380_amd as D

TOKENS = 8          # distinct tokens of a state's stream, then it repeats


def listed():
    dip = dict(frac=0.0, policy="lru", gamma=0.2)
    ca = dict(frac=0.5, policy="lru", gamma=0.2)
    return [
        # the smallest call there is: one fp32 layer that fits the caches of the chip; what a
        # small model or a unit of work under a latency bound sees -- launches and host path
        dict(name="tiny layer f32", kind="layers", d=512, f=1536, L=1, B=1, fmt="f32", r=0.5, x="gaussian", **dip),
        # Phi-3-Mini shaped layers called one by one, plain DIP with heavy-tailed inputs: eight
        # weight copies, so that no cache holds them
        dict(name="phi3-mini layers bf16", kind="layers", d=3072, f=8192, L=8, B=1, fmt="bf16", r=0.5, x="studentt3", **dip),
        # the large model's layers one by one, twice as dense, with LFU caches over a quarter
        dict(name="phi3-medium layers bf16 lfu", kind="layers", d=5120, f=17920, L=4, B=1, fmt="bf16", r=0.5,
             frac=0.25, policy="lfu", gamma=0.2, x="ar1"),
        # a whole decode step of the two stacks the benchmark is quoted on
        dict(name="llama3-8b stack bf16", kind="stack", d=4096, f=14336, L=32, B=1, fmt="bf16", r=0.3, x="ar1", **ca),
        dict(name="phi3-medium stack bf16", kind="stack", d=5120, f=17920, L=40, B=1, fmt="bf16", r=0.3, x="ar1", **ca),
        # the same stack with int4-g128 weights at one, two and eight rows per step
        dict(name="phi3-medium stack int4", kind="stack", d=5120, f=17920, L=40, B=1, fmt="int4", r=0.3, x="ar1", **ca),
        dict(name="phi3-medium int4 batch 2", kind="bstack", d=5120, f=17920, L=40, B=2, fmt="int4", r=0.3, x="ar1", **ca),
        dict(name="phi3-medium int4 batch 8", kind="bstack", d=5120, f=17920, L=40, B=8, fmt="int4", r=0.3, x="ar1", **ca),
        # a batch of three through layers whose sizes are no multiple of any tile
        dict(name="ragged layers bf16 batch 3", kind="batched", d=2056, f=5464, L=4, B=3, fmt="bf16", r=0.3, x="ar1", **ca),
        # Sec. 3.2: the scheme with the row-gathered product
        dict(name="phi3-mini gate pruning bf16", kind="scheme", scheme="gate", d=3072, f=8192, L=4, B=1, fmt="bf16",
             r=0.5, x="studentt3", **dip),
        # the steps of Alg. 1 by hand on one linear layer, as a caller with its own MLP does
        dict(name="single steps f32", kind="ops", d=4096, f=4100, L=1, B=1, fmt="f32", r=0.3, x="ar1", **ca),
        # two memory tiers: the columns the cache brings in cross PCIe
        dict(name="phi3-mini two tiers bf16", kind="tiered", d=3072, f=8192, L=2, B=1, fmt="bf16", r=0.3, x="ar1", **ca),
    ]


def _log(rng, lo, hi, step):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, int(round(v / step)) * step)


def draw(rng):
    kind = rng.choice(["layers", "layers", "stack", "stack", "stack", "bstack", "bstack", "batched", "scheme", "ops", "tiered"])
    c = dict(kind=kind, B=1, L=1)
    c["fmt"] = rng.choice(["bf16", "bf16", "int4", "f32"])
    if kind == "tiered" and c["fmt"] == "int4":
        c["fmt"] = "bf16"
    step = 128 if c["fmt"] == "int4" else 8
    c["d"] = _log(rng, 512, 2048 if kind == "tiered" else 5120, step)
    c["f"] = _log(rng, 2 * c["d"], 3.5 * c["d"], step)
    if kind in ("batched", "bstack"):
        c["B"] = rng.randint(1, 8)
    if kind == "scheme":
        c["scheme"] = rng.choice(["glu", "gate", "up"])
    if kind == "tiered":
        c["L"] = rng.randint(1, 2)
    elif kind != "ops":
        # as many layers as keep the weights below 6 GB (the largest listed stack holds 22 GB)
        most = int(6e9 / (3 * c["d"] * c["f"] * {"f32": 4, "bf16": 2, "int4": 0.516}[c["fmt"]]))
        c["L"] = _log(rng, 1, max(1, min(40, most)), 1)
    c["r"] = round(rng.uniform(0.2, 0.6), 3)
    cached = kind in ("tiered", "ops") or (kind != "scheme" and rng.random() < 0.7)
    c["frac"] = rng.choice([0.25, 0.5, 0.75]) if cached else 0.0
    c["policy"] = rng.choice(["lru", "lru", "lfu"])
    c["gamma"] = rng.choice([0.2, 0.2, 0.1, 1.0])
    c["x"] = rng.choice(["ar1", "ar1", "studentt3", "gaussian"])
    return c


def _k(r, n):
    return max(1, min(n, int(math.floor(r * n + 0.5))))


# ---- inputs ---------------------------------------------------------------------------------
def _tokens(case, shape, g):
    """[TOKENS, *shape] activations on the GPU: iid Gaussian, iid Student-t(3) (heavy tails), or a
    per-feature AR(1) stream with rho 0.8 and unit-variance Laplace noise (what a cache exploits)."""
    normal = lambda: torch.randn(TOKENS, *shape, device="cuda", generator=g)
    if case["x"] == "gaussian":
        return normal()
    if case["x"] == "studentt3":
        z = normal()
        chi2 = sum(normal() ** 2 for _ in range(3))
        return (z / torch.sqrt(chi2 / 3.0)).contiguous()
    u = torch.rand(TOKENS, *shape, device="cuda", generator=g) - 0.5
    eps = -torch.sign(u) * torch.log1p((-2.0 * u.abs()).clamp_min(-0.9999999)) / math.sqrt(2.0)
    out = torch.empty_like(eps)
    out[0] = eps[0]
    for t in range(1, TOKENS):
        out[t] = 0.8 * out[t - 1] + 0.6 * eps[t]
    return out


def _matrix(rows, cols, fmt, g):
    """Weights ~ N(0, 0.02^2), stored feature-major in the case's format (int4: one fp16 scale
    max|w|/7 per 128 consecutive elements, low nibble = even element)."""
    if fmt != "int4":
        w = torch.empty(rows, cols, device="cuda", dtype=torch.bfloat16 if fmt == "bf16" else torch.float32)
        return w.normal_(0.0, 0.02, generator=g), None
    w = torch.empty(rows, cols // 128, 128, device="cuda").normal_(0.0, 0.02, generator=g)
    scales = (w.abs().amax(dim=2) / 7.0).half()
    q = torch.round(w.div_(scales.float().unsqueeze(2))).clamp_(-8, 7).to(torch.int8).view(rows, cols)
    del w
    q = (q & 15).view(torch.uint8)
    return (q[:, 0::2] | (q[:, 1::2] << 4)).contiguous(), scales.contiguous()


def _weight(rows, cols, fmt, g):
    w, scales = _matrix(rows, cols, fmt, g)
    return D.Weight(w) if scales is None else D.Weight(w, scales)


def _pad(n):
    return (n + 63) // 64 * 64


def _caches(case, n, L, g):
    """L caches over n columns, warm with a random resident set, their state ([bits | stamp | meta]
    per layer) in one tensor, as a program that checkpoints it keeps it."""
    words, cap = (n + 31) // 32, int(case["frac"] * n)
    state = torch.zeros(L, _pad(words) + _pad(n) + 64, dtype=torch.int32, device="cuda")
    caches = []
    for l in range(L):
        c = D.Cache(n, cap, D.DIP_LFU if case["policy"] == "lfu" else D.DIP_LRU)
        at = _pad(words)
        c.bits, c.stamp = state[l, :words], state[l, at:at + n]
        c.meta = state[l, at + _pad(n):at + _pad(n) + len(D.META)]
        c.c.bits, c.c.stamp, c.c.meta = c.bits.data_ptr(), c.stamp.data_ptr(), c.meta.data_ptr()
        resident = torch.zeros(words * 32, dtype=torch.int64, device="cuda")
        resident[torch.randperm(n, device="cuda", generator=g)[:cap]] = 1
        packed = (resident.view(words, 32) << torch.arange(32, device="cuda")).sum(dim=1)
        warm = torch.where(packed >= 2 ** 31, packed - 2 ** 32, packed).to(torch.int32)
        D.dip_cache_init(c, warm)
        caches.append(c)
    return caches, state


def _workspace(nbytes):
    return torch.empty(max(256, nbytes), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    d, f, L, B, fmt, kind = (case[k] for k in ("d", "f", "L", "B", "fmt", "kind"))
    k_in, k_mid = _k(case["r"], d), _k(case["r"], f)
    s = dict(case=case, t=0, k_in=k_in, k_mid=k_mid)
    if kind == "ops":
        s["x"] = _tokens(case, (d,), g)
        s["w"] = _weight(d, f, fmt, g)
        (s["cache"],), s["state"] = _caches(case, d, 1, g)
        s["scores"] = torch.empty(d, device="cuda")
        s["mask"] = torch.empty((d + 31) // 32, dtype=torch.int32, device="cuda")
        s["idx"] = torch.empty(k_in, dtype=torch.int32, device="cuda")
        s["y"] = torch.empty(s["w"].c.n_out, device="cuda")
        s["ws"] = _workspace(D.dip_gathered_gemv_workspace_bytes(s["w"], k_in))
        return s
    s["x"] = _tokens(case, (L, d) if B == 1 and kind not in ("batched", "bstack") else (L, B, d), g)
    s["y"] = torch.empty(s["x"].shape[1:], device="cuda")
    s["cin"] = s["cmid"] = None
    if case["frac"] > 0:
        s["cin"], s["state_in"] = _caches(case, d, L, g)
        s["cmid"], s["state_mid"] = _caches(case, f, L, g)
    if kind == "tiered":
        s["mlps"] = []
        for l in range(L):
            pair = []
            for rows, cols, cache in ((d, 2 * f, s["cin"][l]), (f, d, s["cmid"][l])):
                w, _ = _matrix(rows, cols, fmt, g)
                host = torch.empty(w.shape, dtype=w.dtype, pin_memory=True)
                host.copy_(w)
                tw = D.TieredWeight(host, cache.capacity)
                D.dip_tier_init(tw, cache, _workspace(D.dip_tier_init_workspace_bytes(tw)))
                pair.append(tw)
            s["mlps"].append(D.TieredMlp(*pair))
        s["ws"] = _workspace(D.dip_tiered_mlp_forward_workspace_bytes(s["mlps"][0], k_in, k_mid))
        torch.cuda.synchronize()        # the workspaces of the slot fills end here
        return s
    if kind == "scheme" and case["scheme"] != "glu":
        s["mlps"] = [D.MlpSplit(_weight(d, f, fmt, g), _weight(f, d, fmt, g), _weight(f, d, fmt, g)) for _ in range(L)]
        s["ws"] = _workspace(D.dip_partial_pruning_forward_workspace_bytes(s["mlps"][0], k_mid))
        return s
    mlps = s["mlps"] = [D.Mlp(_weight(d, 2 * f, fmt, g), _weight(f, d, fmt, g)) for _ in range(L)]
    if kind in ("stack", "bstack"):
        s["stack"] = D.MlpStack(mlps, s["cin"], s["cmid"])
    if kind == "stack":
        s["ws"] = _workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(s["stack"], k_in, k_mid))
    elif kind == "bstack":
        s["ws"] = _workspace(D.dip_swiglu_mlp_forward_batched_stack_workspace_bytes(s["stack"], B, k_in, k_mid))
    elif kind == "batched":
        s["ws"] = _workspace(D.dip_swiglu_mlp_forward_batched_workspace_bytes(mlps[0], B, k_in, k_mid))
    elif kind == "scheme":
        s["ws"] = _workspace(D.dip_glu_pruning_forward_workspace_bytes(mlps[0], k_mid))
    else:
        s["ws"] = _workspace(D.dip_swiglu_mlp_forward_workspace_bytes(mlps[0], k_in, k_mid))
    return s


def run(s):
    case, k_in, k_mid = s["case"], s["k_in"], s["k_mid"]
    kind, L, B, d, gamma = case["kind"], case["L"], case["B"], case["d"], case["gamma"]
    x, y, ws = s["x"][s["t"]], s["y"], s["ws"]
    s["t"] = (s["t"] + 1) % TOKENS
    if kind == "ops":
        D.dip_ca_scores(x, d, s["cache"].bits, gamma, s["scores"])
        D.dip_prune_topk(s["scores"], d, k_in, s["mask"], s["idx"])
        D.dip_gathered_gemv(s["w"], x, s["idx"], k_in, y, ws)
        D.dip_cache_update(s["cache"], s["mask"])
        return {"scores": s["scores"], "mask": s["mask"], "idx": s["idx"], "y": y, "state": s["state"]}
    cin, cmid = s["cin"] or [None] * L, s["cmid"] or [None] * L
    if kind == "layers":
        for l in range(L):
            D.dip_swiglu_mlp_forward(s["mlps"][l], x[l], k_in, k_mid, cin[l], cmid[l], gamma, y[l], None, ws)
    elif kind == "stack":
        D.dip_swiglu_mlp_forward_stack(s["stack"], x, d, k_in, k_mid, gamma, y, d, ws)
    elif kind == "batched":
        for l in range(L):
            D.dip_swiglu_mlp_forward_batched(s["mlps"][l], x[l], B, k_in, k_mid, cin[l], cmid[l], gamma, y[l],
                                             None, None, None, ws)
    elif kind == "bstack":
        D.dip_swiglu_mlp_forward_batched_stack(s["stack"], x, B * d, B, k_in, k_mid, gamma, y, B * d, ws)
    elif kind == "tiered":
        for l in range(L):
            D.dip_tiered_mlp_forward(s["mlps"][l], x[l], k_in, k_mid, cin[l], cmid[l], gamma, y[l], None, ws)
    elif case["scheme"] == "glu":
        for l in range(L):
            D.dip_glu_pruning_forward(s["mlps"][l], x[l], k_mid, y[l], None, ws)
    else:
        scheme = D.DIP_GATE_PRUNING if case["scheme"] == "gate" else D.DIP_UP_PRUNING
        for l in range(L):
            D.dip_partial_pruning_forward(s["mlps"][l], scheme, x[l], k_mid, y[l], None, ws)
    if case["frac"] > 0:
        return {"y": y, "state_in": s["state_in"], "state_mid": s["state_mid"]}
    return y


# ---- what a pass cannot do without ----------------------------------------------------------
def _union(case, r):
    """Share of the columns that B rows select together: rows are scored against one cache, so
    their masks overlap more than independent ones would (at r = 0.3 with caches over half of
    the columns about 0.43 of the columns at two rows and 0.64 at eight)."""
    B = case["B"]
    return 1.0 - (1.0 - r) ** (B if case["frac"] == 0 else B ** 0.6)


def work(case):
    d, f, L, B, fmt = (case[k] for k in ("d", "f", "L", "B", "fmt"))
    size = {"f32": 4.0, "bf16": 2.0, "int4": 0.5 + 2.0 / 128}[fmt]
    if case["kind"] == "ops":
        k = _k(case["r"], d)
        return {"bytes": k * f * size + 24.0 * d, "flops": 2.0 * k * f}
    r_in, r_mid = _k(case["r"], d) / d, _k(case["r"], f) / f
    if case["kind"] == "scheme":
        first = 2.0 if case["scheme"] == "glu" else 1.0 + r_mid
        elems = (first + r_mid) * d * f
        flops = 2.0 * elems
    else:
        elems = (2.0 * _union(case, r_in) + _union(case, r_mid)) * d * f
        flops = 2.0 * B * (2.0 * r_in + r_mid) * d * f
    return {"bytes": L * (elems * size + 8.0 * B * d), "flops": L * flops}


def tolerance(case):
    # Sums are fp32 (int4 batches of three and more: activation times scale enters as two fp16
    # terms): another order of summation moves an output by a few 1e-7 (1e-5) of its norm.  The
    # mask of the second pruning point is a function of the bits of h, so a pair of columns whose
    # scores agree to that error can trade places: y moves by about 1 / sqrt(k) of its norm, and
    # the cache state by a few entries.
    if case["kind"] == "ops":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}
    h_err = 1e-5 if case["fmt"] == "int4" and case["B"] >= 3 else 3e-7
    rows = case["L"] * case["B"]
    k = _k(case["r"], case["f"])
    # trades to expect: about f keys per octave around the threshold, each as wide as its error
    trades = max(1.0, rows * case["f"] * h_err)
    if rows * case["f"] * h_err < 2e-3:
        return {"rel": 4e-6 if h_err < 1e-6 else 2e-4, "max": 4e-5 if h_err < 1e-6 else 2e-3, "differ": 1e-3}
    return {"rel": min(0.02, 1.5 * math.sqrt(trades / (rows * k))), "max": 0.3, "differ": 2e-3}
