"""Timed cases of the MoE shard library: what a program that serves, profiles or
places mixture-of-experts layers has it do, through the public calls.

Four kinds of case:

* ``layer``: one GPU's share of a MoE layer (router, histogram, dispatch
  positions, expert FFN reading the routed rows, combine) as ``moe_layer`` runs
  it, with the buffers and row-padded weights that a serving loop keeps;
* ``mx``: the same layer with MXFP8 experts (dispatch, quantisation of the
  routed rows, MXFP8 FFN, combine);
* ``expert``: the expert FFN alone on one expert, the point of a
  latency-against-load profile;
* ``placement``: the control path after a window of passes (window push, drift
  test, greedy solve, incremental solve, predicted cost).

The layer shapes are the library's five workloads; token counts run from one
token to the largest batch of each, skews are 0, 1 and 1.5. Router inputs sit on
grids on which every partial sum is exact in fp32, so expert ids are the same
whatever the order of the sums.
"""
import math

import numpy as np
import torch

import paper_2606_00735_amd as moe

# name: H, I, E, k, experts on this GPU, largest T
SHAPES = {
    "tiny": (128, 256, 8, 2, 8, 64),
    "mixtral": (4096, 14336, 8, 2, 8, 4096),
    "qwen3": (2048, 768, 128, 8, 128, 8192),
    "dsv3_shard": (7168, 2048, 256, 8, 32, 16384),
    "maverick_shard": (5120, 8192, 128, 1, 16, 32768),
}
PLACE_E, PLACE_G, PLACE_K = 256, 8, 8  # experts, GPUs and top-k of a placed layer
PLACE_WINDOW = 16                      # passes in the sliding window


def _layer(name, kind, shape, T, alpha):
    return {"name": name, "kind": kind, "shape": shape, "T": T, "alpha": alpha}


def listed():
    return [
        # the fp32 layer at its only size: a handful of short launches
        _layer("tiny_fp32", "layer", "tiny", 64, 1.0),
        # one expert at a few hundred tokens: the middle of a load profile,
        # ragged against every tile height
        {"name": "expert_dsv3_300", "kind": "expert", "shape": "dsv3_shard", "T": 300},
        # decode batches: few tokens, every expert's weights streamed
        _layer("mixtral_decode", "layer", "mixtral", 32, 0.0),
        _layer("qwen3_decode", "layer", "qwen3", 128, 1.0),
        # a chunk of a prompt between decodes: about 60 ragged rows an expert
        _layer("qwen3_chunk", "layer", "qwen3", 1000, 0.0),
        # prefill batches: few large experts; many small ones; shards of
        # larger layers whose remote experts are only counted
        _layer("mixtral_prefill", "layer", "mixtral", 4096, 1.0),
        _layer("qwen3_prefill", "layer", "qwen3", 8192, 1.0),
        _layer("dsv3_prefill", "layer", "dsv3_shard", 16384, 1.0),
        _layer("maverick_prefill", "layer", "maverick_shard", 32768, 0.0),
        # FP8 experts at decode and prefill
        _layer("mx_mixtral_decode", "mx", "mixtral", 32, 0.0),
        _layer("mx_mixtral_prefill", "mx", "mixtral", 4096, 1.0),
        # re-placement of a whole model's experts after a routing drift
        {"name": "placement_58", "kind": "placement", "L": 58, "T": 4096, "alpha": 1.0},
    ]


def _log_int(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n))


def draw(rng):
    u = rng.random()
    if u < 0.08:
        return {"kind": "layer", "shape": "tiny", "T": rng.randint(1, 64), "alpha": rng.choice([0.0, 1.0, 1.5])}
    if u < 0.14:
        return {"kind": "placement", "L": rng.randint(1, 58), "T": _log_int(rng, 64, 4096), "alpha": rng.choice([0.5, 1.0, 1.5])}
    shape = rng.choice(["mixtral", "qwen3", "dsv3_shard", "maverick_shard"])
    if u < 0.30:
        return {"kind": "expert", "shape": shape, "T": _log_int(rng, 1, 4096 if shape == "mixtral" else 8192)}
    T = _log_int(rng, 1, SHAPES[shape][5])
    return {"kind": "mx" if u < 0.5 else "layer", "shape": shape, "T": T, "alpha": rng.choice([0.0, 1.0, 1.5])}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _router(shape, T, alpha, seed, dtype):
    """x [T, H] on the 1/64 grid, w_router [E, H] on the 2^-q grid (sums exact in
    fp32), the skewed per-expert bias and the expert map. The local experts of a
    shard hold one rank of each group of E / E_local consecutive ranks, as a
    load-balancing placement leaves them."""
    H, _, E, _, E_local, _ = SHAPES[shape]
    g = _gen(seed)
    x = torch.randn((T, H), generator=g, device="cuda")
    x = (x * 64.0).round_().clamp_(-255.0, 255.0).mul_(1.0 / 64.0)
    q = int(math.ceil(math.log2(16.0 * math.sqrt(H))))
    w = torch.randn((E, H), generator=g, device="cuda") / math.sqrt(H)
    w = (w * 2.0 ** q).round_().clamp_(-255.0, 255.0).mul_(2.0 ** -q)
    r = np.random.default_rng(int(seed))
    rank = r.permutation(E)  # rank[e] - 0 is the hottest
    bias = (-float(alpha) * np.log(rank + 1.0)).astype(np.float32)
    step = E // E_local
    chosen = {int(j * step + r.integers(step)) for j in range(E_local)}
    local = np.array([e for e in range(E) if int(rank[e]) in chosen])
    emap = np.full(E, -1, np.int32)
    emap[local] = np.arange(E_local, dtype=np.int32)
    return x.to(dtype), w.to(dtype), torch.from_numpy(bias).cuda(), emap


def _experts(n, H, I, seed, dtype):
    g = _gen(int(seed) + 7919)

    def w(rows, cols):
        t = torch.randn((n, rows, cols), generator=g, device="cuda", dtype=dtype)
        return t.mul_(1.0 / math.sqrt(cols))

    return w(I, H), w(I, H), w(H, I)


def _prepare_layer(case, seed):
    shape, T = case["shape"], case["T"]
    H, I, E, k, E_local, _ = SHAPES[shape]
    dt = torch.float32 if shape == "tiny" else torch.bfloat16
    x, wr, bias, emap = _router(shape, T, case["alpha"], seed, dt)
    wg, wu, wd = _experts(E_local, H, I, seed, dt)
    if dt == torch.bfloat16:
        wg, wu, wd = moe.pad_weight_rows(wg), moe.pad_weight_rows(wu), moe.pad_weight_rows(wd)
    return {"kind": "layer", "x": x, "wr": wr, "bias": bias, "k": k, "emap": emap, "w": (wg, wu, wd), "bufs": {},
            "fuse": dt == torch.bfloat16}


def _prepare_mx(case, seed):
    shape, T = case["shape"], case["T"]
    H, I, E, k, E_local, _ = SHAPES[shape]
    x, wr, bias, emap = _router(shape, T, case["alpha"], seed, torch.bfloat16)
    w = tuple(moe.moe_mx_quantize(m) for m in _experts(E_local, H, I, seed, torch.bfloat16))
    dev, M = x.device, T * k
    b = {
        "ids": torch.empty((T, k), dtype=torch.int32, device=dev),
        "weights": torch.empty((T, k), dtype=torch.float32, device=dev),
        "gate_ws": torch.empty(max(1, moe.gate_ws_bytes(T, H, E, x.dtype)), dtype=torch.uint8, device=dev),
        "counts": torch.empty(E, dtype=torch.int32, device=dev),
        "offsets": torch.empty(E_local + 1, dtype=torch.int32, device=dev),
        "hist_ws": torch.empty(moe.hist_ws_bytes(T, k, E, E_local), dtype=torch.uint8, device=dev),
        "x_perm": torch.empty((M, H), dtype=x.dtype, device=dev),
        "perm_src": torch.empty(M, dtype=torch.int32, device=dev),
        "dest": torch.empty(M, dtype=torch.int32, device=dev),
        "xq": moe.MxTensor(torch.empty((M, H), dtype=torch.uint8, device=dev),
                           torch.empty((H // 128, M), dtype=torch.int32, device=dev)),
        "y_perm": torch.empty((M, H), dtype=x.dtype, device=dev),
        "ffn_ws": torch.zeros(moe.ffn_mx_ws_bytes(E_local, H, I, M), dtype=torch.uint8, device=dev),
        "out": torch.empty((T, H), dtype=x.dtype, device=dev),
    }
    return {"kind": "mx", "x": x, "wr": wr, "bias": bias, "k": k, "emap": emap, "w": w, "b": b}


def _prepare_expert(case, seed):
    H, I, _, _, _, _ = SHAPES[case["shape"]]
    M = case["T"]
    x = torch.randn((M, H), generator=_gen(seed), device="cuda", dtype=torch.bfloat16)
    w = tuple(moe.pad_weight_rows(m) for m in _experts(1, H, I, seed, torch.bfloat16))
    off = torch.tensor([0, M], dtype=torch.int32, device="cuda")
    ws = torch.zeros(moe.ffn_ws_bytes(1, H, I, M, x.dtype), dtype=torch.uint8, device="cuda")
    return {"kind": "expert", "x": x, "w": w, "off": off, "ws": ws, "y": torch.empty_like(x)}


def _loads(r, rank, T, alpha):
    """Per-expert counts [L, E] of T tokens whose top-k follow the rank skew."""
    out = np.empty(rank.shape, np.int32)
    for l in range(rank.shape[0]):
        z = -alpha * np.log(rank[l] + 1.0) + r.gumbel(size=(min(T, 512), rank.shape[1]))
        top = np.argpartition(-z, PLACE_K, axis=1)[:, :PLACE_K]
        c = np.bincount(top.reshape(-1), minlength=rank.shape[1])
        out[l] = c * T // z.shape[0]
    return out


def _prepare_placement(case, seed):
    L, T, alpha = case["L"], case["T"], case["alpha"]
    r = np.random.default_rng(int(seed))
    rank = np.stack([r.permutation(PLACE_E) for _ in range(L)])
    before = _loads(r, rank, T, alpha)
    for l in range(L):  # a drift: some pairs of experts trade places
        a = r.permutation(PLACE_E)[:16]
        rank[l, a] = rank[l, a[::-1]]
    after = _loads(r, rank, T, alpha)
    # measured-looking latency curves: flat, then linear, each GPU up to 7 % slower
    n = 2.0 ** np.arange(14)
    t = 40.0 + 0.075 * n
    speed = 1.0 + 0.07 * r.random(PLACE_G)
    kn = torch.from_numpy(np.tile(n, (PLACE_G, 1))).cuda()
    kt = torch.from_numpy(speed[:, None] * t[None, :]).cuda()
    ref = torch.from_numpy(before.astype(np.float64)).cuda()
    assign, _, _ = moe.moe_place_greedy(ref, kn, kt, cap=PLACE_E // PLACE_G)
    ring = torch.zeros((PLACE_WINDOW, L, PLACE_E), dtype=torch.int32, device="cuda")
    return {"kind": "placement", "counts": torch.from_numpy(after).cuda(), "ref": ref, "kn": kn, "kt": kt,
            "assign": assign, "ring": ring, "sums": torch.zeros((L, PLACE_E), dtype=torch.float64, device="cuda")}


def prepare(case, seed):
    return {"layer": _prepare_layer, "mx": _prepare_mx, "expert": _prepare_expert,
            "placement": _prepare_placement}[case["kind"]](case, seed)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    if s["kind"] == "layer":
        r = moe.moe_layer(s["x"], s["wr"], s["bias"], s["k"], s["emap"], *s["w"], bufs=s["bufs"],
                          fuse_gather=s["fuse"])
        return {"ids": r["ids"], "weights": r["weights"], "counts": r["counts"], "out": r["out"]}
    if s["kind"] == "mx":
        b, x, k, emap = s["b"], s["x"], s["k"], s["emap"]
        ids, wts, _ = moe.moe_gate_topk(x, s["wr"], s["bias"], k, ids=b["ids"], weights=b["weights"],
                                        ws=b["gate_ws"])
        counts, offsets, hws = moe.moe_expert_histogram_scan(ids, s["wr"].shape[0], emap, ws=b["hist_ws"],
                                                             counts=b["counts"], offsets=b["offsets"])
        x_perm, _, dest = moe.moe_permute(x, ids, emap, hws, x_perm=b["x_perm"], perm_src=b["perm_src"],
                                          dest=b["dest"])
        xq = moe.moe_mx_quantize(x_perm, out=b["xq"], row_count=offsets[-1:])
        y, _ = moe.moe_grouped_swiglu_ffn_mx(xq, *s["w"], offsets, ws=b["ffn_ws"], y_perm=b["y_perm"])
        out = moe.moe_unpermute_combine(y, wts, dest, x.shape[0], out=b["out"])
        return {"ids": ids, "weights": wts, "counts": counts, "out": out}
    if s["kind"] == "expert":
        y, _ = moe.moe_grouped_swiglu_ffn(s["x"], *s["w"], s["off"], ws=s["ws"], y_perm=s["y"])
        return y
    # placement: the pass's counts enter the window (its one filled slot is
    # replaced on a repeated pass), then the drift test, a fresh solve and the
    # incremental update of the placement in use, each with its predicted cost
    moe.moe_window_push(s["counts"], s["ring"], s["sums"], 0)
    d, trigger = moe.moe_drift_distance(s["sums"], s["ref"], delta=0.05)
    fresh, loads, targets = moe.moe_place_greedy(s["sums"], s["kn"], s["kt"], cap=PLACE_E // PLACE_G)
    updated = s["assign"].clone()
    swaps = moe.moe_place_incremental(s["sums"], s["kn"], s["kt"], updated, eps=0.03)
    cost = moe.moe_placement_cost(s["sums"], updated, s["kn"], s["kt"])
    return {"d": d, "trigger": trigger, "fresh": fresh, "loads": loads, "targets": targets, "updated": updated,
            "swaps": swaps, "cost": cost}


# ---------------------------------------------------------------------------
# Work, tolerance, 64-bit results
# ---------------------------------------------------------------------------
def _routed(case):
    """Expected rows and active experts of the local share, from sampled tokens."""
    _, _, E, k, E_local, _ = SHAPES[case["shape"]]
    r = np.random.default_rng(1)
    n = min(case["T"], 512)
    z = r.standard_normal((n, E)) - case["alpha"] * np.log(np.arange(E) + 1.0)
    top = np.argpartition(-z, k - 1, axis=1)[:, :k] if k < E else np.tile(np.arange(E), (n, 1))
    share = np.bincount(top.reshape(-1), minlength=E) / n  # rows per token, by rank
    mid = share.reshape(E_local, -1).mean(axis=1)          # the expected local expert of each group of ranks
    return float(mid.sum()) * case["T"], float((1.0 - (1.0 - np.minimum(mid, 1.0)) ** case["T"]).sum())


def work(case):
    if case["kind"] == "placement":
        L, E, G = case["L"], PLACE_E, PLACE_G
        return {"bytes": float(L * E * (4 + 8 + 8 + 4 + 4 + 4 + 4) + L * G * 8 * 5), "flops": float(L * E * (G + 8))}
    H, I, E, k, E_local, _ = SHAPES[case["shape"]]
    T = case["T"]
    if case["kind"] == "expert":
        return {"bytes": 3.0 * H * I * 2 + 2.0 * T * H * 2, "flops": 6.0 * H * I * T}
    rows, active = _routed(case)
    es = 4 if case["shape"] == "tiny" else 2
    wbytes = 3.0 * H * I * active * (1.03125 if case["kind"] == "mx" else es)
    return {"bytes": wbytes + (2.0 * T * H + E * H) * es + T * k * 8.0, "flops": 6.0 * H * I * rows + 2.0 * T * H * E}


def tolerance(case):
    if case["kind"] == "placement":
        return "exact"
    if case.get("shape") == "tiny":
        return {"rel": 2e-6}
    # bf16 results (and, for MXFP8, codes of h) rounded from fp32 sums taken in
    # another order
    return {"rel": 1e-2, "max": 0.5}


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "placement":
        w = s["counts"].double()
        dot, na, nb = (w * s["ref"]).sum(1), w.square().sum(1).sqrt(), s["ref"].square().sum(1).sqrt()
        return {"d": 1.0 - dot / (na * nb), "trigger": None, "fresh": None, "loads": None, "targets": None,
                "updated": None, "swaps": None, "cost": [None, None, None]}
    if work(case)["flops"] > 4e11:
        return None
    H, I, E, k, E_local, _ = SHAPES[case["shape"]]

    def ffn(x, e):
        if case["kind"] == "mx":
            wg, wu, wd = (_mx_values(m.codes[e], m.scales[e]) for m in s["w"])
            q = _mx_rounded(x)
        else:
            wg, wu, wd = (m[e].double() for m in s["w"])
            q = x.double()
        g = q @ wg.t()
        h = g / (1.0 + torch.exp(-g)) * (q @ wu.t())
        return h @ wd.t()

    if case["kind"] == "expert":
        return ffn(s["x"], 0)
    x, T = s["x"], case["T"]
    z = ((x.double() @ s["wr"].double().t()).float() + s["bias"]).double()
    top, ids = torch.sort(z, dim=1, descending=True, stable=True)
    top, ids = top[:, :k], ids[:, :k]
    wts = torch.exp(top - top[:, :1])
    wts = wts / wts.sum(1, keepdim=True)
    out = torch.zeros((T, H), dtype=torch.float64, device=x.device)
    for e in range(E):
        if s["emap"][e] < 0:
            continue
        t, j = torch.nonzero(ids == e, as_tuple=True)
        if t.numel():
            out.index_add_(0, t, wts[t, j].unsqueeze(1) * ffn(x[t], int(s["emap"][e])))
    return {"ids": ids.int(), "weights": wts, "counts": torch.bincount(ids.reshape(-1), minlength=E).int(),
            "out": out}


def _mx_values(codes, scales):
    """Values of MXFP8 codes [R, K] with scale dwords [K/128, R], in 64 bits."""
    R, K = codes.shape
    c = scales.t().contiguous().view(torch.uint8).reshape(R, K // 32).double()
    v = codes.contiguous().view(torch.float8_e4m3fn).float().double().reshape(R, K // 32, 32)
    return (v * torch.exp2(c - 127.0).unsqueeze(2)).reshape(R, K)


def _mx_rounded(x):
    """Rows of x rounded to MXFP8 (32-element blocks, power-of-two scales)."""
    R, K = x.shape
    v = x.double().reshape(R, K // 32, 32)
    top = v.abs().amax(2, keepdim=True)
    s = torch.floor(torch.log2(torch.where(top > 0, top, torch.ones_like(top)))) - 8.0
    s = torch.exp2(s.clamp(-127.0, 127.0))
    q = (v / s).clamp(-448.0, 448.0).float().to(torch.float8_e4m3fn).float().double()
    return (q * s).reshape(R, K)
