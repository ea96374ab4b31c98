"""The 4-wave GEMM launches (256-row tile, small and mid tiles, splits) against
the 8-wave ones, bit for bit: both add each output's products over K in ascending
order and cut K and the tiles at the same places.

Which kernels a call takes depends on how many rows it is told, or may, expect
(waves_for), and K >= 4096 is where 4 waves are considered. The same routed rows
run three times: as rows of a layer of 256 experts (few expected: 8 waves), of a
layer of just these experts (4 waves where that many rows suit them) and of an
unknown layer with at least 1024 rows of M_cap per expert (both kernels launched,
the offsets choose). MXFP8 calls know M_cap alone: experts without rows bring it
under 1024 per expert (8 waves). The results are also held to fp32 or 64-bit computations."""
import pytest
import torch

import gpu_helpers as G
import paper_2606_00735_amd as moe

pytestmark = pytest.mark.gpu

CASES = [
    # H, I, rows per expert
    (4096, 4096, [700, 700]),                           # gate/up on 4 waves
    (4224, 4096, [1, 64, 65, 128, 129, 255, 256, 257]),  # every row class, at its edges
    (4224, 512, [1100]),                                # 20 tiles: split along K
    (4224, 640, [1300, 0, 1100]),                       # an empty expert, full and ragged last tiles
    (4096, 4224, [4736, 4700]),                         # down in 256-column tiles, a split last round
    (4096, 4096, [5, 0, 20]),                           # room for many rows, few there: 8 waves
]
IDS = [f"H{h}-I{i}-E{len(r)}-M{sum(r)}" for h, i, r in CASES]


def _inputs(H, I, rows, seed, empty=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def rnd(*s, scale=1.0):
        return torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16).mul_(scale)

    E, M = len(rows), sum(rows)
    off = torch.tensor([0] + list(torch.tensor(rows + [0] * empty).cumsum(0)), dtype=torch.int32, device="cuda")
    return (rnd(M, H), rnd(E, I, H, scale=H ** -0.5), rnd(E, I, H, scale=H ** -0.5), rnd(E, H, I, scale=I ** -0.5),
            off)


def _reference(x, wg, wu, wd, rows):
    h, y, mag, r0 = [], [], [], 0
    for e, n in enumerate(rows):
        xe = x[r0:r0 + n].float()
        gate, up = xe @ wg[e].float().t(), xe @ wu[e].float().t()
        he = (gate * torch.sigmoid(gate) * up).bfloat16().float()
        h.append(he)
        y.append(he @ wd[e].float().t())
        mag.append(he.abs() @ wd[e].float().abs().t())
        r0 += n
    return torch.cat(h), torch.cat(y), torch.cat(mag)


def _np(t, M):
    """Rows to compare on the host: all of a small call, else the ends of it."""
    t = t[:M]
    return (t if M <= 3000 else torch.cat([t[:600], t[M // 2 - 300:M // 2 + 300], t[-600:]])).float().cpu().numpy()


@pytest.mark.parametrize("H,I,rows", CASES, ids=IDS)
def test_bf16(H, I, rows):
    print("CASE large tile bf16", H, I, rows, flush=True)
    x, wg, wu, wd, off = _inputs(H, I, rows, 1)
    M, E = x.shape[0], len(rows)
    cap = max(M, 1024 * E)
    perm = torch.randperm(M, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    src = torch.zeros(cap, dtype=torch.int32, device="cuda")
    src[:M] = perm.int()  # row r of the experts' input is token perm[r] of the shuffled tokens
    tokens = torch.empty_like(x)
    tokens[perm] = x
    got = []
    for layer in (256, E, 0):
        y = torch.full((cap, H), float("nan"), dtype=x.dtype, device="cuda")
        ws = torch.zeros(moe.ffn_ws_bytes(E, H, I, cap, x.dtype), dtype=torch.uint8, device="cuda")
        moe.moe_grouped_swiglu_ffn_gather(tokens, src, 1, wg, wu, wd, off, ws=ws, y_perm=y, experts=layer)
        torch.cuda.synchronize()
        assert int(ws[:moe.FFN_COUNTER_BYTES].view(torch.int32).abs().sum()) == 0, f"work counters, layer of {layer}"
        assert bool(y[M:].isnan().all()), "rows past the last expert are left alone"
        got.append((moe.ffn_hidden(ws, cap, I, x.dtype)[:M].clone(), y[:M]))
    for h, y in got[1:]:
        assert torch.equal(h, got[0][0]) and torch.equal(y, got[0][1])
    xb = torch.zeros((cap, H), dtype=x.dtype, device="cuda")
    xb[:M] = x
    y, _ = moe.moe_grouped_swiglu_ffn(xb, wg, wu, wd, off)
    if max(rows) > 128:  # with fewer rows the permuted call may split differently
        assert torch.equal(y[:M], got[0][1]), "permuted rows"
    h, y, mag = _reference(x, wg, wu, wd, rows)
    G.check_bf16(_np(got[0][0], M), _np(h, M), "h")
    G.check_bf16(_np(got[0][1], M), _np(y, M), "y", scale=_np(mag, M))


def _values(codes, scales):
    """The values of MXFP8 codes [R, K] with scale dwords [K/128, R], and the scale
    of each, in 64 bits."""
    R, K = codes.shape
    c = scales.t().contiguous().view(torch.uint8).reshape(R, K // 32).double()
    s = torch.exp2(c - 127.0).repeat_interleave(32, dim=1)
    return codes.contiguous().view(torch.float8_e4m3fn).float().double() * s, s


@pytest.mark.parametrize("H,I,rows", CASES, ids=IDS)
def test_mx(H, I, rows):
    """H = 4224 and I = 4224: an odd number (33) of 128-element chunks."""
    print("CASE large tile mx", H, I, rows, flush=True)
    M, E = sum(rows), len(rows)
    cap = max(M, 1024 * E)
    empty = cap // 1024 + 1 - E
    x, wg, wu, wd, off = _inputs(H, I, rows, 3, empty)
    xb = torch.zeros((cap, H), dtype=x.dtype, device="cuda")
    xb[:M] = x
    xq = moe.moe_mx_quantize(xb)
    w = [moe.moe_mx_quantize(t) for t in (wg, wu, wd)]
    w8 = [moe.MxTensor(torch.cat([t.codes, t.codes[:1].expand(empty, -1, -1)]),
                       torch.cat([t.scales, t.scales[:1].expand(empty, -1, -1)])) for t in w]
    got = []
    for wt, o in ((w8, off), (w, off[:E + 1].contiguous())):
        y = torch.full((cap, H), float("nan"), dtype=x.dtype, device="cuda")
        y, ws = moe.moe_grouped_swiglu_ffn_mx(xq, *wt, o, y_perm=y)
        torch.cuda.synchronize()
        assert int(ws[:moe.FFN_COUNTER_BYTES].view(torch.int32).abs().sum()) == 0, "work counters"
        assert bool(y[M:].isnan().all()), "rows past the last expert are left alone"
        at = moe.FFN_COUNTER_BYTES + (cap * I + 255) // 256 * 256  # h codes, then their scales
        codes = ws[moe.FFN_COUNTER_BYTES:moe.FFN_COUNTER_BYTES + M * I].view(M, I).clone()
        scales = ws[at:at + I // 128 * cap * 4].view(torch.int32).view(I // 128, cap)[:, :M].clone()
        got.append((codes, scales, y[:M]))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    codes, scales, y = got[1]
    xv = _values(xq.codes[:M], xq.scales[:, :M])[0]
    hv, step = _values(codes, scales)
    r0 = 0
    for e, n in enumerate(rows):
        r, r0 = slice(r0, r0 + n), r0 + n
        g, u, d = (_values(t.codes[e], t.scales[e])[0] for t in w)
        a, b = xv[r] @ g.t(), xv[r] @ u.t()
        h = a * torch.sigmoid(a) * b
        # fp32 sums of K products: K 2^-23 of their magnitudes; |silu'| <= 1.1
        da, db = (H * 2.0 ** -23 * (xv[r].abs() @ t.abs().t()) for t in (g, u))
        dh = 1.1 * da * (b.abs() + db) + a.abs() * db
        # E4M3: half a step is 2^-4 of the value, or 2^-10 of the scale below its
        # normal range; above 448 scales (the block's largest values) 2^-3
        assert bool(((hv[r] - h).abs() <= 2.0 ** -3 * (h.abs() + dh) + 2.0 ** -10 * step[r] + dh).all()), f"h {e}"
        ref = hv[r] @ d.t()
        dy = I * 2.0 ** -23 * (hv[r].abs() @ d.abs().t())
        assert bool(((y[r].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + dy).all()), f"y {e}"


@pytest.mark.parametrize("layer", [0, 1])
def test_captured(layer):
    """Both kernels launched and the offsets choosing (layer unknown), or 4 waves:
    replays of a graph give the eager bits, with other rows in between."""
    H, I, rows = 4224, 512, [1100]
    x, wg, wu, wd, off = _inputs(H, I, rows, 5)
    M = x.shape[0]
    src = torch.arange(M, dtype=torch.int32, device="cuda")
    ws = torch.zeros(moe.ffn_ws_bytes(1, H, I, M, x.dtype), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)

    def call():
        moe.moe_grouped_swiglu_ffn_gather(x, src, 1, wg, wu, wd, off, ws=ws, y_perm=y, experts=layer)

    call()
    torch.cuda.synchronize()
    few = off.clone()
    few[1] = 40  # a launch for the 8-wave kernel where the offsets choose
    full, want = off.clone(), []
    for o in (full, few):
        off.copy_(o)
        y.fill_(float("nan"))
        call()
        want.append(y.clone())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in (0, 1, 0, 1):
        off.copy_((full, few)[i])
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), want[i].view(torch.int16)), i
