"""The 4-wave GEMM launches (large 256-row tile, even and odd chunk counts,
small and mid tiles, decode schedule, splits) against the 8-wave ones.

Which kernel a launch takes depends on M_cap per local expert, so the same
routed rows run twice: with M_cap just their number (8 waves, unless the rows
themselves are many) and with M_cap raised to 4096 rows per expert or more (4 waves).
Both sum each output over K in ascending order, so unsplit results agree bit
for bit; split ones (M_cap also sizes the workspace) within the bf16 rule of
gpu_helpers. The bf16 results are also held to a plain fp32 computation."""
import pytest
import torch

import gpu_helpers as G
import paper_2606_00735_amd as moe

pytestmark = pytest.mark.gpu

CASES = [
    # H, I, rows per expert: chunk counts H/64, I/64 of 2 to 64;
    # rows at the edges of the 64-, 128- and 256-row classes, empty experts,
    # full and ragged last tiles
    (128, 256, [1, 64, 65, 128, 129, 255, 256, 257]),
    (384, 640, [300, 0, 513, 191]),
    (896, 128, [1000, 2, 320]),
    (2048, 384, [257, 255, 640, 60]),
    (256, 2048, [5]),
    (1024, 512, [16, 3, 0, 60]),
    (4096, 384, [5000, 4500]),  # enough tiles for the down GEMM's 256-column ones
]


def _inputs(H, I, rows, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def rnd(*s, scale=1.0):
        return (torch.randn(*s, generator=g, device="cuda") * scale).bfloat16()

    E, M = len(rows), sum(rows)
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32, device="cuda")
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


def _np(t):
    return t.float().cpu().numpy()


@pytest.mark.parametrize("H,I,rows", CASES, ids=[f"H{h}-I{i}-E{len(r)}" for h, i, r in CASES])
def test_bf16(H, I, rows):
    print("CASE large tile bf16", H, I, rows, flush=True)
    x, wg, wu, wd, off = _inputs(H, I, rows, 1)
    M = x.shape[0]
    cap = max(M, 4096 * len(rows), 2**25 // H)
    xb = torch.zeros((cap, H), dtype=x.dtype, device="cuda")
    xb[:M] = x
    y8, ws8 = moe.moe_grouped_swiglu_ffn(x, wg, wu, wd, off)
    y4 = torch.full((cap, H), float("nan"), dtype=x.dtype, device="cuda")
    y4, ws4 = moe.moe_grouped_swiglu_ffn(xb, wg, wu, wd, off, y_perm=y4)
    perm = torch.randperm(M, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    src = torch.zeros(cap, dtype=torch.int32, device="cuda")
    src[:M] = perm.int()  # row r of the experts' input is token perm[r] of the shuffled tokens
    tokens = torch.empty_like(x)
    tokens[perm] = x
    yg, _ = moe.moe_grouped_swiglu_ffn_gather(tokens, src, 1, wg, wu, wd, off)
    torch.cuda.synchronize()
    assert int(ws4[:16384].view(torch.int32).abs().sum()) == 0, "work counters"
    assert bool(y4[M:].isnan().all()), "rows past the last expert are left alone"
    assert torch.equal(yg[:M], y4[:M]), "gathered rows"
    h, y, mag = _reference(x, wg, wu, wd, rows)
    G.check_bf16(_np(moe.ffn_hidden(ws4, cap, I, x.dtype)[:M]), _np(h), "h")
    G.check_bf16(_np(y4[:M]), _np(y), "y", scale=_np(mag))
    G.check_bf16(_np(y4[:M]), _np(y8), "4 against 8 waves", scale=_np(mag))


@pytest.mark.parametrize("H,I,rows", CASES, ids=[f"H{h}-I{i}-E{len(r)}" for h, i, r in CASES])
def test_mx(H, I, rows):
    """H = 384, 896 and I = 384, 640: an odd number of 128-element chunks."""
    print("CASE large tile mx", H, I, rows, flush=True)
    x, wg, wu, wd, off = _inputs(H, I, rows, 3)
    M = x.shape[0]
    cap = max(M, 4096 * len(rows), 2**25 // H)
    xb = torch.zeros((cap, H), dtype=x.dtype, device="cuda")
    xb[:M] = x
    w = [moe.moe_mx_quantize(t) for t in (wg, wu, wd)]
    y8, _ = moe.moe_grouped_swiglu_ffn_mx(moe.moe_mx_quantize(x), *w, off)
    y4 = torch.full((cap, H), float("nan"), dtype=x.dtype, device="cuda")
    y4, _ = moe.moe_grouped_swiglu_ffn_mx(moe.moe_mx_quantize(xb), *w, off, y_perm=y4)
    torch.cuda.synchronize()
    assert bool(y4[M:].isnan().all()), "rows past the last expert are left alone"
    a, b = y4[:M].float(), y8.float()
    # a code of h one step off (a tie decided the other way by another order
    # of the fp32 sums) moves an output by at most 2^-3 of one product
    assert float((a - b).norm()) <= 2e-3 * float(b.norm())
    _, y, _ = _reference(x, wg, wu, wd, rows)
    assert float((a - y).norm()) <= 0.08 * float(y.norm())  # E4M3 rounding of x, w and h: about 0.04
