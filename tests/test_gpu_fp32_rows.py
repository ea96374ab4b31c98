"""The fp32 FFN's rows: more than one pass of the grid, rows of no expert before,
between and after the experts' own, offsets that go down (that expert has none),
and a launch whose M_cap is mostly rows of remote experts.

Bound of an fp32 dot product of K terms in any order: (K + 2) 2^-24 sum |a b|."""
import pytest
import torch

import paper_2606_00735_amd as moe
from test_gpu_many_layers import best_us

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24

CASES = [
    # H, I, M_cap, offsets
    (8, 8, 9000, [0, 2500, 2500, 8999]),          # several passes over the rows
    (32, 40, 3000, [5, 9, 9, 1400, 2990]),        # rows before the first expert and after the last
    (16, 8, 40, [7, 3, 20, 20, 35]),              # expert 0: 7 to 3, i.e. none
    (8, 260, 5000, [0, 1, 1, 4000]),              # several blocks of columns
    (8, 8, 2000, [0] * 70 + [1500, 1600]),        # more experts than one lookup takes
    (8, 8, 12, [-4, 5, 90]),                      # clamped to [0, M_cap]
]


@pytest.mark.parametrize("H,I,cap,off", CASES, ids=[f"H{c[0]}-I{c[1]}-cap{c[2]}-E{len(c[3]) - 1}" for c in CASES])
def test_rows(H, I, cap, off):
    print("CASE fp32 rows", H, I, cap, off[:6], flush=True)
    E = len(off) - 1
    g = torch.Generator(device="cuda").manual_seed(H + cap)

    def rnd(*s):
        return torch.randn(*s, generator=g, device="cuda") * s[-1] ** -0.5

    x, wg, wu, wd = rnd(cap, H), rnd(E, I, H), rnd(E, I, H), rnd(E, H, I)
    y = torch.full((cap, H), float("nan"), device="cuda")
    y, ws = moe.moe_grouped_swiglu_ffn(x, wg, wu, wd, torch.tensor(off, dtype=torch.int32, device="cuda"), y_perm=y)
    torch.cuda.synchronize()
    h = moe.ffn_hidden(ws, cap, I, x.dtype).double()
    none = torch.ones(cap, dtype=torch.bool, device="cuda")
    for e in range(E):
        a = min(max(off[e], 0), cap)
        b = min(max(off[e + 1], a), cap)
        rows = torch.arange(a, b, device="cuda")
        rows = rows[none[rows]]
        if rows.numel() == 0:
            continue
        none[rows] = False
        xe, he = x[rows].double(), h[rows]
        p, u = xe @ wg[e].double().t(), xe @ wu[e].double().t()
        dp, du = ((H + 2) * EPS * (xe.abs() @ w[e].double().abs().t()) for w in (wg, wu))
        # |silu'| <= 1.1 and |silu(p)| <= |p|; expf, division and products: 8 roundings
        ref = p * torch.sigmoid(p) * u
        assert bool(((he - ref).abs() <= 1.1 * dp * (u.abs() + du) + p.abs() * du + 8 * EPS * ref.abs()).all()), e
        dy = (I + 2) * EPS * (he.abs() @ wd[e].double().abs().t())
        assert bool(((y[rows].double() - he @ wd[e].double().t()).abs() <= dy).all()), e
    assert bool(y[none].isnan().all()), "rows of no expert are left alone"


def test_remote_rows_cost_little():
    """128 rows with M_cap = 128 and with M_cap = 65536: about the same time (a
    block per row of M_cap takes twenty times as long)."""
    H, I = 128, 256
    w = [torch.randn(s, device="cuda") * s[-1] ** -0.5 for s in ((1, I, H), (1, I, H), (1, H, I))]
    off = torch.tensor([0, 128], dtype=torch.int32, device="cuda")
    us = []
    for cap in (128, 65536):
        x = torch.randn((cap, H), device="cuda")
        y = torch.empty_like(x)
        ws = torch.zeros(moe.ffn_ws_bytes(1, H, I, cap, x.dtype), dtype=torch.uint8, device="cuda")
        us.append(best_us(lambda: moe.moe_grouped_swiglu_ffn(x, *w, off, ws=ws, y_perm=y)))
    print("fp32 us", us, flush=True)
    assert us[1] <= 4.0 * us[0]
