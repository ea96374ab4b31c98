"""What every block of a grouped GEMM derives from the expert offsets (tiles and
rows of the experts before its own, counts by size): experts at the edges of the
waves that scan them, empty ones at either end, one far larger than the rest, on
the decode schedule and in rounds of tiles."""
import pytest
import torch

import gpu_helpers as G
import paper_2606_00735_amd as moe

pytestmark = pytest.mark.gpu
H = I = 128


def _rows(E, kind):
    g = torch.Generator().manual_seed(E)
    if kind == "decode":  # at most 16 rows an expert
        r = torch.randint(0, 17, (E,), generator=g)
    else:                 # tiles of every class
        r = torch.tensor([0, 1, 17, 64, 65, 129, 257])[torch.randint(0, 7, (E,), generator=g)]
        r[E // 2] = 700
    if E > 2:
        r[0] = r[E - 1] = 0
    return r.tolist()


@pytest.mark.parametrize("kind", ["decode", "rounds"])
@pytest.mark.parametrize("E", [1, 63, 64, 65, 128, 193, 256])
def test_offsets_to_tiles(E, kind):
    print("CASE expert scan", E, kind, flush=True)
    rows = _rows(E, kind)
    M = sum(rows)
    g = torch.Generator(device="cuda").manual_seed(E)

    def rnd(*s):
        return (torch.randn(*s, generator=g, device="cuda") * s[-1] ** -0.5).bfloat16()

    x, wg, wu, wd = rnd(M + 3, H) * 8, rnd(E, I, H), rnd(E, I, H), rnd(E, H, I)
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32, device="cuda")
    y = torch.full((M + 3, H), float("nan"), dtype=x.dtype, device="cuda")
    y, ws = moe.moe_grouped_swiglu_ffn(x, wg, wu, wd, off, y_perm=y)
    torch.cuda.synchronize()
    assert int(ws[:moe.FFN_COUNTER_BYTES].view(torch.int32).abs().sum()) == 0, "work counters"
    assert bool(y[M:].isnan().all()), "rows past the last expert are left alone"
    e = torch.repeat_interleave(torch.arange(E), torch.tensor(rows)).cuda()
    h = torch.empty((M, I), device="cuda")
    ref = torch.empty((M, H), device="cuda")
    mag = torch.empty((M, H), device="cuda")
    for i in range(E):
        s = (e == i).nonzero().flatten()
        if s.numel():
            a, u = x[s].float() @ wg[i].float().t(), x[s].float() @ wu[i].float().t()
            h[s] = (a * torch.sigmoid(a) * u).bfloat16().float()
            ref[s] = h[s] @ wd[i].float().t()
            mag[s] = h[s].abs() @ wd[i].float().abs().t()
    G.check_bf16(moe.ffn_hidden(ws, M + 3, I, x.dtype)[:M].float().cpu().numpy(), h.cpu().numpy(), "h")
    G.check_bf16(y[:M].float().cpu().numpy(), ref.cpu().numpy(), "y", scale=mag.cpu().numpy())
