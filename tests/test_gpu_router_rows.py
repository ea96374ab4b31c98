"""The router's K-split tiles at the row counts where their partial logits leave
by another way (64 of a tile's 256 rows): one tile and a ragged last one. Inputs
sit on grids where every sum is exact, so the logits are."""
import pytest
import torch

import paper_2606_00735_amd as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,H", [(256, 2048), (128, 5120)])
@pytest.mark.parametrize("T", [1, 31, 63, 64, 65, 255, 257, 320, 321])
def test_logits(T, E, H):
    print("CASE router rows", T, E, H, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randint(-16, 17, (T, H), generator=g, device="cuda").bfloat16() / 16
    w = torch.randint(-16, 17, (E, H), generator=g, device="cuda").bfloat16() / 16
    b = torch.randint(-16, 17, (E,), generator=g, device="cuda").float() / 16
    lg = torch.full((T, E), float("nan"), device="cuda")
    ids, _, _ = moe.moe_gate_topk(x, w, b, 4, logits=lg)
    torch.cuda.synchronize()
    z = x.double() @ w.double().t() + b.double()
    assert torch.equal(lg.double(), z)
    assert torch.equal(ids.long(), torch.sort(z, dim=1, descending=True, stable=True)[1][:, :4])
