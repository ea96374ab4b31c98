"""A load sweep measures each load on the kernels that a call of that load takes:
the time of a small load does not depend on the largest one in the list."""
import pytest
import torch

import paper_2606_00735_amd as moe

pytestmark = pytest.mark.gpu


def test_mx_small_load_beside_a_large_one():
    """64 rows, DSV3-shaped: 4-wave kernels (for the large loads) take 1.3 times as
    long; beside a large load the reduction launches come on top."""
    H, I, n = 7168, 2048, 8
    g = torch.Generator(device="cuda").manual_seed(1)
    w = [moe.moe_mx_quantize(torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) * s[-1] ** -0.5)
         for s in ((n, I, H), (n, I, H), (n, H, I))]
    us = []
    for Ms in ([64], [64, 4096]):
        x = moe.moe_mx_quantize(torch.randn((max(Ms), H), generator=g, device="cuda", dtype=torch.bfloat16))
        us.append(min(float(moe.moe_load_sweep_mx(x, *w, Ms, warmup=5, iters=50)[0][0]) for _ in range(3)))
    print("64 rows, us: alone", us[0], "beside 4096", us[1], flush=True)
    assert us[1] <= 1.2 * us[0]
