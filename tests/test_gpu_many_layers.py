"""Placement of many layers at once: outputs where the models stay in global
memory (more layers than CUs and more than 1024 knots) and where LDS holds them,
against the oracle; and that a launch of many small layers keeps several blocks
on a CU (its time, against a launch of one block a CU)."""
import numpy as np
import pytest
import torch

import paper_2606_00735_amd as moe
from oracle import placement_oracle as P

pytestmark = pytest.mark.gpu


def _problem(L, E, G, nk, seed):
    r = np.random.default_rng(seed)
    W = r.uniform(0.0, 100.0, (L, E)) ** 2
    kn = np.cumsum(r.uniform(1.0, 4.0, (G, nk)), axis=1) * W.sum(1).mean() / (2 * G * nk)
    kt = 20.0 + np.cumsum(r.uniform(0.0, 3.0, (G, nk)), axis=1)
    return W, kn, kt, r.integers(0, G, (L, E))


def _dev(a, dt=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt)


def best_us(call, n=20):
    """The shortest of several timed runs of n calls, us a call."""
    for _ in range(5):
        call()
    best = float("inf")
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / n * 1e3)
    return best


@pytest.mark.parametrize("L,E,G,nk", [(300, 65, 64, 17), (300, 65, 64, 16), (259, 9, 3, 2), (2, 65, 64, 17)])
def test_matches_oracle(L, E, G, nk):
    print("CASE many layers", L, E, G, nk, flush=True)
    W, kn, kt, start = _problem(L, E, G, nk, E + nk)
    dW, dn, dt = _dev(W), _dev(kn), _dev(kt)
    a, n, tau = (t.cpu().numpy() for t in moe.moe_place_greedy(dW, dn, dt))
    u = _dev(start, torch.int32)
    swaps = moe.moe_place_incremental(dW, dn, dt, u, eps=0.02, max_swaps=3).cpu().numpy()
    u = u.cpu().numpy()
    c = [t.cpu().numpy() for t in moe.moe_placement_cost(dW, _dev(start, torch.int32), dn, dt)]
    for l in sorted({0, 1, L // 2, L - 1}):
        ra, rn, rt = P.greedy_placement(W[l], kn, kt)
        assert np.array_equal(a[l], ra) and np.array_equal(n[l], rn) and np.array_equal(tau[l], rt), f"layer {l}"
        ru, rs = P.incremental_update(start[l], W[l], kn, kt, eps=0.02, max_swaps=3)
        assert np.array_equal(u[l], ru) and swaps[l] == rs, f"layer {l}"
        cn = P.gpu_loads(start[l], W[l], G)
        assert np.array_equal(c[0][l], cn), f"layer {l}"
        assert np.array_equal(c[1][l], [P.latency(kn[g], kt[g], cn[g]) for g in range(G)]), f"layer {l}"
        assert c[2][l].max() == P.layer_latency(start[l], W[l], kn, kt, grouped=True), f"layer {l}"


def test_blocks_share_a_cu():
    """1024 small layers are at most four blocks a CU: about the time of 64 (one
    block a CU would take four times as long)."""
    def times(L):
        W, kn, kt, start = _problem(L, 64, 8, 4, 7)
        W, kn, kt, a = _dev(W), _dev(kn), _dev(kt), _dev(start, torch.int32)
        lo, ta = (torch.empty((L, 8), dtype=torch.float64, device="cuda") for _ in range(2))
        sw = torch.empty(L, dtype=torch.int32, device="cuda")
        u = a.clone()

        def incremental():  # one swap a call, from wherever the last left it
            moe.moe_place_incremental(W, kn, kt, u, eps=0.0, max_swaps=1, n_swaps=sw)

        return (best_us(lambda: moe.moe_place_greedy(W, kn, kt, assign=a, loads=lo, targets=ta)),
                best_us(incremental))

    few, many = times(64), times(1024)
    print("greedy, incremental us: 64 layers", few, "1024 layers", many, flush=True)
    assert many[0] <= 2.0 * few[0]
    assert many[1] <= 2.0 * few[1]


@pytest.mark.parametrize("L,E", [(1, 12), (257, 3), (600, 63), (4096, 16), (65, 64), (300, 130)])
def test_drift_matches_oracle(L, E):
    print("CASE drift", L, E, flush=True)
    W, _, _, _ = _problem(L, E, 2, 1, L)
    V, _, _, _ = _problem(L, E, 2, 1, L + 1)
    W[0] = 0.0
    d, trig = moe.moe_drift_distance(_dev(W), _dev(V), delta=0.05)
    d = d.cpu().numpy()
    for l in range(L):
        assert d[l] == P.cosine_distance(W[l], V[l]), f"layer {l}"
    assert int(trig.item()) == int(d.max() > 0.05)


def test_drift_of_few_experts():
    """The same loads as 4096 layers of 16 experts and as 1024 of 64: about the
    same time (with waves three quarters empty the first takes 2.7 times as long)."""
    W, _, _, _ = _problem(1024, 64, 2, 1, 3)
    us = []
    for L, E in ((1024, 64), (4096, 16)):
        w, d = _dev(W).view(L, E), torch.empty(L, dtype=torch.float64, device="cuda")
        t = torch.empty(1, dtype=torch.int32, device="cuda")
        us.append(best_us(lambda: moe.moe_drift_distance(w, w, d=d, trigger=t)))
    print("drift us", us, flush=True)
    assert us[1] <= 1.7 * us[0]
