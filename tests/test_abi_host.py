"""CPU tests of the C ABI: the library loads, exports what include/moe.h
declares, and rejects bad arguments on the host before launching anything.

None of these calls reaches a kernel launch (every one fails validation or is
a workspace-size query), so they run without a GPU.
"""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2606_00735_amd as moe
from paper_2606_00735_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INVALID, UNSUPPORTED, WORKSPACE = 1, 2, 3


@pytest.fixture(scope="module")
def L():
    return moe.load_library()


def declared_functions():
    text = open(os.path.join(ROOT, "include", "moe.h")).read()
    return sorted(set(re.findall(r"^\s*(?:moe_status|const char\*|int|size_t)\s+(moe_\w+)\s*\(", text, re.M)))


def test_header_declares_the_six_entry_points():
    names = declared_functions()
    for n in ("moe_gate_topk", "moe_expert_histogram_scan", "moe_permute", "moe_grouped_swiglu_ffn",
              "moe_unpermute_combine", "moe_load_sweep"):
        assert n in names
    assert set(names) == set(_lib.EXPORTED)


def test_library_exports_every_declared_symbol(L):
    import subprocess
    out = subprocess.run(["nm", "-D", "--defined-only", moe.LIB_PATH], capture_output=True, text=True).stdout
    exported = set(re.findall(r" T (moe_\w+)$", out, re.M))
    for n in declared_functions():
        assert n in exported, n
        assert hasattr(L, n)


def test_version_and_status_strings(L):
    assert L.moe_abi_version() == 3
    assert L.moe_status_string(0) == b"ok"
    assert L.moe_status_string(3) == b"workspace too small"
    assert L.moe_status_string(99) == b"unknown status"


FAKE = ctypes.c_void_p(0x10000)      # aligned, never dereferenced: validation fails first
MISALIGNED = ctypes.c_void_p(0x10004)


@pytest.mark.parametrize("T,H,E,k,dt,expect", [
    (4, 128, 8, 9, 1, INVALID),     # k > E
    (4, 128, 8, 0, 1, INVALID),     # k = 0
    (4, 128, 300, 2, 1, INVALID),   # E > 256
    (4, 128, 32, 17, 1, INVALID),   # k > 16
    (-1, 128, 8, 2, 1, INVALID),    # T < 0
    (4, 100, 8, 2, 0, INVALID),     # H % 8
    (4, 72, 8, 2, 1, UNSUPPORTED),  # bf16 needs H % 64
    (4, 128, 8, 2, 7, INVALID),     # bad dtype
])
def test_gate_topk_validation(L, T, H, E, k, dt, expect):
    st = L.moe_gate_topk(FAKE, FAKE, None, T, H, E, k, dt, None, FAKE, FAKE, None, None, None)
    assert st == expect


def test_gate_topk_workspace(L):
    """The router's workspace: a size query that launches nothing, 0 where it
    is not used, and the size checked when one is given."""
    n = ctypes.c_size_t(123)
    assert L.moe_gate_topk(None, None, None, 16384, 7168, 256, 8, 1, None, None, None, None, ctypes.byref(n),
                           None) == 0
    big = n.value
    assert big >= 16384 * 256 * 4 and big % 256 == 0
    for T, H, E in ((1, 2048, 128), (128, 2048, 128), (4096, 5120, 128), (8192, 5120, 128), (8193, 5120, 128),
                    (16384, 5120, 128), (512, 7168, 256),
                    (32, 4096, 8),
                    (16, 4096, 8), (256, 2048, 96)):
        assert L.moe_gate_topk(None, None, None, T, H, E, 1, 1, None, None, None, None, ctypes.byref(n),
                               None) == 0
        assert n.value >= T * E * 4, (T, H, E)
    # (no GPU here: the launcher assumes 256 CUs, so rows of 5120 split up to
    # 16384 tokens, 128 blocks of 128 tokens)
    for T, H, E, dt in ((16384, 7168, 256, 0), (8192, 2048, 128, 1), (16385, 5120, 128, 1), (32768, 5120, 128, 1),
                        (16384, 4096, 8, 1),
                        (4096, 2048, 96, 1),
                        (257, 4096, 8, 1), (32, 1088, 8, 1), (1, 4096, 8, 1), (15, 4096, 8, 1)):
        n = ctypes.c_size_t(123)
        assert L.moe_gate_topk(None, None, None, T, H, E, 2, dt, None, None, None, None, ctypes.byref(n),
                               None) == 0
        assert n.value == 0, (T, H, E, dt)
    n = ctypes.c_size_t(big - 1)
    assert L.moe_gate_topk(FAKE, FAKE, None, 16384, 7168, 256, 8, 1, None, FAKE, FAKE, FAKE, ctypes.byref(n),
                           None) == WORKSPACE
    assert L.moe_gate_topk(FAKE, FAKE, None, 16384, 7168, 256, 8, 1, None, FAKE, FAKE, FAKE, None,
                           None) == INVALID
    n = ctypes.c_size_t(big)
    assert L.moe_gate_topk(FAKE, FAKE, None, 16384, 7168, 256, 8, 1, None, FAKE, FAKE, MISALIGNED,
                           ctypes.byref(n), None) == INVALID


def test_gate_topk_null_and_alignment(L):
    assert L.moe_gate_topk(None, FAKE, None, 4, 128, 8, 2, 1, None, FAKE, FAKE, None, None, None) == INVALID
    assert L.moe_gate_topk(MISALIGNED, FAKE, None, 4, 128, 8, 2, 1, None, FAKE, FAKE, None, None, None) == INVALID
    assert L.moe_gate_topk(None, None, None, 0, 128, 8, 2, 1, None, None, None, None, None, None) == 0  # T=0 no-op


def _hist(L, emap, T=64, k=2, E=8, E_local=None, ws=FAKE, nbytes=10 ** 9):
    emap = np.asarray(emap, np.int32)
    E_local = int((emap >= 0).sum()) if E_local is None else E_local
    n = ctypes.c_size_t(nbytes)
    return L.moe_expert_histogram_scan(FAKE, T, k, E, emap.ctypes.data_as(ctypes.c_void_p), E_local,
                                       ctypes.c_void_p(None), FAKE, ws, ctypes.byref(n), None), n.value


def test_histogram_workspace_query(L):
    st, n = _hist(L, np.arange(8), ws=ctypes.c_void_p(None), nbytes=0)
    assert st == 0 and n >= 1 * 8 * 4
    st, n2 = _hist(L, np.arange(8), T=16384, k=8, E=256, ws=ctypes.c_void_p(None), nbytes=0)
    assert st == 0 and n2 >= 256 * 4 and n2 > n
    st, _ = _hist(L, np.arange(8), nbytes=n - 1)
    assert st == WORKSPACE


@pytest.mark.parametrize("emap", [
    [0, 1, 2, 3, 4, 5, 6, 6],          # slot used twice
    [0, 1, 2, 3, 4, 5, 6, 8],          # slot out of range
    [0, 1, 2, 3, 4, 5, -2, 7],         # below -1
    [-1, 1, 2, 3, 4, 5, 6, 7],         # slot 0 unused
])
def test_histogram_rejects_bad_expert_map(L, emap):
    emap = np.asarray(emap, np.int32)
    st, _ = _hist(L, emap, E_local=7 if (emap == -1).any() else 8)
    assert st == INVALID


def test_histogram_counts_pointer_required(L):
    st, _ = _hist(L, np.arange(8))   # counts = NULL
    assert st == INVALID


def test_permute_validation(L):
    emap = np.arange(8, dtype=np.int32)
    p = emap.ctypes.data_as(ctypes.c_void_p)
    # M_cap < T*k
    assert L.moe_permute(FAKE, FAKE, p, FAKE, 10 ** 9, 64, 128, 2, 8, 8, 100, 1, FAKE, FAKE, FAKE,
                         None) == INVALID
    # workspace too small
    assert L.moe_permute(FAKE, FAKE, p, FAKE, 8, 64, 128, 2, 8, 8, 128, 1, FAKE, FAKE, FAKE, None) == WORKSPACE
    # E_local does not match the map
    assert L.moe_permute(FAKE, FAKE, p, FAKE, 10 ** 9, 64, 128, 2, 8, 7, 128, 1, FAKE, FAKE, FAKE,
                         None) == INVALID


def test_ffn_validation_and_query(L):
    n = ctypes.c_size_t(0)
    assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 8, 4096, 14336, 0, 0, 8192, 1, None, None,
                                    ctypes.byref(n), None) == 0
    assert n.value >= 8192 * 14336 * 2
    for H, I in ((4096, 14300), (4000, 14336)):
        assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 8, H, I, 0, 0, 64, 1, None, None,
                                        ctypes.byref(n), None) == UNSUPPORTED
    assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 300, 128, 128, 0, 0, 64, 1, None, None,
                                    ctypes.byref(n), None) == UNSUPPORTED
    n = ctypes.c_size_t(10)
    assert L.moe_grouped_swiglu_ffn(FAKE, FAKE, FAKE, FAKE, FAKE, 8, 128, 256, 0, 0, 64, 1, FAKE, FAKE,
                                    ctypes.byref(n), None) == WORKSPACE


def test_ffn_weight_row_strides(L):
    # padded rows: accepted (and the workspace does not depend on them)
    n, m = ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 8, 4096, 14336, 0, 0, 64, 1, None, None,
                                    ctypes.byref(n), None) == 0
    assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 8, 4096, 14336, 4160, 14344, 64, 1, None, None,
                                    ctypes.byref(m), None) == 0
    assert n.value == m.value
    # fp32: a multiple of 4 elements; bf16: of 8 (16-byte rows)
    assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 8, 128, 256, 132, 260, 64, 0, None, None,
                                    ctypes.byref(m), None) == 0
    for gu, dn, dt in ((4095, 0, 1), (4100, 0, 1), (0, 14337, 1), (0, 14340, 1), (130, 0, 0), (4097, 0, 1),
                       (1 << 21, 0, 1), (-8, 0, 1)):
        H, I = (4096, 14336) if dt == 1 else (128, 256)
        assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, 8, H, I, gu, dn, 64, dt, None, None,
                                        ctypes.byref(m), None) == INVALID, (gu, dn, dt)
        assert L.moe_grouped_swiglu_ffn_gather(None, None, 64, 2, None, None, None, None, 8, H, I, gu, dn, 64, 1,
                                               None, None, ctypes.byref(m), None) in (INVALID, UNSUPPORTED)
    Ms = np.array([1, 2], np.int32)
    assert L.moe_load_sweep(None, None, None, None, 1, 2048, 768, 2056, 776, 1, Ms.ctypes.data_as(ctypes.c_void_p),
                            2, 1, 5, None, None, ctypes.byref(m), None, None, None) == 0
    assert L.moe_load_sweep(None, None, None, None, 1, 2048, 768, 2047, 0, 1, Ms.ctypes.data_as(ctypes.c_void_p),
                            2, 1, 5, None, None, ctypes.byref(m), None, None, None) == INVALID


def test_ffn_gather_validation_and_query(L):
    n, m = ctypes.c_size_t(0), ctypes.c_size_t(0)
    args = (8, 4096, 14336, 0, 0, 8192)
    assert L.moe_grouped_swiglu_ffn_gather(None, None, 4096, 2, None, None, None, None, *args, 1, None, None,
                                           ctypes.byref(n), None) == 0
    assert L.moe_grouped_swiglu_ffn(None, None, None, None, None, *args, 1, None, None, ctypes.byref(m), None) == 0
    assert n.value == m.value  # the same workspace
    # fp32 has no gathering variant
    assert L.moe_grouped_swiglu_ffn_gather(None, None, 64, 2, None, None, None, None, 8, 128, 128, 0, 0, 128, 0,
                                           None, None, ctypes.byref(n), None) == UNSUPPORTED
    for T, k in ((0, 2), (64, 0), (64, 17)):
        assert L.moe_grouped_swiglu_ffn_gather(None, None, T, k, None, None, None, None, 8, 128, 128, 0, 0, 128,
                                               1, None, None, ctypes.byref(n), None) == INVALID
    # row offsets into x must fit 32 bits
    assert L.moe_grouped_swiglu_ffn_gather(None, None, 1 << 20, 1, None, None, None, None, 8, 4096, 128, 0, 0,
                                           1 << 20, 1, None, None, ctypes.byref(n), None) == UNSUPPORTED
    n = ctypes.c_size_t(10)
    assert L.moe_grouped_swiglu_ffn_gather(FAKE, FAKE, 64, 2, FAKE, FAKE, FAKE, FAKE, 8, 128, 256, 0, 0, 128, 1,
                                           FAKE, FAKE, ctypes.byref(n), None) == WORKSPACE
    n = ctypes.c_size_t(1 << 30)
    assert L.moe_grouped_swiglu_ffn_gather(FAKE, None, 64, 2, FAKE, FAKE, FAKE, FAKE, 8, 128, 256, 0, 0, 128, 1,
                                           FAKE, FAKE, ctypes.byref(n), None) == INVALID
    assert L.moe_grouped_swiglu_ffn_gather(FAKE, ctypes.c_void_p(0x10002), 64, 2, FAKE, FAKE, FAKE, FAKE, 8, 128,
                                           256, 0, 0, 128, 1, FAKE, FAKE, ctypes.byref(n), None) == INVALID
    assert L.moe_grouped_swiglu_ffn_gather(MISALIGNED, FAKE, 64, 2, FAKE, FAKE, FAKE, FAKE, 8, 128, 256, 0, 0, 128,
                                           1, FAKE, FAKE, ctypes.byref(n), None) == INVALID


def test_combine_validation(L):
    assert L.moe_unpermute_combine(FAKE, FAKE, FAKE, 4, 0, 128, 8, 1, FAKE, None) == INVALID
    assert L.moe_unpermute_combine(FAKE, FAKE, FAKE, 4, 2, 100, 8, 1, FAKE, None) == INVALID
    assert L.moe_unpermute_combine(FAKE, FAKE, FAKE, 4, 2, 128, 8, 1, MISALIGNED, None) == INVALID
    assert L.moe_unpermute_combine(None, None, None, 0, 2, 128, 8, 1, None, None) == 0


def test_sweep_validation(L):
    Ms = np.array([1, 2, 4], np.int32)
    p = Ms.ctypes.data_as(ctypes.c_void_p)
    n = ctypes.c_size_t(0)
    assert L.moe_load_sweep(None, None, None, None, 1, 2048, 768, 0, 0, 1, p, 3, 1, 5, None, None,
                            ctypes.byref(n), None, None, None) == 0
    assert n.value >= 4 * 768 * 2
    bad = np.array([1, 0], np.int32)
    assert L.moe_load_sweep(None, None, None, None, 1, 2048, 768, 0, 0, 1, bad.ctypes.data_as(ctypes.c_void_p),
                            2, 1, 5, None, None, ctypes.byref(n), None, None, None) == INVALID
    assert L.moe_load_sweep(None, None, None, None, 0, 2048, 768, 0, 0, 1, p, 3, 1, 5, None, None,
                            ctypes.byref(n), None, None, None) == INVALID


def test_binding_refuses_cpu_tensors():
    import torch
    x = torch.zeros(4, 128, dtype=torch.bfloat16)
    w = torch.zeros(8, 128, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="GPU"):
        moe.moe_gate_topk(x, w, None, 2)


# ---------------------------------------------------------------- placement path
D8 = ctypes.c_void_p(0x10000)       # 8-byte aligned fake device pointer, never dereferenced


def test_fit_latency_model_matches_oracle_bitwise():
    from oracle import placement_oracle as P
    rng = np.random.default_rng(5)
    for _ in range(20):
        n = int(rng.integers(1, 20))
        loads = rng.choice(np.arange(1, 9000), n, replace=False)
        lat = rng.uniform(1, 1000, n).astype(np.float32)
        kn, kt = moe.moe_fit_latency_model(loads, lat)
        rn, rt = P.fit_latency_model(loads.tolist(), lat.astype(np.float64).tolist())
        assert np.array_equal(kn, rn) and np.array_equal(kt, rt)


@pytest.mark.parametrize("loads,lats", [([1, 1], [1.0, 2.0]), ([0, 2], [1.0, 2.0]), ([1, 2], [1.0, np.nan]),
                                        ([], [])])
def test_fit_latency_model_rejects(L, loads, lats):
    ld = np.asarray(loads, np.int32)
    lt = np.asarray(lats, np.float32)
    out = np.zeros(max(1, len(ld)))
    st = L.moe_fit_latency_model(ld.ctypes.data_as(ctypes.c_void_p), lt.ctypes.data_as(ctypes.c_void_p), len(ld),
                                 out.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p))
    assert st == INVALID


@pytest.mark.parametrize("Lyr,E,G,nk,cap,expect", [
    (4, 0, 8, 4, 0, INVALID),        # E < 1
    (4, 2000, 8, 4, 0, UNSUPPORTED),  # E > 1024
    (4, 64, 65, 4, 0, UNSUPPORTED),   # G > 64
    (4, 64, 8, 65, 0, UNSUPPORTED),   # nk > 64
    (4, 64, 8, 4, 7, INVALID),        # cap * G < E
    (4, 64, 8, 4, -1, INVALID),
    (-1, 64, 8, 4, 0, INVALID),
    (0, 64, 8, 4, 0, 0),              # L = 0: no-op
])
def test_place_greedy_validation(L, Lyr, E, G, nk, cap, expect):
    st = L.moe_place_greedy(D8, Lyr, E, D8, D8, G, nk, cap, FAKE, None, None, None)
    assert st == expect


def test_place_incremental_and_drift_validation(L):
    assert L.moe_place_incremental(D8, 4, 64, D8, D8, 8, 4, -0.1, 10, FAKE, None, None) == INVALID
    assert L.moe_place_incremental(D8, 4, 64, D8, D8, 8, 4, float("nan"), 10, FAKE, None, None) == INVALID
    assert L.moe_place_incremental(D8, 4, 64, D8, D8, 8, 4, 0.03, -1, FAKE, None, None) == INVALID
    assert L.moe_place_incremental(D8, 4, 64, D8, D8, 8, 4, 0.03, 10, None, None, None) == INVALID
    assert L.moe_place_incremental(D8, 0, 64, D8, D8, 8, 4, 0.03, 10, None, None, None) == 0
    assert L.moe_drift_distance(D8, D8, 4, 0, 0.05, D8, None, None) == INVALID
    assert L.moe_drift_distance(D8, D8, 4, 8, float("inf"), D8, None, None) == INVALID
    assert L.moe_drift_distance(MISALIGNED, D8, 4, 8, 0.05, D8, None, None) == INVALID
    assert L.moe_window_push(FAKE, FAKE, D8, 4, 8, 10, 10, None) == INVALID   # slot >= window
    assert L.moe_window_push(FAKE, FAKE, D8, 4, 8, 0, 0, None) == INVALID     # window < 1
    assert L.moe_window_push(None, None, None, 0, 8, 10, 3, None) == 0        # L = 0: no-op


def test_mx_validation_and_query(L):
    """MXFP8 entry points: shapes off the 128 grid are unsupported, missing or
    misaligned operands invalid, the workspace query sized for h codes and
    their scale dwords."""
    n = ctypes.c_size_t(0)
    assert L.moe_grouped_swiglu_ffn_mx(None, None, None, None, None, None, None, None, None, 8, 4096, 14336, 0, 0,
                                       8192, None, None, ctypes.byref(n), None) == 0
    assert n.value >= 8192 * 14336 + (14336 // 128) * 8192 * 4
    for H, I in ((4096, 14300), (4000, 14336)):
        assert L.moe_grouped_swiglu_ffn_mx(None, None, None, None, None, None, None, None, None, 8, H, I, 0, 0, 64,
                                           None, None, ctypes.byref(n), None) == UNSUPPORTED
    assert L.moe_grouped_swiglu_ffn_mx(None, None, None, None, None, None, None, None, None, 300, 128, 128, 0, 0, 64,
                                       None, None, ctypes.byref(n), None) == UNSUPPORTED
    n = ctypes.c_size_t(10)
    assert L.moe_grouped_swiglu_ffn_mx(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 8, 128, 256, 0, 0, 64,
                                       FAKE, FAKE, ctypes.byref(n), None) == WORKSPACE
    # quantiser: K % 128, dtype, null and misaligned pointers
    assert L.moe_mx_quantize(FAKE, 1, 1, 4, 200, 0, None, FAKE, FAKE, None) == UNSUPPORTED
    assert L.moe_mx_quantize(FAKE, 7, 1, 4, 256, 0, None, FAKE, FAKE, None) == INVALID
    assert L.moe_mx_quantize(FAKE, 1, 1, 4, 256, 0, None, None, FAKE, None) == INVALID
    assert L.moe_mx_quantize(MISALIGNED, 1, 1, 4, 256, 0, None, FAKE, FAKE, None) == INVALID
    assert L.moe_mx_quantize(FAKE, 1, 2, 4, 256, 0, FAKE, FAKE, FAKE, None) == INVALID   # row count: batch 1 only
    assert L.moe_mx_quantize(None, 1, 0, 4, 256, 0, None, None, None, None) == 0     # empty: no-op
    # GEMMs
    assert L.moe_grouped_gemm_mx(FAKE, FAKE, FAKE, FAKE, FAKE, 2, 100, 256, 0, 64, FAKE, None) == UNSUPPORTED
    assert L.moe_grouped_gemm_mx(FAKE, FAKE, None, FAKE, FAKE, 2, 128, 256, 0, 64, FAKE, None) == INVALID
    assert L.moe_grouped_gemm_mx(FAKE, FAKE, FAKE, FAKE, FAKE, -1, 128, 256, 0, 64, FAKE, None) == INVALID
    assert L.moe_grouped_swiglu_mx(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 2, 128, 384, 0, 64, FAKE, None,
                                   None) == INVALID
    assert L.moe_grouped_swiglu_mx(None, None, None, None, None, None, None, 0, 128, 384, 0, 64, None, None,
                                   None) == 0


def test_mx_sweep_validation(L):
    Ms = np.array([1, 8], np.int32)
    pM = Ms.ctypes.data_as(ctypes.c_void_p)
    n = ctypes.c_size_t(0)
    args = [FAKE] * 8
    assert L.moe_load_sweep_mx(*args, 1, 4096, 14336, 0, 0, pM, 2, 1, 3, None, None, ctypes.byref(n), None, None,
                               None) == 0
    assert n.value >= 8 * 14336
    assert L.moe_load_sweep_mx(*args, 1, 4096, 14300, 0, 0, pM, 2, 1, 3, None, None, ctypes.byref(n), None, None,
                               None) == UNSUPPORTED
    assert L.moe_load_sweep_mx(*args, 0, 4096, 14336, 0, 0, pM, 2, 1, 3, None, None, ctypes.byref(n), None, None,
                               None) == INVALID
    assert L.moe_load_sweep_mx(*args, 1, 4096, 14336, 0, 0, pM, 2, 1, 0, None, None, ctypes.byref(n), None, None,
                               None) == INVALID
    n = ctypes.c_size_t(16)
    assert L.moe_load_sweep_mx(*args, 1, 4096, 14336, 0, 0, pM, 2, 1, 3, FAKE, FAKE, ctypes.byref(n), FAKE, None,
                               None) == WORKSPACE


def test_mx_weight_row_strides(L):
    """Padded MXFP8 code rows: a multiple of 16 bytes, at least K, checked
    before anything else is looked at."""
    n, m = ctypes.c_size_t(0), ctypes.c_size_t(0)
    nul = [None] * 9
    assert L.moe_grouped_swiglu_ffn_mx(*nul, 8, 4096, 14336, 0, 0, 64, None, None, ctypes.byref(n), None) == 0
    assert L.moe_grouped_swiglu_ffn_mx(*nul, 8, 4096, 14336, 4224, 14464, 64, None, None, ctypes.byref(m),
                                       None) == 0
    assert n.value == m.value
    for gu, dn in ((4100, 0), (4095, 0), (0, 14344), (0, 14335), (1 << 21, 0)):
        assert L.moe_grouped_swiglu_ffn_mx(*nul, 8, 4096, 14336, gu, dn, 64, None, None, ctypes.byref(m),
                                           None) == INVALID, (gu, dn)
    assert L.moe_mx_quantize(None, 1, 0, 4, 256, 384, None, None, None, None) == 0
    for ld in (264, 255, -16):
        assert L.moe_mx_quantize(None, 1, 0, 4, 256, ld, None, None, None, None) == INVALID
    assert L.moe_grouped_gemm_mx(None, None, None, None, None, 0, 128, 256, 272, 64, None, None) == 0
    assert L.moe_grouped_gemm_mx(None, None, None, None, None, 0, 128, 256, 200, 64, None, None) == INVALID
    assert L.moe_grouped_swiglu_mx(None, None, None, None, None, None, None, 0, 128, 384, 136, 64, None, None,
                                   None) == INVALID
    Ms = np.array([1, 8], np.int32)
    assert L.moe_load_sweep_mx(*([FAKE] * 8), 1, 4096, 14336, 4224, 0, Ms.ctypes.data_as(ctypes.c_void_p), 2, 1, 3,
                               None, None, ctypes.byref(n), None, None, None) == 0
    assert L.moe_load_sweep_mx(*([FAKE] * 8), 1, 4096, 14336, 4104, 0, Ms.ctypes.data_as(ctypes.c_void_p), 2, 1, 3,
                               None, None, ctypes.byref(n), None, None, None) == INVALID


def test_ffn_gather_of_checks_the_layer(L):
    """E = 0 (not known) or E_local <= E <= 256; the rest as the gather call's."""
    n = ctypes.c_size_t(0)
    for E in (-1, 7, 257):
        assert L.moe_grouped_swiglu_ffn_gather_of(None, None, 64, 2, None, None, None, None, E, 8, 128, 128, 0, 0, 128,
                                                  1, None, None, ctypes.byref(n), None) == _lib.MOE_ERR_INVALID_ARG
    want = ctypes.c_size_t(0)
    assert L.moe_grouped_swiglu_ffn_gather(None, None, 64, 2, None, None, None, None, 8, 128, 128, 0, 0, 128, 1, None,
                                           None, ctypes.byref(want), None) == _lib.MOE_OK
    for E in (0, 8, 256):
        assert L.moe_grouped_swiglu_ffn_gather_of(None, None, 64, 2, None, None, None, None, E, 8, 128, 128, 0, 0, 128,
                                                  1, None, None, ctypes.byref(n), None) == _lib.MOE_OK
        assert n.value == want.value
