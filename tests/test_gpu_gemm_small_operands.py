"""Split GEMM configurations on operands near the ends of FP32's range, and on the
shortest sums, against the FP32 MFMA loop of configuration 0.

Bounds: the relative 2-norm error against FP64 may not pass that of the FP32 sums, or
1e-7 where that is smaller (one rounding of the result is 3e-8).
"""
import numpy as np
import pytest
import torch

from helpers import need_gpu, to_dev
pytestmark = pytest.mark.gpu

CONFIGS = [*range(32, 45)]


def api():
    need_gpu()
    from paper_2402_02190_amd import api as a
    return a


def run(a, cfg, A, B, ta=False, splits=1):
    M, K = (A.shape[1], A.shape[0]) if ta else A.shape
    N = B.shape[1]
    a.autotune_reset()
    a.autotune_set(f"{'T' if ta else 'N'}N|{M}x{N}x{K}", cfg, splits)
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    a.gemm(to_dev(A), to_dev(B), C, ta, False, ws=ws)
    return C.cpu().numpy()


@pytest.mark.parametrize("cfg", CONFIGS)
def test_split_gemm_with_a_near_maximal_value_in_every_sum(cfg):
    """Its bfloat16 part is infinite, so every result is summed again in FP32: the bits of
    the FP32 loop, at tiles' edges, in all layouts, with split-K."""
    a = api()
    rng = np.random.default_rng(cfg)
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    try:
        for M, N, K in ((130, 66, 77), (33, 7, 160)):
            for ta in (False, True):
                for tb in (False, True):
                    A = rng.standard_normal((M, K)).astype(np.float32)
                    A[np.arange(M), rng.integers(0, K, M)] = 3.4e38
                    B = (rng.standard_normal((K, N)) * 1e-3).astype(np.float32)
                    A, B = to_dev(A.T.copy() if ta else A), to_dev(B.T.copy() if tb else B)
                    for splits in (1, 3) if cfg in (32, 40) else (1,):
                        out = []
                        for c in (0, cfg):
                            a.autotune_reset()
                            a.autotune_set(f"{'T' if ta else 'N'}{'T' if tb else 'N'}|{M}x{N}x{K}", c, splits)
                            C = torch.empty((M, N), dtype=torch.float32, device="cuda")
                            a.gemm(A, B, C, ta, tb, ws=ws)
                            out.append(C.cpu().numpy())
                        assert np.isfinite(out[0]).all()
                        if splits == 1:
                            assert np.array_equal(*out), (cfg, M, N, K, ta, tb)
                        else:  # other split ranges
                            assert np.allclose(*out, rtol=1e-5), (cfg, M, N, K, ta, tb)
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("cfg", CONFIGS)
def test_split_gemm_keeps_the_bits_of_small_and_large_operands(cfg):
    """Operands from FP32's subnormals to 1e37, with results in its normal range: bfloat16
    thirds of an operand below 2^-110 would fall under bfloat16's smallest value."""
    a = api()
    rng = np.random.default_rng(cfg)
    try:
        for sa, sb in ((1e-34, 1.0), (1.0, 1e-36), (1e-37, 1e2), (1e3, 1e-39), (1e-40, 1e6), (1e-18, 1e-17),
                       (1e-37, 1e37), (1e30, 1e-30), (1e34, 1e2), (1e18, 1e17)):
            for ta, M, N, K in ((False, 70, 66, 96), (True, 40, 66, 129)):
                A = (rng.standard_normal((K, M) if ta else (M, K)) * sa).astype(np.float32)
                B = (rng.standard_normal((K, N)) * sb).astype(np.float32)
                ref = (A.T if ta else A).astype(np.float64) @ B.astype(np.float64)
                err = [np.linalg.norm((run(a, c, A, B, ta) - ref) / np.linalg.norm(ref)) for c in (0, cfg)]
                assert err[1] <= max(err[0], 1e-7), (cfg, sa, sb, ta, err)
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("cfg", CONFIGS)
def test_split_gemm_of_one_or_two_products_per_sum(cfg):
    """Sums of one and two products, where the terms that the splitting leaves out count
    for more than FP32's rounding: the bits of the FP32 loop.  Tiles' edges, all layouts;
    and graphs of one and two rows among larger ones."""
    a = api()
    rng = np.random.default_rng(cfg)
    try:
        for K in (1, 2):
            for M, N in ((130, 66), (7, 33)):
                for ta in (False, True):
                    for tb in (False, True):
                        A = rng.standard_normal((K, M) if ta else (M, K)).astype(np.float32)
                        B = rng.standard_normal((N, K) if tb else (K, N)).astype(np.float32)
                        out = []
                        for c in (0, cfg):
                            a.autotune_reset()
                            a.autotune_set(f"{'T' if ta else 'N'}{'T' if tb else 'N'}|{M}x{N}x{K}", c, 1)
                            C = torch.empty((M, N), dtype=torch.float32, device="cuda")
                            a.gemm(to_dev(A), to_dev(B), C, ta, tb)
                            out.append(C.cpu().numpy())
                        assert np.array_equal(*out), (cfg, K, M, N, ta, tb)
        ptr = np.array([0, 1, 3, 40, 41], np.int32)
        n, G, M, N = 41, 4, 40, 24
        dg = a.DeviceGraph(np.zeros(n + 1, np.int32), np.zeros(0, np.int32), None, ptr)
        A = rng.standard_normal((n, M)).astype(np.float32)
        B = rng.standard_normal((n, N)).astype(np.float32)
        out = []
        for c in (0, cfg):
            a.autotune_reset()
            a.autotune_set(f"TN|g2:{G}|{M}x{N + 1}x{n}", c, 1)
            C = torch.full((G, M, N), np.nan, dtype=torch.float32, device="cuda")
            bg = torch.full((G, M), np.nan, dtype=torch.float32, device="cuda")
            a.gemm_grouped_k(dg, to_dev(A), to_dev(B), C, bg, ws=torch.empty(1 << 20, dtype=torch.uint8, device="cuda"))
            out.append(C.cpu().numpy())
        for g in (0, 1, 3):
            assert np.array_equal(out[0][g], out[1][g]), (cfg, "graph", g)
    finally:
        a.autotune_reset()
