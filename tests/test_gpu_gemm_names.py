"""The kernel that runs is the one that the profiler names: every octet, row and direct
configuration, those that stand in where one cannot run, and operands past 2^31 bytes."""
import numpy as np
import pytest
import torch

from helpers import assert_close_array, need_gpu, say, to_dev
pytestmark = pytest.mark.gpu

SUBSTITUTE_TN = "64x64x32_w2x2_bf3"        # for A in registers, A stored [K, M]
SUBSTITUTE_DIRECT = "32x64x32_w1x2_ord"    # for the direct tiles


def api():
    need_gpu()
    from paper_2402_02190_amd import api as a
    return a


def only_family(a, call):
    a.profile_begin()
    call()
    torch.cuda.synchronize()
    fam = [f for f in a.profile_end() if f.startswith("gemm_") and not f.startswith("gemm_splitk")]
    assert len(fam) == 1, fam
    return fam[0]


@pytest.mark.parametrize("cfg", range(32, 52))
def test_a_forced_configuration_runs_under_its_name(cfg):
    a = api()
    M, N, K = 70, 66, 96
    try:
        for ta, tb in ((False, False), (False, True), (True, False), (True, True)):
            A = torch.randn((K, M) if ta else (M, K), device="cuda")
            B = torch.randn((N, K) if tb else (K, N), device="cuda")
            C = torch.empty((M, N), device="cuda")
            a.autotune_reset()
            a.autotune_set(f"{'T' if ta else 'N'}{'T' if tb else 'N'}|{M}x{N}x{K}", cfg, 1)
            name = a.autotune_table()[0]["choice"].split("/")[0]
            if ta and 40 <= cfg < 45:
                name = SUBSTITUTE_TN
            layout = f"{'t' if ta else 'n'}{'t' if tb else 'n'}"
            assert only_family(a, lambda: a.gemm(A, B, C, ta, tb)) == f"gemm_{layout}_{name}"
    finally:
        a.autotune_reset()


def test_the_direct_tiles_of_grouped_products_and_bias_gradients():
    a = api()
    ptr = np.array([0, 130, 131, 200], np.int32)
    n, G, M, N = 200, 3, 40, 24
    dg = a.DeviceGraph(np.zeros(n + 1, np.int32), np.zeros(0, np.int32), None, ptr)
    A, B, W = (torch.randn(s, device="cuda") for s in ((n, M), (n, N), (G, M, N)))
    C, Cg, bg = (torch.empty(s, device="cuda") for s in ((n, N), (G, M, N), (G, M)))
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    try:
        a.autotune_reset()
        a.autotune_set(f"NN|g1:{G}|{n}x{N}x{M}", 51, 1)
        a.autotune_set(f"TN|g2:{G}|{M}x{N + 1}x{n}", 51, 1)
        assert only_family(a, lambda: a.gemm_grouped_rows(dg, A, W, C, False)) == f"gemm_nn_byrow_{SUBSTITUTE_DIRECT}"
        assert only_family(a, lambda: a.gemm_grouped_k(dg, A, B, Cg, bg, ws=ws)) == f"gemm_tn_byk_{SUBSTITUTE_DIRECT}"
        # and the tuner times a kernel under its own name only
        a.autotune_reset()
        a.autotune_begin()
        a.gemm_grouped_rows(dg, A, W, C, False)
        a.gemm_grouped_k(dg, A, B, Cg, bg, ws=ws)
        for _, choice, _, heuristic_us in a.autotune_end():
            assert "direct" not in choice and heuristic_us > 0, choice
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("cfg,name", [(32, "64x64x32_w2x2_bf3"), (41, "128x64x32_rows_bf3"),
                                      (45, "64x64x32_w2x2_ord"), (51, SUBSTITUTE_DIRECT)])
def test_octet_operands_past_2gib(cfg, name):
    """A and C of 2.15 GB: rows sampled at the ends and between match FP64; and the weight
    gradient over that many rows in 1,024 splits."""
    a = api()
    M, N, K = 8_400_000, 64, 64
    say(f"operands past 2 GiB, cfg {cfg}")
    torch.manual_seed(cfg)
    A, B = torch.randn((M, K), device="cuda"), torch.randn((N, K), device="cuda")
    C = torch.empty((M, N), device="cuda")
    try:
        a.autotune_reset()
        a.autotune_set(f"NT|{M}x{N}x{K}", cfg, 1)
        assert only_family(a, lambda: a.gemm(A, B, C, False, True)) == f"gemm_nt_{name}"
        idx = torch.as_tensor(np.unique(np.concatenate([[0, 1, M - 2, M - 1], np.random.default_rng(cfg).integers(
            0, M, 2000)])), device="cuda")
        ref = A[idx].cpu().numpy().astype(np.float64) @ B.cpu().numpy().astype(np.float64).T
        assert_close_array(C[idx].cpu().numpy(), ref, 2e-6, f"cfg {cfg} sampled rows")
        if cfg in (32, 45):
            D = torch.empty((K, N), device="cuda")
            ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
            a.autotune_set(f"TN|{K}x{N}x{M}", cfg, 1024)
            assert only_family(a, lambda: a.gemm(A, C, D, True, False, ws=ws)) == f"gemm_tn_{name}"
            ref = sum((x.T.contiguous().double() @ y.double() for x, y in zip(A.split(1 << 20), C.split(1 << 20))),
                      torch.zeros((K, N), dtype=torch.float64, device="cuda"))
            # sums of 8,203 products per split: 1.2e-6 at 4,096 for FP32, growing by the root; twice that
            assert_close_array(D.cpu().numpy(), ref.cpu().numpy(), 3.4e-6, f"cfg {cfg} weight gradient")
    finally:
        a.autotune_reset()
        del A, C
        torch.cuda.empty_cache()
