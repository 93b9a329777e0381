"""The octet GEMM kernels (configurations 32 and up: three-way bfloat16 splitting, the
same with A in registers, and FP32 MFMAs in order) against FP64, at tile edges.

Tolerance: a product of two FP32 values formed from their bfloat16 thirds leaves out
terms below 2^-25 of it, and an FP32 sum of K products in tiles errs by at most a few
ulps times sqrt(K) of the summed magnitudes; the repository's GEMM bar of 2e-6
(relative to the result's rms, K <= 300 here) holds that with a wide margin.
"""
import numpy as np
import pytest
import torch

from helpers import assert_close_array, need_gpu, to_dev
pytestmark = pytest.mark.gpu

SPLIT, ROWS, ORDERED = range(32, 40), range(40, 45), range(45, 51)
FIRST_ORDERED = 45


def api():
    need_gpu()
    from paper_2402_02190_amd import api as a
    return a


def key_of(ta, tb, M, N, K):
    return f"{'T' if ta else 'N'}{'T' if tb else 'N'}|{M}x{N}x{K}"


@pytest.mark.parametrize("cfg", [*SPLIT, *ROWS, *ORDERED])
def test_octet_gemm_every_config_layout_and_edge(cfg):
    """Every layout, split counts with empty ranges among them, sizes at and around the
    tiles (off every multiple of 4, multiples of 4, one value), bias, beta and ReLU; the
    ordered configurations give the bits of the first configuration's loop."""
    a = api()
    rng = np.random.default_rng(cfg)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    try:
        for M, N, K in ((333, 130, 77), (128, 132, 76), (1, 1, 1), (65, 33, 33), (31, 64, 288)):
            for ta in (False, True):
                for tb in (False, True):
                    A = rng.standard_normal((K, M) if ta else (M, K)).astype(np.float32)
                    B = rng.standard_normal((N, K) if tb else (K, N)).astype(np.float32)
                    C0 = rng.standard_normal((M, N)).astype(np.float32)
                    bias = rng.standard_normal(N).astype(np.float32)
                    ref = (A.T if ta else A).astype(np.float64) @ (B.T if tb else B).astype(np.float64)
                    ref = np.maximum(ref + 0.5 * C0 + bias, 0.0)
                    for splits in (1, 3, 40):
                        out = []
                        for c in (cfg, 0) if cfg >= FIRST_ORDERED else (cfg,):
                            a.autotune_reset()
                            a.autotune_set(key_of(ta, tb, M, N, K), c, splits)
                            C = to_dev(C0)
                            a.gemm(to_dev(A), to_dev(B), C, ta, tb, beta=0.5, bias=to_dev(bias), relu=True, ws=ws)
                            out.append(C.cpu().numpy())
                        what = f"cfg {cfg} {key_of(ta, tb, M, N, K)} splits {splits}"
                        assert_close_array(out[0], ref, 2e-6, what)
                        if len(out) == 2:
                            assert np.array_equal(out[0], out[1]), what
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("cfg", [32, 35, 37, 40, 41, 44])
def test_split_gemm_is_no_further_from_fp64_than_fp32_mfma(cfg):
    """Over contraction lengths of the layers and of the weight gradients (TN), with
    positive data (the longest sums) and with values over twelve orders of magnitude."""
    a = api()
    rng = np.random.default_rng(cfg)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    try:
        for ta, M, N, K in ((False, 192, 96, 64), (False, 192, 96, 256), (True, 64, 96, 20000)):
            if ta and cfg >= 40:
                continue
            for kind in ("normal", "positive", "wide"):
                A = rng.standard_normal((K, M) if ta else (M, K))
                B = rng.standard_normal((K, N))
                if kind == "positive":
                    A, B = np.abs(A), np.abs(B)
                if kind == "wide":
                    A = A * 10.0 ** rng.uniform(-6, 6, A.shape)
                A, B = A.astype(np.float32), B.astype(np.float32)
                ref = (A.T if ta else A).astype(np.float64) @ B.astype(np.float64)
                err = {}
                for c in (0, cfg):
                    a.autotune_reset()
                    a.autotune_set(key_of(ta, False, M, N, K), c, 8 if ta else 1)
                    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
                    a.gemm(to_dev(A), to_dev(B), C, ta, False, ws=ws)
                    err[c] = np.linalg.norm(C.cpu().numpy() - ref) / np.linalg.norm(ref)
                # below 1e-7 (one rounding of the result is 3e-8) there is nothing to lose
                assert err[cfg] <= max(err[0], 1e-7), (cfg, kind, M, N, K, err)
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("cfg", [32, 39, 40, 44])
def test_split_gemm_infinities_nan_and_overflow(cfg):
    """Infinite, NaN and near-maximal operands give what plain FP32 sums give."""
    a = api()
    rng = np.random.default_rng(cfg)
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    M, N, K = 70, 50, 64
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((K, N)).astype(np.float32)
    A[3, 5], A[4, 6], A[9, 9], A[11, 1] = np.inf, np.nan, -np.inf, 3.4e38
    B[7, 1], B[5, 8] = 1.0, 0.0
    B[1, :] = 1e-3
    B[1, 0] = 8.0
    try:
        for splits in (1, 3):
            out = []
            for c in (0, cfg):
                a.autotune_reset()
                a.autotune_set(key_of(False, False, M, N, K), c, splits)
                C = torch.empty((M, N), dtype=torch.float32, device="cuda")
                a.gemm(to_dev(A), to_dev(B), C, False, False, ws=ws)
                out.append(C.cpu().numpy())
            for f in (np.isnan, np.isposinf, np.isneginf):
                assert np.array_equal(f(out[0]), f(out[1])), f.__name__
            fin = np.isfinite(out[0])
            assert fin.sum() > 0.9 * fin.size and np.isposinf(out[0]).any()
            assert np.allclose(out[0][fin], out[1][fin], rtol=1e-5, atol=1e-5)
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("cfg", [32, 35, 37, 38, 41, 44, 45, 47, 48])
def test_octet_gemm_over_the_graphs_of_a_batch(cfg):
    """By rows and by K over ragged graphs (one empty, one of a single row), widths off
    the multiples of 4, with the bias gradient and split-K."""
    a = api()
    rng = np.random.default_rng(cfg)
    ptr = np.concatenate([[0], np.cumsum([130, 0, 1, 37, 64, 200])]).astype(np.int32)
    n, G = int(ptr[-1]), len(ptr) - 1
    dg = a.DeviceGraph(np.zeros(n + 1, np.int32), np.zeros(0, np.int32), None, ptr)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    try:
        for tb in (False, True):
            for K, N in ((24, 40), (66, 33)):
                a.autotune_reset()
                a.autotune_set(f"{'NT' if tb else 'NN'}|g1:{G}|{n}x{N}x{K}", cfg, 1)
                A = rng.standard_normal((n, K)).astype(np.float32)
                B = rng.standard_normal((G, N, K) if tb else (G, K, N)).astype(np.float32)
                C = torch.full((n, N), np.nan, dtype=torch.float32, device="cuda")
                a.gemm_grouped_rows(dg, to_dev(A), to_dev(B), C, tb)
                ref = np.vstack([A[x:y].astype(np.float64) @ (B[g].T if tb else B[g])
                                 for g, (x, y) in enumerate(zip(ptr[:-1], ptr[1:]))])
                assert_close_array(C.cpu().numpy(), ref, 2e-6, f"cfg {cfg} rows tb={tb} {K}x{N}")
        for M, N in ((40, 24), (33, 65)):
            for splits in (1, 3):
                a.autotune_reset()
                a.autotune_set(f"TN|g2:{G}|{M}x{N + 1}x{n}", cfg, splits)
                A = rng.standard_normal((n, M)).astype(np.float32)
                B = rng.standard_normal((n, N)).astype(np.float32)
                C = torch.full((G, M, N), np.nan, dtype=torch.float32, device="cuda")
                bg = torch.full((G, M), np.nan, dtype=torch.float32, device="cuda")
                a.gemm_grouped_k(dg, to_dev(A), to_dev(B), C, bg, ws=ws)
                for g, (x, y) in enumerate(zip(ptr[:-1], ptr[1:])):
                    what = f"cfg {cfg} K {M}x{N} splits {splits} graph {g}"
                    assert_close_array(C[g].cpu().numpy(), A[x:y].astype(np.float64).T @ B[x:y], 2e-6, what)
                    assert_close_array(bg[g].cpu().numpy(), A[x:y].astype(np.float64).sum(0), 2e-6, what)
    finally:
        a.autotune_reset()


def first_plan_splits(key):
    """Split count of the 64x64x32 tiling: about 512 blocks, at least 4 K steps each."""
    layout, *probs = key.split("|")
    dims = [tuple(int(x) for x in p.split("x")) for p in probs]
    if layout != "TN":
        return 1
    tiles = sum(-(-m // 64) * -(-(n - (n % 2)) // 64) for m, n, _ in dims)
    steps = max(-(-k // 32) for _, _, k in dims)
    if tiles >= 512 or steps < 8:
        return 1
    return max(1, min(-(-512 // tiles), max(1, steps // 4)))


@pytest.mark.parametrize("kind,n,hidden,S,layers", [("sage", 700, 32, 10, 2), ("gcn", 1000, 64, 32, 2),
                                                    ("sage", 5000, 96, 64, 1)])
def test_training_step_keeps_the_ordered_sums(kind, n, hidden, S, layers):
    """An untuned training step gives, bit for bit, what it gives with every product on
    the first configuration (64x64x32, FP32 MFMAs, k in order): logits, loss terms and
    gradients, after one step and after three."""
    from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver
    from workloads import init_params, random_regular_graph
    a = api()
    g = random_regular_graph(n, 5 if n % 2 == 0 else 4, 3)
    lam = np.logspace(-1, 1, S).astype(np.float32)
    p = init_params(kind, n, layers, hidden, S, seed=2)
    sol = CPRASolver(a.DeviceGraph.from_csr(g), CPRAConfig("mis", kind, layers, hidden, S), lam)
    try:
        a.autotune_reset()
        sol.load_params(p)
        keys = [e[0] for e in sol.autotune()]
        out = []
        for first in (False, True):
            a.autotune_reset()
            if first:
                for k in keys:
                    a.autotune_set(k, 0, first_plan_splits(k))
            sol.load_params(p)
            for steps in (1, 2):
                for _ in range(steps):
                    sol.step()
                out.append([t.cpu().numpy() for t in (sol.Z, sol.terms, sol.grads)])
        for x, y in zip(out[:2], out[2:]):
            for u, v in zip(x, y):
                assert np.array_equal(u, v)
    finally:
        a.autotune_reset()
        sol.close()
