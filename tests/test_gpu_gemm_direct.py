"""The direct GEMM kernel (configuration 51: one 16x16 tile per wavefront, operands
straight from memory) at the edges of its tiles, of its 4- and 16-value steps of K and of
the 64 in flight.  Its sums run over K in order, so it gives the bits of the ordered
32x32 tiles (configuration 48), which other tests compare with FP64."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, to_dev
from test_gpu_gemm_octets import first_plan_splits, key_of

pytestmark = pytest.mark.gpu

DIRECT, ORDERED = 51, 48


def api():
    need_gpu()
    from paper_2402_02190_amd import api as a
    return a


@pytest.mark.parametrize("pad", [0, 1, 4])
@pytest.mark.parametrize("M,N", [(1, 1), (15, 17), (16, 16), (33, 47), (100, 64)])
def test_direct_gemm_gives_the_ordered_bits(M, N, pad):
    """Every layout, padded rows (float4 loads or not), splits with empty ranges, bias,
    beta and ReLU; NaN and infinity stay in their rows and columns."""
    a = api()
    rng = np.random.default_rng(100 * M + N + pad)
    ws = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")

    def matrix(r, c):
        t = torch.full((r, c + pad), float("nan"), device="cuda")[:, :c]  # padding is never used
        x = rng.standard_normal((r, c)).astype(np.float32)
        x[rng.random((r, c)) < 0.002] = rng.choice([np.inf, -np.inf, np.nan])
        t.copy_(to_dev(x))
        return t

    try:
        for K in (1, 3, 4, 15, 16, 17, 36, 63, 64, 65, 100, 128, 200, 321):
            for ta in (False, True):
                for tb in (False, True):
                    A, B = matrix(*((K, M) if ta else (M, K))), matrix(*((N, K) if tb else (K, N)))
                    C0 = to_dev(rng.standard_normal((M, N)).astype(np.float32))
                    bias = to_dev(rng.standard_normal(N).astype(np.float32))
                    for splits in (1, 3):
                        out = []
                        for c in (DIRECT, ORDERED):
                            a.autotune_reset()
                            a.autotune_set(key_of(ta, tb, M, N, K), c, splits)
                            C = C0.clone()
                            a.gemm(A, B, C, ta, tb, beta=0.5, bias=bias, relu=True, ws=ws)
                            out.append(C.cpu().numpy())
                        assert np.array_equal(out[0], out[1], equal_nan=True), f"{key_of(ta, tb, M, N, K)} {splits}"
    finally:
        a.autotune_reset()


@pytest.mark.parametrize("kind,n,hidden,S,layers", [("gcn", 100, 32, 10, 2), ("gcn", 251, 64, 33, 3),
                                                    ("sage", 60, 16, 8, 2), ("gcn", 3000, 64, 32, 1)])
def test_small_training_step_keeps_the_ordered_sums(kind, n, hidden, S, layers):
    """Products of two pieces, with masks, addends and sigmoid outputs, as an untuned step
    of a small graph runs them: the bits of every product on the first configuration."""
    from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver
    from workloads import init_params, random_regular_graph
    a = api()
    sol = CPRASolver(a.DeviceGraph.from_csr(random_regular_graph(n, 4, 3)), CPRAConfig("mis", kind, layers, hidden, S),
                     np.logspace(-1, 1, S).astype(np.float32))
    p = init_params(kind, n, layers, hidden, S, seed=2)
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
            for _ in range(2):
                sol.step()
            out.append([t.cpu().numpy() for t in (sol.Z, sol.terms, sol.grads, sol.params)])
        for u, v in zip(*out):
            assert np.array_equal(u, v)
    finally:
        a.autotune_reset()
        sol.close()
