"""Aggregation past the 32-bit row offsets: the 64-bit kernels of every vector width,
several vectors per lane and the shuffled entries of rows that many lanes share.

Values of few mantissa bits make every sum exact but for the factors' roundings, which
are reproduced here, so the results are compared bit for bit."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, say, to_dev
from workloads import csr_from_edges, disjoint_union, random_regular_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [2, 32, 100, 128, 260])
@pytest.mark.parametrize("name", ["sparse", "dense"])
def test_rows_of_2_to_24_bytes_and_more(name, width):
    need_gpu()
    from paper_2402_02190_amd import api
    if name == "sparse":  # degrees around the 8 entries of a chunk, and none
        g = disjoint_union([random_regular_graph(18, d, d) for d in (7, 9)] + [csr_from_edges(2, [], [])])
    else:                 # two vectors per lane
        g = random_regular_graph(28, 17, 1)
    say(f"wide rows {name} width={width} n={g.n}")
    dg = api.DeviceGraph.from_csr(g)
    rng = np.random.default_rng(width)
    Xh = (rng.integers(-2048, 2048, (g.n, width)) / 64).astype(np.float32)
    X = torch.empty((g.n, (1 << 22) + 4), device="cuda")[:, :width]
    X.copy_(to_dev(Xh))
    add, mask = (rng.standard_normal((g.n, width)).astype(np.float32) for _ in range(2))
    deg = np.diff(g.row_ptr)
    inv = np.where(deg > 0, np.float32(1.0) / np.maximum(deg, 1).astype(np.float32), 0).astype(np.float32)
    Y = torch.full((g.n, width), 7.0, device="cuda")
    for transpose in (False, True):
        want = np.zeros((g.n, width), np.float32)
        for i in range(g.n):
            for j in g.col_idx[g.row_ptr[i]:g.row_ptr[i + 1]]:
                term = Xh[j].astype(np.float64) * (np.float64(inv[j]) if transpose else 1.0)
                want[i] = (term + want[i]).astype(np.float32)  # one rounding per entry
        if not transpose:
            want = want * inv[:, None]
        api.aggregate_mean(dg, X, Y, transpose=transpose)
        assert np.array_equal(Y.cpu().numpy(), want), f"transpose={transpose}"
        api.aggregate_mean(dg, X, Y, transpose=transpose, add=to_dev(add), mask=to_dev(mask))
        assert np.array_equal(Y.cpu().numpy(), np.where(mask > 0, want + add, 0)), f"epilogue, transpose={transpose}"
