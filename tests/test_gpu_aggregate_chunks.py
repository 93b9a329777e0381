"""Aggregation at the edges of its chunks of entries and of its 32-bit addresses.

A row's sum runs in CSR order in float32, one add per entry (a fused multiply-add with
the entry's factor when transposed): both are reproduced exactly here, so the results
are compared bit for bit."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, say, to_dev
from workloads import csr_from_edges, disjoint_union, erdos_renyi_graph, random_regular_graph

pytestmark = pytest.mark.gpu


def graph(name):
    if name == "sparse":   # degrees around the 8 entries of a chunk, isolated nodes
        return disjoint_union([random_regular_graph(40, d, d) for d in (2, 7, 8, 9, 16, 17)]
                              + [csr_from_edges(3, [], []), erdos_renyi_graph(61, 0.1, 3)])
    if name == "dense":    # two vectors per lane
        return disjoint_union([random_regular_graph(60, d, d) for d in (11, 16, 25)] + [csr_from_edges(2, [], [])])
    n = 700                # a hub
    return csr_from_edges(n, np.zeros(n - 1, int), np.arange(1, n))


def fma32(a, b, c):
    """float32 fma: the product of two float32 is exact in float64, whose rounded sum
    rounds again only on a tie of the 24th bit, which these inputs do not reach."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


@pytest.mark.parametrize("ld", ["tight", "padded", "wide"])
@pytest.mark.parametrize("width", [1, 3, 6, 27, 32, 64, 100, 260])
@pytest.mark.parametrize("name", ["sparse", "dense", "hub"])
def test_chunked_sums_are_exact(name, width, ld):
    need_gpu()
    from paper_2402_02190_amd import api
    g = graph(name)
    if ld == "wide" and (width > 6 or name != "sparse"):
        pytest.skip("one stride of 2^24 bytes is enough")
    say(f"aggregate {name} width={width} ld={ld}")
    # "wide": a row stride past the 24-bit factors, so 64-bit addresses (a few rows only)
    if ld == "wide":
        g = random_regular_graph(12, 9, 1)
    dg = api.DeviceGraph.from_csr(g)
    stride = {"tight": width, "padded": width + 4, "wide": (1 << 22) + 4}[ld]
    rng = np.random.default_rng(width)
    # few mantissa bits: every partial sum is exact, up to the factors' roundings
    Xh = (rng.integers(-2048, 2048, (g.n, width)) / 64).astype(np.float32)
    X = torch.empty((g.n, stride), device="cuda")[:, :width]
    X.copy_(to_dev(Xh))
    Y = torch.full((g.n, width), 7.0, device="cuda")
    deg = np.diff(g.row_ptr)
    inv = np.where(deg > 0, np.float32(1.0) / np.maximum(deg, 1).astype(np.float32), 0).astype(np.float32)
    add = rng.standard_normal((g.n, width)).astype(np.float32)
    for transpose in (False, True):
        want = np.zeros((g.n, width), np.float32)
        for i in range(g.n):
            for j in g.col_idx[g.row_ptr[i]:g.row_ptr[i + 1]]:
                want[i] = fma32(np.full(width, inv[j]), Xh[j], want[i]) if transpose else want[i] + Xh[j]
        if not transpose:
            want = want * inv[:, None]
        api.aggregate_mean(dg, X, Y, transpose=transpose)
        assert np.array_equal(Y.cpu().numpy(), want), f"transpose={transpose}"
        api.aggregate_mean(dg, X, Y, transpose=transpose, add=to_dev(add), relu=True)
        assert np.array_equal(Y.cpu().numpy(), np.maximum(want + add, 0)), f"addend, transpose={transpose}"
