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
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(np.float32)


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


@pytest.mark.parametrize("n,degree,width", [(8200, 3, 256), (24_600, 5, 128), (65_600, 13, 64)])
def test_column_slices_are_exact(n, degree, width):
    """Tables past the sizes from which the columns are dealt to the XCDs in slices: rows
    that no block of a slice may miss or do twice, every epilogue operand.  The sums are
    taken here over all rows at once, one entry of every row after the other."""
    need_gpu()
    from paper_2402_02190_amd import api
    g = random_regular_graph(n, degree, 1)
    say(f"column slices n={n} degree={degree} width={width}")
    dg = api.DeviceGraph.from_csr(g)
    rng = np.random.default_rng(n)
    Xh = (rng.integers(-2048, 2048, (n, width)) / 64).astype(np.float32)
    add, mask = (rng.standard_normal((n, width)).astype(np.float32) for _ in range(2))
    bias = rng.standard_normal(width).astype(np.float32)
    X, Y = to_dev(Xh), torch.full((n, width + 32), 7.0, device="cuda")
    inv = np.float32(1.0) / np.float32(degree)
    cols = g.col_idx.reshape(n, degree)
    total, scaled = np.zeros((n, width), np.float32), np.zeros((n, width), np.float32)
    for e in range(degree):
        total = total + Xh[cols[:, e]]
        scaled = fma32(np.float32(inv), Xh[cols[:, e]], scaled)
    api.aggregate_mean(dg, X, Y[:, :width], add=to_dev(add), bias=to_dev(bias), relu=True)
    assert np.array_equal(Y[:, :width].cpu().numpy(), np.maximum(total * inv + add + bias, 0))
    api.aggregate_mean(dg, X, Y[:, :width], transpose=True, add=to_dev(add), mask=to_dev(mask))
    assert np.array_equal(Y[:, :width].cpu().numpy(), np.where(mask > 0, scaled + add, 0))
    assert torch.all(Y[:, width:] == 7.0)
