"""Structural features where nodes of all sizes share a wavefront: a run of large nodes
among small ones, hubs, and the graph sizes around the choice of lanes per node.  Integer
counts and one rounding per feature: exact."""
import numpy as np
import pytest
import torch  # noqa: F401

from helpers import need_gpu, say
from oracle import warmstart as W
from workloads import csr_from_edges, random_channels

pytestmark = pytest.mark.gpu


def ring_edges(first, n, d):
    """n nodes from `first` on, each joined to its d nearest (d even)."""
    u = np.repeat(np.arange(n), d // 2)
    return first + u, first + (u + np.tile(np.arange(1, d // 2 + 1), n)) % n


@pytest.mark.parametrize("n", [4095, 4096, 8191, 8192, 8195])
@pytest.mark.parametrize("large", [(34, 48, 50), (100,), (16, 32)])
def test_features_of_large_nodes_among_small_ones(n, large):
    """Rings of the large degrees side by side at the graph's start and at its end, a
    sparse ring between them, and two hubs joined to every 50th node."""
    need_gpu()
    from paper_2402_02190_amd import api
    from paper_2402_02190_amd.warmstart import WarmStartNet
    edges, at = [], 0
    for d in large:
        edges.append(ring_edges(at, d + 40, d))
        at += d + 40
    tail = ring_edges(n - 160, 160, large[-1])
    edges += [ring_edges(at, n - 160 - at, 4), tail]
    for hub in (at + 7, n - 9):
        t = np.arange(0, n, 50)
        edges.append((np.full(t.size, hub), t))
    u, v = np.concatenate([e[0] for e in edges]), np.concatenate([e[1] for e in edges])
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    pair = np.unique(lo[lo != hi] * np.int64(n) + hi[lo != hi])
    g = csr_from_edges(n, pair // n, pair % n)
    say(f"features, n={n}, nnz={g.col_idx.size}, degrees {large}")
    rand = random_channels(n, 14, seed=3)
    feat, tri = WarmStartNet(1, 16, 64, 32, 14).features(api.DeviceGraph.from_csr(g), rand, triangles=True)
    fo, to = W.node_features(g, rand, 16)
    assert np.array_equal(tri.cpu().numpy()[:n], to)
    assert np.array_equal(feat.cpu().numpy().view(np.uint16)[:n], W.bf16_bits(fo))
