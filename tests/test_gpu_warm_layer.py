"""The warm-start network's fused forward layer and its node features at the edges of
their tiles: rows around a wavefront's 32, degrees around a node's 16 lanes and around
the degree above which lists are searched.

The aggregated activations are FP32 sums in CSR order with one rounding: exact.  A
layer's output is compared with 64 bits on its own bf16 operands; FP32 accumulation of
2 in + 1 terms is off by at most (2 in + 1) 2^-24 sum |terms|, and half as much again is
allowed for the sums inside the matrix unit."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, say
from oracle import warmstart as W
from workloads import (csr_from_edges, disjoint_union, erdos_renyi_graph, init_mpnn_params, random_channels,
                       random_regular_graph)

pytestmark = pytest.mark.gpu


def api():
    need_gpu()
    from paper_2402_02190_amd import api as a
    return a


def ring(n, d):
    """Every node joined to its d nearest (d even): d neighbours, many triangles."""
    u = np.repeat(np.arange(n), d // 2)
    v = (u + np.tile(np.arange(1, d // 2 + 1), n)) % n
    return csr_from_edges(n, u, v)


def clique(n):
    return csr_from_edges(n, *np.triu_indices(n, 1))


@pytest.mark.parametrize("degrees", [[14, 16, 18], [30, 32], [32, 34], [2, 70, 4]])
def test_features_around_the_compared_degrees(degrees):
    from paper_2402_02190_amd.warmstart import WarmStartNet
    a = api()
    parts = [ring(d + 35, d) for d in degrees] + [clique(33), clique(17), clique(3), csr_from_edges(1, [], [])]
    rng = np.random.default_rng(sum(degrees))
    g = disjoint_union([parts[i] for i in rng.permutation(len(parts))])
    say(f"features of rings of {degrees}, n={g.n}")
    rand = random_channels(g.n, 14, seed=3)
    feat, tri = WarmStartNet(1, 16, 64, 32, 14).features(a.DeviceGraph.from_csr(g), rand, triangles=True)
    fo, to = W.node_features(g, rand, 16)
    assert np.array_equal(tri.cpu().numpy()[: g.n], to)
    assert np.array_equal(feat.cpu().numpy().view(np.uint16)[: g.n], W.bf16_bits(fo))


def values(t):
    return W.from_bf16_bits(t.cpu().numpy().view(np.uint16))


@pytest.mark.parametrize("n,graph", [(1, "empty"), (31, "star"), (32, "random"), (33, "star"), (129, "random"),
                                     (385, "random")])
@pytest.mark.parametrize("in_dim,hidden,S,L", [(16, 32, 32, 1), (48, 32, 96, 2), (64, 64, 128, 2), (32, 64, 64, 3)])
def test_layer_on_its_own_operands(n, graph, in_dim, hidden, S, L):
    from paper_2402_02190_amd.warmstart import WarmStartNet
    a = api()
    g = {"empty": lambda: csr_from_edges(n, [], []),
         "star": lambda: csr_from_edges(n, np.zeros(n - 1, int), np.arange(1, n)),
         "random": lambda: erdos_renyi_graph(n, min(1.0, 6.0 / n), n)}[graph]()
    say(f"layer n={n} {graph} {in_dim}->{hidden}->{S} L={L}")
    dg = a.DeviceGraph.from_csr(g)
    net = WarmStartNet(L, in_dim, hidden, S, in_dim - 2)
    p = init_mpnn_params(in_dim, hidden, S, L, seed=n)
    rng = np.random.default_rng(n)
    for ly in p["layers"]:
        ly["b"] = (0.1 * rng.standard_normal(ly["b"].shape)).astype(np.float32)
    net.load_params(p)
    feat = net.features(dg, random_channels(n, in_dim - 2, seed=n))
    ws = net.workspace(dg)
    Z = net.forward(dg, feat, ws)
    saved = lambda k, which: values(a.mpnn_saved(dg, net.cfg, ws, k, which, n))
    for k in range(L):
        H = (values(feat) if k == 0 else saved(k, 0))[:n, : in_dim if k == 0 else hidden]
        A = saved(k, 1)[:n, : H.shape[1]]
        want = np.zeros_like(H, dtype=np.float32)
        for i in range(n):
            lo, hi = g.row_ptr[i], g.row_ptr[i + 1]
            s = np.zeros(H.shape[1], np.float32)
            for j in g.col_idx[lo:hi]:
                s = (s + H[j].astype(np.float32)).astype(np.float32)
            want[i] = s * np.float32(1.0 / (hi - lo)) if hi > lo else 0.0
        assert np.array_equal(W.bf16_bits(A), W.bf16_bits(want)), f"aggregate of layer {k}"
        X = np.concatenate([H, A], 1).astype(np.float64)
        ly = p["layers"][k]
        B = np.concatenate([values_of(ly["Ws"]), values_of(ly["Wn"])], 1)
        exact = X @ B.T + ly["b"]
        bound = 1.5 * (X.shape[1] + 1) * 2.0 ** -24 * (np.abs(X) @ np.abs(B.T) + np.abs(ly["b"]))
        if k == L - 1:
            err = np.abs(Z.cpu().numpy()[:n].astype(np.float64) - exact)
        else:
            got = saved(k + 1, 0)[:n, :hidden]
            exact = np.maximum(exact, 0.0)
            bound = bound + 2.0 ** -8 * np.abs(exact)  # the rounding of the stored activation
            err = np.abs(got - exact)
        assert np.all(err <= bound), f"layer {k}: {np.max(err - bound)}"


def values_of(w):
    return W.from_bf16_bits(W.bf16_bits(w)).astype(np.float64)
