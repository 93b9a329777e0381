"""Bit-packed decoding: rounding and scoring without weighted values, and the pairwise
Hamming analysis, against the integer oracle.  Everything is exact."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, to_dev
from oracle import evaluate as oev
from workloads import csr_from_edges, disjoint_union, erdos_renyi_graph, random_regular_graph

pytestmark = pytest.mark.gpu


def api():
    need_gpu()
    from paper_2402_02190_amd import api as a
    return a


def star(n):
    """A hub of degree n - 1 (past every counter's range) as the first node, and as the
    last one of a copy."""
    hub = csr_from_edges(n, np.zeros(n - 1, int), np.arange(1, n))
    last = csr_from_edges(n, np.full(n - 1, n - 1), np.arange(n - 1))
    return disjoint_union([hub, last])


GRAPHS = {
    "one_node": lambda: csr_from_edges(1, np.zeros(0, int), np.zeros(0, int)),
    "regular": lambda: random_regular_graph(258, 20, 3),
    "star": lambda: star(700),
    "batch": lambda: disjoint_union([erdos_renyi_graph(300, 0.03, 1), csr_from_edges(0, [], []),
                                     random_regular_graph(256, 5, 2), csr_from_edges(1, [], []),
                                     erdos_renyi_graph(70, 0.5, 4)]),
}


@pytest.mark.parametrize("S", [1, 10, 16, 17, 63, 64, 65, 130, 132])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_packed_round_eval_is_exact(name, S):
    """Rows, heads and words at their edges, padded leading dimensions, outputs left out,
    and a workspace with room for the row-gathering kernel only: the same counts."""
    a = api()
    g = GRAPHS[name]()
    dg = a.DeviceGraph.from_csr(g)
    G = dg.n_graphs
    rng = np.random.default_rng(S)
    pad = 4 if S % 4 == 0 else 3  # float4 rows of Z where S allows
    Z = rng.standard_normal((g.n, S + pad)).astype(np.float32)
    Z[rng.random(Z.shape) < 0.05] = 0.0
    Z[rng.random(Z.shape) < 0.01] = np.nan
    Z[rng.random(Z.shape) < 0.01] = np.inf
    Zd = to_dev(Z)[:, :S]
    Xo = (Z[:, :S] > 0).astype(np.uint8)
    full = a.round_eval_workspace_bytes(dg, S)
    for problem in ("mis", "maxcut"):
        ev = oev.evaluate(Xo, g, problem)
        pid = a.MIS if problem == "mis" else a.MAXCUT
        for ws_bytes, want_x in ((full, True), (full, False)):
            X = torch.full((g.n, S + pad), 7, dtype=torch.uint8, device="cuda")
            val, vio = (torch.full((G * S,), -1, dtype=torch.int64, device="cuda") for _ in range(2))
            ph = torch.full((G,), -1, dtype=torch.int64, device="cuda")
            ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
            for _ in range(2):  # a second call on a used workspace
                a.round_eval(dg, pid, Zd, X[:, :S] if want_x else None, val, vio, None, ph, ws=ws)
            if want_x:
                assert np.array_equal(X.cpu().numpy()[:, :S], Xo) and (X[:, S:] == 7).all()
            for gi, e in enumerate(ev):
                sl = slice(gi * S, (gi + 1) * S)
                assert int(ph[gi]) == e["pair_hamming"]
                assert np.array_equal(val[sl].cpu().numpy(), e["size" if problem == "mis" else "cut_edges"])
                assert np.array_equal(vio[sl].cpu().numpy(),
                                      e["violations"] if problem == "mis" else np.zeros(S, np.int64))
        # with weighted values wanted, the row-gathering kernel: the same counts
        wv = torch.empty(G * S, dtype=torch.float64, device="cuda")
        val2, vio2 = torch.empty_like(val), torch.empty_like(vio)
        a.round_eval(dg, pid, Zd, None, val2, vio2, wv, None)
        assert torch.equal(val, val2) and torch.equal(vio, vio2)


@pytest.mark.parametrize("N,S", [(1, 1), (63, 16), (64, 17), (65, 3), (4096, 33), (10001, 100), (130, 257), (0, 5)])
def test_pairwise_hamming_at_word_and_tile_edges(N, S):
    """Full and padded matrices, each output alone and together, duplicates among the
    heads, histogram bins from 0 to N."""
    a = api()
    rng = np.random.default_rng(N + S)
    base = rng.random((N, max(1, S // 2))) < 0.4
    X = base[:, rng.integers(0, base.shape[1], S)]
    if S > 2 and N:
        X[:, 1] = ~X[:, 0]  # distance N
    X = X.astype(np.uint8)
    Xd = torch.zeros((max(N, 1), S + 2), dtype=torch.uint8, device="cuda")
    Xd[:N, :S] = to_dev(X, torch.uint8)
    Do = (X[:, :, None] != X[:, None, :]).sum(0) if N * S * S < 5e7 else \
        np.array([[int((X[:, i] != X[:, j]).sum()) for j in range(S)] for i in range(S)])
    Do = Do.astype(np.int64).reshape(S, S)
    up = Do[np.triu_indices(S, 1)]
    ho = np.bincount(up, minlength=N + 1)
    uo = len({X[:, s].tobytes() for s in range(S)})
    for want in ((1, 1, 1), (1, 0, 0), (0, 1, 0), (0, 0, 1)):
        D = torch.full((S, S + 1), -1, dtype=torch.int32, device="cuda") if want[0] else None
        h = torch.full((N + 1,), -5, dtype=torch.int64, device="cuda") if want[1] else None
        u = torch.full((1,), -1, dtype=torch.int32, device="cuda") if want[2] else None
        a.pairwise_hamming(Xd[:N, :S], None if D is None else D[:, :S], h, u)
        if D is not None:
            assert np.array_equal(D[:, :S].cpu().numpy(), Do)
        if h is not None:
            assert np.array_equal(h.cpu().numpy(), ho)
        if u is not None:
            assert int(u) == uo
