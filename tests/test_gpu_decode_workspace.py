"""Rounding and scoring in a workspace with room for the row-gathering kernel only, as
earlier workspace queries gave it: the counts of the bit-packed path."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, to_dev
from oracle import evaluate as oev
from workloads import disjoint_union, erdos_renyi_graph, random_regular_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 3, 10, 16])
@pytest.mark.parametrize("problem", ["mis", "maxcut"])
def test_round_eval_without_room_for_the_packed_words(problem, S):
    need_gpu()
    from paper_2402_02190_amd import api
    g = disjoint_union([random_regular_graph(3000, 20, 3), erdos_renyi_graph(1200, 0.01, 1)])
    dg = api.DeviceGraph.from_csr(g)
    rng = np.random.default_rng(S)
    Z = rng.standard_normal((g.n, S)).astype(np.float32)
    Zd, Xo = to_dev(Z), (Z > 0).astype(np.uint8)
    pid = api.MIS if problem == "mis" else api.MAXCUT
    n_out = dg.n_graphs * S

    def run(nbytes):
        X = torch.full((g.n, S), 7, dtype=torch.uint8, device="cuda")
        val, vio = (torch.full((n_out,), -1, dtype=torch.int64, device="cuda") for _ in range(2))
        ph = torch.full((dg.n_graphs,), -1, dtype=torch.int64, device="cuda")
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        api.round_eval(dg, pid, Zd, X, val, vio, None, ph, ws=ws)
        return [t.cpu().numpy() for t in (X, val, vio, ph)]

    full = api.round_eval_workspace_bytes(dg, S)
    low, high = 0, full  # the smallest accepted size: refusals are made on the host
    while high - low > 256:
        mid = (low + high) // 512 * 256
        try:
            run(mid)
            high = mid
        except api.CpraError:
            low = mid
    words = g.n * 8
    assert high < words < full  # no room for the packed words
    packed, gathered = run(full), run(high)
    for a, b in zip(packed, gathered):
        assert np.array_equal(a, b)
    assert np.array_equal(gathered[0], Xo)
    for gi, e in enumerate(oev.evaluate(Xo, g, problem)):
        sl = slice(gi * S, (gi + 1) * S)
        assert np.array_equal(gathered[1][sl], e["size" if problem == "mis" else "cut_edges"])
        assert int(gathered[3][gi]) == e["pair_hamming"]
