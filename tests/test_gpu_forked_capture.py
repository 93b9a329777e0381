"""Captured training steps that fork their weight gradients to the second stream (two
trained layers and 2^20 values per layer input and more), against the same steps on one
stream: the same kernels on the same data, so the same bits after every replay, with
eager work and synchronisations between the replays."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, say
from workloads import (disjoint_union, erdos_renyi_graph, init_params, init_params_per_graph,
                       random_regular_graph)

pytestmark = pytest.mark.gpu

N = 16400  # x 64 columns: just past 2^20 values


def batch(n_graphs):
    sizes = np.full(n_graphs, N // n_graphs)
    sizes[0] += N - sizes.sum()
    return disjoint_union([erdos_renyi_graph(int(m), 5.0 / m, i) for i, m in enumerate(sizes)])


CASES = {
    # square layers: backward gathers into alternating buffers while the previous layer's
    # weight gradients still read theirs
    "square6": (lambda: random_regular_graph(N, 4, 1), dict(layer_kind="gcn", n_layers=6, hidden=64, S=64)),
    # a widening first layer (its input gradient before the gather) below square ones
    "widening5": (lambda: random_regular_graph(N, 5, 2),
                  dict(layer_kind="sage", n_layers=5, hidden=64, S=32, in_dim=16)),
    "widening_recomputed": (lambda: random_regular_graph(N, 5, 2),
                            dict(layer_kind="sage", n_layers=4, hidden=64, S=100, in_dim=16, recompute=True)),
    "frozen_first": (lambda: random_regular_graph(N, 4, 3),
                     dict(layer_kind="sage", n_layers=4, hidden=64, S=32, train_from_layer=1)),
    "per_graph": (lambda: batch(7), dict(layer_kind="sage", n_layers=3, hidden=64, S=16, per_graph_weights=True)),
}


def run(dg, p, kw, lam, early, env, monkeypatch):
    from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver
    for k in ("CPRA_SIDE_FIRST", "CPRA_OVERLAP", "CPRA_WGRAD_LATE"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    problem = "mis" if lam is not None else "maxcut"
    sol = CPRASolver(dg, CPRAConfig(problem=problem, T=20, **kw), lam)
    seen = []
    try:
        sol.load_params(p)
        if early:  # fires by itself: every step counts as stalled
            sol.enable_early_stopping(1e30, 3)
        sol.capture()
        scratch = torch.ones(1 << 20, device="cuda")
        for _ in range(6):
            sol.replay(1)
            scratch.mul_(1.0001)
            torch.cuda.synchronize()
            seen.append([x.clone() for x in (sol.params, sol.m, sol.v, sol.Z, sol.dZ, sol.grads, sol.terms,
                                             sol.step_counter)])
        state = sol.early_stop_state() if early else None
    finally:
        sol.close()
    return seen, state


@pytest.mark.parametrize("early", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_forked_replays_equal_one_stream(name, early, monkeypatch):
    need_gpu()
    from paper_2402_02190_amd import api
    gfn, kw = CASES[name]
    g = gfn()
    widths = [kw.get("in_dim", kw["hidden"])] + [kw["hidden"]] * (kw["n_layers"] - 1)
    assert g.n * max(widths[kw.get("train_from_layer", 0):]) >= 1 << 20
    dg = api.DeviceGraph.from_csr(g)
    lam = np.logspace(-1, 1, kw["S"]).astype(np.float32) if g.n_graphs == 1 else None
    make = dict(seed=5, in_dim=kw.get("in_dim"))
    p = (init_params_per_graph(kw["layer_kind"], g.n, kw["n_layers"], kw["hidden"], kw["S"], g.n_graphs, **make)
         if kw.get("per_graph_weights") else
         init_params(kw["layer_kind"], g.n, kw["n_layers"], kw["hidden"], kw["S"], **make))
    want, stop = run(dg, p, kw, lam, early, {"CPRA_OVERLAP": "0"}, monkeypatch)
    assert not early or stop["stopped"]
    for env in ({}, {"CPRA_SIDE_FIRST": "1"}):
        say(f"forked replays of {name}, early stopping {early}, {env or 'main first'}")
        got, state = run(dg, p, kw, lam, early, env, monkeypatch)
        assert state == stop
        for step, (a, b) in enumerate(zip(want, got)):
            for what, x, y in zip(("params", "m", "v", "Z", "dZ", "grads", "terms", "counter"), a, b):
                assert torch.equal(x, y), (name, env, f"replay {step}", what)
