"""Which tuned plans a training step takes: its own and those that the caller inserts,
not those that the tuning of a forward or of a plain product left for the same shape."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, say
pytestmark = pytest.mark.gpu


def setup():
    need_gpu()
    from paper_2402_02190_amd import api
    from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver
    from workloads import init_params, random_regular_graph
    n, hidden, S = 30000, 128, 64
    sol = CPRASolver(api.DeviceGraph.from_csr(random_regular_graph(n, 5, 3)), CPRAConfig("mis", "gcn", 1, hidden, S),
                     np.logspace(-1, 1, S).astype(np.float32))
    return api, sol, init_params("gcn", n, 1, hidden, S, seed=2)


def after_a_step(sol, p):
    sol.load_params(p)
    sol.step()
    return [t.cpu().numpy() for t in (sol.Z, sol.terms, sol.grads, sol.params)]


def families(api, call):
    api.profile_begin()
    call()
    torch.cuda.synchronize()
    return api.profile_end()


def test_plans_tuned_by_other_calls_leave_a_step_alone():
    api, sol, p = setup()
    try:
        api.autotune_reset()
        first = after_a_step(sol, p)
        api.autotune_begin()
        sol.forward()
        table = api.autotune_end()
        say("  tuned by a forward:", [(k, c) for k, c, _, _ in table])
        assert table  # (a split plan, the faster kind by far at this shape)
        fam = families(api, sol.step)
        assert not any("_bf3" in f for f in fam), sorted(fam)
        for x, y in zip(first, after_a_step(sol, p)):
            assert np.array_equal(x, y)
        # a step's own tuning replaces the entry, and both calls take it then
        sol.autotune()
        tuned = {e["key"]: e["choice"] for e in api.autotune_table()}
        name = "gemm_nt_" + tuned[table[0][0]].split("/")[0]
        assert name in families(api, sol.step) and name in families(api, sol.forward)
    finally:
        api.autotune_reset()
        sol.close()


@pytest.mark.parametrize("cfg,name", [(32, "gemm_nt_64x64x32_w2x2_bf3"), (45, "gemm_nt_64x64x32_w2x2_ord")])
def test_an_inserted_plan_holds_for_a_step(cfg, name):
    api, sol, p = setup()
    try:
        api.autotune_reset()
        sol.load_params(p)
        sol.autotune()
        keys = [e["key"] for e in api.autotune_table() if e["key"].startswith("NT")]
        api.autotune_reset()
        for k in keys:
            api.autotune_set(k, cfg, 1)
        assert name in families(api, sol.step)
    finally:
        api.autotune_reset()
        sol.close()


def test_a_saved_entry_of_two_products_holds_for_the_one_they_became():
    """Earlier tables name the two products of a linear-first layer (H Ws^T and H Wn^T)
    side by side; their entry is found by the product of both."""
    need_gpu()
    from paper_2402_02190_amd import api
    from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver
    from workloads import random_regular_graph
    n, hidden, S = 3000, 64, 16
    sol = CPRASolver(api.DeviceGraph.from_csr(random_regular_graph(n, 4, 3)), CPRAConfig("mis", "gcn", 1, hidden, S),
                     np.logspace(-1, 1, S).astype(np.float32))
    one, two = f"NT|{n}x{2 * S}x{hidden}", f"NT|{n}x{S}x{hidden}|{n}x{S}x{hidden}"
    try:
        for entries, family in (({two: 3}, "gemm_nt_128x64x32_w2x2"), ({two: 3, one: 10}, "gemm_nt_64x64x16_w2x2_p2")):
            api.autotune_reset()
            for k, cfg in entries.items():
                api.autotune_set(k, cfg, 1)
            for call in (sol.forward, sol.step):
                fam = families(api, call)
                assert family in fam, (entries, sorted(fam))
    finally:
        api.autotune_reset()
        sol.close()


def test_a_forward_gives_a_steps_logits():
    """To FP32 rounding by themselves; to the bit when a table names every product, and
    with a frozen prefix."""
    api, sol, p = setup()
    try:
        api.autotune_reset()
        sol.load_params(p)
        sol.autotune()
        keys = [e["key"] for e in api.autotune_table()]
        for table in (False, True):
            api.autotune_reset()
            if table:
                for k in keys:
                    api.autotune_set(k, 32, 1)
            sol.load_params(p)
            sol.step()
            Z = sol.Z.clone()
            sol.load_params(p)
            sol.forward()
            rel = float((sol.Z - Z).double().norm() / Z.double().norm())
            assert rel <= 1e-6, rel
            assert not table or torch.equal(sol.Z, Z)
    finally:
        api.autotune_reset()
        sol.close()
    from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver
    from workloads import init_params, random_regular_graph
    n, S = 30000, 64
    frozen = CPRASolver(api.DeviceGraph.from_csr(random_regular_graph(n, 5, 3)),
                        CPRAConfig("mis", "gcn", 2, 128, S, train_from_layer=1),
                        np.logspace(-1, 1, S).astype(np.float32))
    try:
        frozen.load_params(init_params("gcn", n, 2, 128, S, seed=2))
        frozen.forward()
        Z = frozen.Z.clone()
        frozen.step()
        assert torch.equal(frozen.Z, Z)
    finally:
        frozen.close()
