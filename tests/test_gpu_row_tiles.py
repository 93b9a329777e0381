"""The row-tile maps of grouped products: graphs of sizes around the tile heights, empty
ones among them, and graph counts around the threads of the scan and past the counts
that one launch takes.  Small whole numbers: exact."""
import numpy as np
import pytest
import torch

from helpers import need_gpu, to_dev
from workloads import csr_from_edges, disjoint_union

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [45, 46, 48])  # tiles of 64, 128 and 32 rows
@pytest.mark.parametrize("graphs", [2, 63, 255, 256, 257, 700, 4096, 4097])
def test_every_row_meets_its_graphs_weights(graphs, cfg):
    need_gpu()
    from paper_2402_02190_amd import api
    rng = np.random.default_rng(graphs)
    sizes = rng.choice([0, 1, 2, 31, 32, 33, 64, 65, 128, 129], graphs) if graphs <= 700 else rng.integers(0, 40, graphs)
    sizes[-1] = 0 if graphs % 2 else 130
    g = disjoint_union([csr_from_edges(int(s), [], []) for s in sizes])
    dg = api.DeviceGraph.from_csr(g)
    n = int(sizes.sum())
    A = rng.integers(-8, 9, (n, 4)).astype(np.float32)
    B = rng.integers(-8, 9, (graphs, 4, 8)).astype(np.float32)
    C = torch.full((n, 8), 7.0, device="cuda")
    try:
        api.autotune_reset()
        api.autotune_set(f"NN|g1:{graphs}|{n}x8x4", cfg, 1)
        api.gemm_grouped_rows(dg, to_dev(A), to_dev(B), C)
    finally:
        api.autotune_reset()
    want = np.einsum("nk,nkj->nj", A, np.repeat(B, sizes, axis=0))
    assert np.array_equal(C.cpu().numpy(), want)
