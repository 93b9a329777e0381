"""The peak that bench.py sets a GEMM family's rate against is that of the pipe it uses."""
import pytest

import bench


@pytest.mark.parametrize("family,peak", [("gemm_nn_64x64x32_w2x2_bf3", 2500.0 / 6),
                                         ("gemm_tn_byk_128x64x32_rows_bf3", 2500.0 / 6),
                                         ("gemm_nt_64x64x32_w2x2_ord", 157.3),
                                         ("gemm_tn_64x64x16_w2x2_ring", 157.3)])
def test_peak_of_a_gemm_family(family, peak):
    r = bench.roofline_entry(family, (10, 1.0, 2e11, 0.0, 0.0), "C4")  # 10 launches of 0.1 ms, 20 GFLOP each
    assert r["bound"] == "mfma" and r["peak"] == pytest.approx(peak)
    assert r["achieved"] == pytest.approx(200.0) and r["frac"] == pytest.approx(200.0 / peak)
