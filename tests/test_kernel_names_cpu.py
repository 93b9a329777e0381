"""The profiler's families of the octet, row and direct GEMM kernels and of the
aggregation against the names that rocprofv3 prints for their instantiations."""
import os

import pytest

from paper_2402_02190_amd import traffic as TR


@pytest.mark.parametrize("family,name,other", [
    ("gemm_nt_64x64x32_w2x2_bf3", "k_gemm_oct<64, 64, 32, 2, 2, false, true, true, true, 0>(a)",
     "k_gemm_oct<64, 64, 32, 2, 2, false, true, true, false, 0>(a)"),
    ("gemm_tn_byk_32x64x32_w1x2_ord", "k_gemm_oct<32, 64, 32, 1, 2, true, false, true, false, 2>(a)",
     "k_gemm_oct<32, 64, 32, 1, 2, true, false, true, false, 0>(a)"),
    ("gemm_nn_byrow_128x64x32_rows_bf3", "k_gemm_rows<64, 4, false, false, 1>(a)", "k_gemm_rows<64, 4, true, false, 1>(a)"),
    ("gemm_tn_16x16x32_direct_ord", "k_gemm_direct<true, false, true>(a)", "k_gemm_direct<false, false, true>(a)"),
    ("aggregate", "k_aggregate<4, 2, false, true, 2>(a)", "k_aggregate<4, 2, true, true, 2>(a)"),
    ("aggregate_transposed", "k_aggregate<4, 1, true, true, 8>(a)", "k_aggregate<4, 1, false, true, 8>(a)"),
])
def test_family_matches_its_kernel_only(family, name, other):
    assert TR.kernel_pattern(family).search(name)
    assert not TR.kernel_pattern(family).search(other)
    assert all(os.path.exists(p) for p in TR.source_files(family))
