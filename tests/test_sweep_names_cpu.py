"""The size sweep's summary finds its two kernels in a trace under their present names."""
import pytest

from paper_2402_02190_amd.profile_summary import _sweep_kernel

NS = "void cpra::(anonymous namespace)::"


@pytest.mark.parametrize("name,family", [
    (NS + "k_loss<1, 4, false>(cpra::(anonymous namespace)::LossArgs)", "loss_fwd_bwd"),
    (NS + "k_aggregate<4, 1, false, true, 2>(cpra::(anonymous namespace)::AggArgs)", "aggregate"),
    (NS + "k_aggregate<4, 2, false, false, 8>(cpra::(anonymous namespace)::AggArgs)", "aggregate"),
    (NS + "k_aggregate<4, 1, true, true, 2>(cpra::(anonymous namespace)::AggArgs)", None),
    (NS + "k_sigmoid(long, float const*, float*)", None),
])
def test_sweep_kernel_names(name, family):
    assert _sweep_kernel(name) == family
