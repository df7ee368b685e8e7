"""Resource use of the built direct-load kernels (CPU: reads the code objects
in libbssn_hip.so).  They are the only route of periodic grids with an odd number
of points in x or in mixed precision, and of rows that are not 16-byte
aligned.
"""
import pytest

from test_kernel_resources import _kernels, _select


@pytest.fixture(scope="module")
def kernels():
    return _kernels()


def test_order4_constraints_fit_two_waves_per_simd(kernels):
    for k, v in _select(kernels, r"13k_constraintsILi4E").items():
        # vgpr_count counts the accumulation registers too
        assert v["vgpr_count"] <= 256, k
        assert not v["private_segment_fixed_size"], k


def test_order8_periodic_fp32_stage_spills_little(kernels):
    # one thread per point does not fit 512 registers here: at most 8 of them
    # in scratch
    (v,) = _select(kernels, r"7k_stageILi8ELb1ELi1E").values()
    assert v["private_segment_fixed_size"] <= 32
