"""Names that the rocprofv3 summary gives the halo form's kernels: residual, middle
and last stage apart, whether their accesses are streamed or not."""
import pytest

from paper_2107_14027_amd import rocprof_summary as rs


@pytest.mark.parametrize("stg,short", [(0, "k_lines_halo<3,double>"), (1, "k_lines_halo_stage<3,double>"),
                                       (5, "k_lines_halo_stage<3,double>"), (2, "k_lines_halo_last<3,double>"),
                                       (6, "k_lines_halo_last<3,double>")])
def test_halo_stage_kernels(stg, short):
    name = "void fr::(anonymous namespace)::k_lines<3, double, true, %d>(double const*)" % stg
    assert rs.short(name) == short
