"""The rules by which projection and attention calls choose their kernels (host code)."""
import pytest

from plans import gemm_plan


@pytest.mark.parametrize("m,n,k", [(2049, 512, 4096), (4096, 512, 4096), (2304, 3584, 18944), (3072, 1024, 8192), (5000, 1024, 4096)])
def test_k_is_sliced_at_thousands_of_rows_where_few_columns_leave_the_chip_idle(m, n, k):
    """In one slice the launch has fewer workgroups than the chip has compute units, or a last round that is nearly empty:
    1.15 to 1.6 times the time of the sliced launch."""
    p = gemm_plan(m, n, k)
    assert p.split_k > 1, (p.tile, p.split_k)


@pytest.mark.parametrize("m,n,k", [(6144, 24576, 4096), (12288, 37888, 3584), (4096, 12288, 4096)])
def test_k_is_not_sliced_where_the_tiles_fill_the_chip(m, n, k):
    assert gemm_plan(m, n, k).split_k == 1
