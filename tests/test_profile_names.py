"""The benchmark's profile summary tells the stepper's passes by their kernels' names."""
import pytest

import bench


@pytest.mark.parametrize("name,expect", [
    ("void evx::col_kernel<1024, 0, 0, 8>(evx::ColArgs)", "y_forward"),
    ("void evx::col_kernel<1024, 0, 1, 8>(evx::ColArgs)", "y_inverse"),
    ("void evx::col_kernel<1024, 0, 3, 8>(evx::ColArgs)", "z_fused_update"),
    ("void evx::col_kernel<1024, 0, 2, 8>(evx::ColArgs)", None),
    ("void evx::row_kernel<512, 0, 0, false>(evx::RowArgs)", "x_fused_fprime"),
    ("void evx::row_kernel<512, 0, 1, false>(evx::RowArgs)", None),
    ("void evx::row_kernel_batch<512, 0, 0>(evx::RowArgs, evx::PassBatch)", None)])
def test_pass_of_kernel(name, expect):
    assert bench._pass_of_kernel(name) == expect
