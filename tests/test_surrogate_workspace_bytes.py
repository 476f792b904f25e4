"""The network's workspace sizes, through the C ABI without a GPU: what the header states a voxel, for
windows that are no cubes too, growing by equal amounts a window, and refused for empty grids."""
import ctypes

import pytest

from paper_2507_21748_amd import evx, surrogate


def size(nx, ny, nz, train):
    surrogate._lib()
    nb = ctypes.c_size_t()
    st = evx._LIB.evx_surrogate_workspace_bytes(nx, ny, nz, train, ctypes.byref(nb))
    return nb.value if st == 0 else -st


@pytest.mark.parametrize("grid", [(1, 1, 1), (9, 9, 9), (72, 72, 72), (1000, 1, 1), (1, 1, 4000),
                                  (3, 500, 7), (300, 20, 20), (1 << 30, 1, 1)])
def test_bytes_a_voxel(grid):
    voxels = grid[0] * grid[1] * grid[2]
    one = size(*grid, 1)
    # X0, nine 32-channel BF16 fields and two FP32 ones: 2 + 9 * 64 + 8 = 586 bytes a voxel
    assert 586 * voxels <= one <= 610 * voxels + (60 << 20)
    assert size(*grid, -3) == one  # any other value asks for one window
    each = size(*grid, 2) - one
    assert [size(*grid, k) - one for k in (3, 5)] == [2 * each, 4 * each]
    assert 128 * voxels <= size(*grid, 0) <= 140 * voxels + (1 << 20)


def test_refused_grids():
    assert size(0, 4, 4, 1) == size(4, -1, 4, 0) == -2
