"""The spectral state's order in memory, which a caller may keep in a file and resume from."""
import numpy as np
import pytest
import torch

from paper_2507_21748_amd import evx
from paper_2507_21748_amd.inputs import quench_field

pytestmark = pytest.mark.gpu


# columns per tile: those of a 256-lane workgroup of the z transform (one lane each at length 16)
@pytest.mark.parametrize("nz,cols", [(16, 256), (32, 64), (100, 32), (128, 16), (256, 16)])
def test_state_is_tile_major(nz, cols):
    evx.load()
    ny, nx = 20, 32
    plan = evx.Plan((nz, ny, nx), "periodic", "spectral")
    c = quench_field((nz, ny, nx), 0.1, 0.05, seed=11)
    plan.begin(torch.from_numpy(c).cuda())
    s = torch.view_as_complex(plan.state().view(torch.float32).reshape(-1, 2)).cpu().numpy()
    ref = np.fft.rfftn(c.astype(np.float64))
    groups = (nx // 2 + 1 + 7) // 8
    nseq = groups * ny * 8
    assert s.size == -(-nseq // cols) * cols * nz
    seq = np.arange(nseq)
    x, y = seq // (8 * ny) * 8 + seq % 8, seq // 8 % ny
    live = x <= nx // 2
    seq, x, y = seq[live], x[live], y[live]
    k = np.arange(nz)[:, None]
    got = s[(seq // cols * nz + k) * cols + seq % cols]
    # FP32 transforms of three axes: a few eps per stage, relative to the largest coefficient
    assert np.abs(got - ref[:, y, x]).max() <= 1e-5 * np.abs(ref).max()
