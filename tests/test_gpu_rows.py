"""The x pass at every shape of its lane map, against the FP64 oracle: lane counts that are no
multiple of 8 columns (lengths 50, 100 and 400 have 5, 5 and 20 lanes a row, 40, 96 and 200 have 2,
8 and 10), one lane a row (lengths up to 20), rows that do not fill the last workgroup, group tails
of 1 to 7 dead columns, and the real-row passes through begin and end.  Relative L2 1e-5 after one
step and 2e-5 after three (a step's forward and inverse transforms round at a few FP32 ulps, 6e-8,
with the logarithm of the length)."""
import os

import numpy as np
import pytest

from oracle import ch
from oracle.ch import CHParams as OParams
from paper_2507_21748_amd.inputs import quench_field
from tests.test_gpu_ch import gpu_run, rel_l2

pytestmark = pytest.mark.gpu

ch.WORKERS = min(16, os.cpu_count() or 1)

X_LENGTHS = [8, 12, 20, 24, 40, 48, 80, 96, 100, 192, 200, 320, 400]
MIXED = ("zero_flux", "periodic", "zero_flux")  # one complex column per cosine bin


@pytest.mark.parametrize("nx", X_LENGTHS)
@pytest.mark.parametrize("bc", ["periodic", "zero_flux", MIXED], ids=["periodic", "cosine", "mixed"])
def test_row_lengths(evx_gpu, nx, bc):
    shape = (6, 10, nx)  # 60 rows: no multiple of any workgroup's rows
    print(f"row pass {shape} {bc}", flush=True)
    p = OParams(dt=0.5)
    c0 = quench_field(shape, 0.1, 0.3, seed=71)
    assert rel_l2(gpu_run(evx_gpu, c0, bc, "stencil7", 1, p),
                  ch.ch_step(c0.astype(np.float64), p, bc, "stencil7")) <= 1e-5
    assert rel_l2(gpu_run(evx_gpu, c0, bc, "stencil7", 3, p),
                  ch.ch_run(c0, 3, p, bc, "stencil7")) <= 2e-5
