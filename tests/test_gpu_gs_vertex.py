"""Gray-Scott on grids with a vertex-centred z and a Dirichlet axis: the species' spectral states are
read mirrored by one lane of the z pass and stored by another.  One z length per form of the transform
(one lane, several lanes, several waves a column), against the FP64 oracle, relative L2 1e-5 after one
step and 2e-5 after four (a step's transforms round at a few FP32 ulps)."""
import os

import pytest

from oracle import ch, gray_scott as gs
from paper_2507_21748_amd.inputs import quench_field
from tests.test_gpu_gs import gpu_gs, rel_l2

pytestmark = pytest.mark.gpu

ch.WORKERS = min(16, os.cpu_count() or 1)

VX = "zero_flux_vertex"


@pytest.mark.parametrize("nz", [7, 9, 25, 33, 101, 129, 257])
@pytest.mark.parametrize("bc", [("periodic", "dirichlet"), ("dirichlet", "periodic"),
                                (VX, "dirichlet")], ids=["x", "y", "vertex-y"])
def test_states_on_a_vertex_z(evx_gpu, nz, bc):
    shape = (nz, 13 if bc[0] == VX else 12, 16)
    print(f"gray-scott states {shape} {bc}", flush=True)
    p = gs.GSParams(dt=0.8)
    u0 = quench_field(shape, 0.7, 0.3, seed=75)
    v0 = quench_field(shape, 0.2, 0.2, seed=76)
    for n, bound in ((1, 1e-5), (4, 2e-5)):
        got = gpu_gs(evx_gpu, u0, v0, (VX, *bc), "stencil7", n, p)
        for a, b in zip(got, gs.gs_run(u0, v0, n, p, (VX, *bc), "stencil7")):
            assert rel_l2(a, b) <= bound
