"""The two-species x pass (both species' rows, the reaction between the transforms) at the edges of
its forms: rows that do not fill a workgroup, lane counts that are no multiple of 8 columns, packed
species on cosine rows, complex cosine columns, vertex-centred rows, and Dirichlet signs, which the
constant feed alone does not carry.  Against the FP64 oracle, relative L2 1e-5 after one step (real
rows in) and 2e-5 after four (the spectral form): a step's transforms round at a few FP32 ulps."""
import os

import pytest

from oracle import ch, gray_scott as gs
from paper_2507_21748_amd.inputs import quench_field
from tests.test_gpu_gs import gpu_gs, rel_l2

pytestmark = pytest.mark.gpu

ch.WORKERS = min(16, os.cpu_count() or 1)

CASES = [
    ((6, 10, 40), "periodic"),
    ((6, 10, 200), "periodic"),
    ((6, 10, 12), "zero_flux"),
    ((6, 10, 100), "zero_flux"),
    ((6, 10, 400), "zero_flux"),
    ((12, 10, 48), "dirichlet"),
    ((6, 12, 64), ("dirichlet", "dirichlet", "periodic")),
    ((6, 10, 96), ("zero_flux", "periodic", "dirichlet")),
    ((6, 10, 33), ("periodic", "zero_flux", "zero_flux_vertex")),
    ((9, 10, 24), ("zero_flux_vertex", "periodic", "zero_flux")),
]


@pytest.mark.parametrize("shape,bc", CASES)
def test_two_species_rows(evx_gpu, shape, bc):
    print(f"two-species rows {shape} {bc}", flush=True)
    p = gs.GSParams(dt=0.8)
    u0 = quench_field(shape, 0.7, 0.3, seed=73)
    v0 = quench_field(shape, 0.2, 0.2, seed=74)
    for n, bound in ((1, 1e-5), (4, 2e-5)):
        got = gpu_gs(evx_gpu, u0, v0, bc, "stencil7", n, p)
        for a, b in zip(got, gs.gs_run(u0, v0, n, p, bc, "stencil7")):
            assert rel_l2(a, b) <= bound
