"""The fused variable-mobility stencil at the edges of its 32 x 32 columns: grids narrower than a
halo, one column and a remainder, exact multiples, and z ranges of one block and several, on
periodic, zero-flux and mixed axes.  One step against the FP64 oracle: the field within 1e-5 and
its increment within 1e-4 relative L2 (the stencil's differences amplify FP32 rounding of phi by
about its coefficients, 1e2 x 6e-8, against increments of order one)."""
import pytest

from oracle import ch_varmob as vm
from paper_2507_21748_amd.inputs import quench_field
from tests.test_gpu_vm import P, gpu_vm, rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4, 8), (6, 8, 32), (64, 32, 40), (16, 64, 64), (10, 100, 40), (128, 24, 96)]
BCS = ["periodic", "zero_flux", ("zero_flux", "periodic", "zero_flux"),
       ("periodic", "zero_flux", "periodic")]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", BCS, ids=["periodic", "zero_flux", "zpz", "pzp"])
def test_stencil_columns(evx_gpu, shape, bc):
    print(f"stencil columns {shape} {bc}", flush=True)
    phi0 = quench_field(shape, 0.5, 0.2, seed=83)
    got = gpu_vm(evx_gpu, phi0, bc, "stencil7", 1, P)
    ref = vm.vm_step(phi0.astype("float64"), P, bc, "stencil7")
    assert rel_l2(got, ref) <= 1e-5
    assert rel_l2(got - phi0, ref - phi0) <= 1e-4
