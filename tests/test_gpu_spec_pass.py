"""The z pass that carries the adjoint's and the energy's spectral work, at the lengths where it can
go wrong: one stage and several, lane counts that are no power of two (its block sum), the shortest
and longest, ragged last workgroups, complex and pair columns, every weight of the Parseval sum.
Checks and bounds are those of the adjoint's and diagnostics' own parity tests (one step 1e-5, energy
1e-6: a few FP32 ulps of the transforms)."""
import pytest

from tests import test_gpu_adjoint as base

pytestmark = pytest.mark.gpu

MIX = ("periodic", "zero_flux", "zero_flux")
CASES = [((n, 6, 12), bc) for n in (4, 10, 50, 100, 200, 256, 384) for bc in ("periodic", "zero_flux")]
CASES += [((40, 10, 20), MIX), ((512, 4, 8), "periodic"), ((400, 5 * 2, 16), "dirichlet"),
          ((24, 20, 16), ("zero_flux", "periodic", "dirichlet")), ((1024, 4, 8), "periodic")]


@pytest.mark.parametrize("shape,bc", CASES)
def test_adjoint_and_energy(evx_gpu, shape, bc):
    print(f"spectral z pass {shape} {bc}", flush=True)
    base.test_one_adjoint_step(evx_gpu, shape, bc, "stencil7")
    base.test_diagnostics(evx_gpu, shape, bc, "stencil7")
