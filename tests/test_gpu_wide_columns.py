"""Column passes on the wide workgroups of large grids (z lengths 64 and 128, y or z lengths 50 and
100), against the narrow ones of small grids: a field repeated along its periodic axes steps as the
field itself.  Each side is within 1e-5 of the exact step (relative L2, as everywhere), so the two are
within 2e-5, and after three steps within 4e-5.  And a stored state resumes to the bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P, Z, D, V = "periodic", "zero_flux", "dirichlet", "zero_flux_vertex"
CASES = [((64, 256, 256), (P, P, P), (1, 2, 2)),
         ((128, 128, 128), (Z, P, P), (1, 2, 4)),
         ((33, 256, 256), (V, P, P), (1, 2, 2)),      # transform length 64
         ((65, 128, 128), (V, P, P), (1, 2, 4)),      # 128
         ((50, 128, 128), (P, P, P), (1, 2, 2)),
         ((100, 96, 96), (D, P, P), (1, 2, 2)),
         ((51, 96, 96), (V, P, P), (1, 2, 2)),        # 100
         ((96, 50, 96), (P, Z, P), (4, 1, 4)),
         ((96, 100, 100), (P, P, P), (2, 1, 2))]


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("shape,bc,tile", CASES)
@pytest.mark.parametrize("kind", ["semi-implicit", "etd1", "allen-cahn", "reaction"])
def test_tiled_field(evx_gpu, shape, bc, tile, kind):
    evx = evx_gpu
    print(f"wide columns {shape} {bc} x {tile} {kind}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(91)
    c0 = torch.rand(shape, generator=g, device="cuda").mul_(0.6).sub_(0.3)
    small = evx.Plan(shape, bc, "stencil7")
    large = evx.Plan(tuple(n * k for n, k in zip(shape, tile)), bc, "stencil7")
    for n, bound in ((1, 2e-5), (3, 4e-5)):
        a, b = c0.clone(), c0.repeat(tile)
        for plan, c in ((small, a), (large, b)):
            if kind == "reaction":
                plan.rd_step(c, n, evx.RDParams(dt=0.2, a1=1.0, a2=0.0, a3=-1.0))
            else:
                plan.step(c, n, evx.CHParams(
                    dt=0.5, integrator=evx.ETD1 if kind == "etd1" else evx.SEMI_IMPLICIT,
                    model=evx.ALLEN_CAHN if kind == "allen-cahn" else evx.CAHN_HILLIARD))
        assert _rel(b, a.repeat(tile)) <= bound


@pytest.mark.parametrize("shape,bc", [((128, 256, 512), (P, P, P)), ((100, 192, 192), (Z, P, Z))])
def test_state_resumes(evx_gpu, shape, bc):
    evx = evx_gpu
    g = torch.Generator(device="cuda").manual_seed(92)
    c0 = torch.rand(shape, generator=g, device="cuda").mul_(0.6).sub_(0.3)
    q = evx.CHParams(dt=0.5)
    a, b = torch.empty_like(c0), torch.empty_like(c0)
    plan = evx.Plan(shape, bc, "stencil7")
    plan.begin(c0)
    plan.advance(2, q)
    saved = plan.state().clone()
    plan.advance(2, q)
    plan.end(a)
    other = evx.Plan(shape, bc, "stencil7")
    other.state().copy_(saved)
    other.restore()
    other.advance(2, q)
    other.end(b)
    assert torch.equal(a, b)
