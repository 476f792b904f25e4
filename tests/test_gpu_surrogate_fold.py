"""The mass projection on planes of so many columns that its sums are folded first: just past the
line, a ragged last fold, and two planes.  As in the projection's other tests, against the same field
without it: one FP32 rounding of values of order one (2e-7), the mean kept to 1e-6."""
import pytest
import torch

from paper_2507_21748_amd.surrogate import Net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1024, 1025), (1, 1500, 1100), (3, 1040, 1024)])
def test_projection_of_many_columns(evx_gpu, shape):
    print(f"mass projection {shape}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    c = torch.randn(shape, generator=g, device="cuda").mul_(0.5)
    net = Net(seed=3)
    free = net.infer(c).clone()
    shift = (free.double() - c.double()).mean()
    for _ in range(2):  # the sums of a second call are its own
        kept = net.infer(c, conserve_mass=True)
        assert float((kept.double() - (free.double() - shift)).abs().max()) <= 2e-7 * float(
            1 + free.abs().max())
        assert abs(float(kept.double().mean() - c.double().mean())) <= 1e-6
