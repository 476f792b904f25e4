"""Inference with the mass projection where the last layer's workgroups, which leave the projection's
sums, are ragged: fields narrower than a tile, one column and a remainder, one plane.  Against the
same field without it: the shift is the FP64 mean of the increments, rounded once, so results agree
to one FP32 rounding of values of order one (2e-7), and the mean is kept to 1e-6."""
import pytest
import torch

from paper_2507_21748_amd.surrogate import Net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 5, 7), (3, 16, 16), (9, 17, 33), (40, 20, 18)])
def test_projection_sums(evx_gpu, shape):
    print(f"mass projection {shape}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    c = torch.randn(shape, generator=g, device="cuda").mul_(0.5)
    net = Net(seed=3)
    free = net.infer(c).clone()
    kept = net.infer(c, conserve_mass=True)
    shift = (free.double() - c.double()).mean()
    assert float((kept.double() - (free.double() - shift)).abs().max()) <= 2e-7 * float(
        1 + free.abs().max())
    assert abs(float(kept.double().mean() - c.double().mean())) <= 1e-6
