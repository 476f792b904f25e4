"""The z update's reciprocal against the IEEE division, bit for bit: all 2^23 mantissas at exponents
over the range its callers keep to (2^-100 to 2^120), and what it returns past it.  And the range is
kept: time steps so large that a denominator would leave it, against the FP64 oracle."""
import ctypes
import os

import numpy as np
import pytest
import torch

from oracle import ch, gray_scott as gs, reaction_diffusion as rd
from oracle.ch import CHParams
from paper_2507_21748_amd.inputs import quench_field
from tests.test_gpu_ch import rel_l2
from tests.test_gpu_gs import gpu_gs

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip", "libreciprocal.so")


def reciprocals(first, count):
    """evx_rcp of the floats whose bits are first, first + 1, ... (count of them)."""
    lib = ctypes.CDLL(LIB)
    lib.evx_test_reciprocal.argtypes = [ctypes.c_uint, ctypes.c_uint, ctypes.c_void_p,
                                        ctypes.c_void_p]
    out = torch.empty(count, dtype=torch.float32, device="cuda")
    assert lib.evx_test_reciprocal(first, count, out.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream) == 0
    return out.cpu().numpy()


@pytest.mark.parametrize("exponent", [-100, -61, -30, -1, 0, 1, 2, 7, 24, 63, 100, 119])
def test_every_mantissa(evx_gpu, exponent):
    first = (127 + exponent) << 23
    got = reciprocals(first, 1 << 23)
    x = np.arange(first, first + (1 << 23), dtype=np.uint32).view(np.float32)
    assert np.array_equal(got.view(np.uint32), (np.float32(1) / x).view(np.uint32))


def test_past_the_range(evx_gpu):
    for e in range(120, 128):
        got = reciprocals((127 + e) << 23, 1 << 16)
        assert np.all(got >= 0) and np.all(got <= 2.0 ** -120)
    assert reciprocals(0x7F800000, 1)[0] < 2.0 ** -127   # infinity
    assert np.isnan(reciprocals(0x7FC00000, 1)[0])


SHAPE = (12, 16, 20)
BOUND = 1e-5  # one step, as everywhere: its transforms round at a few FP32 ulps


@pytest.mark.parametrize("bc", ["periodic", "zero_flux"])
@pytest.mark.parametrize("dt", [1e30, 5e34, 2e35])
def test_cahn_hilliard_steps(evx_gpu, bc, dt):
    p = CHParams(dt=dt)
    c0 = quench_field(SHAPE, 0.0, 0.01, seed=81)
    plan = evx_gpu.Plan(SHAPE, bc, "spectral")
    c = torch.from_numpy(c0).cuda()
    plan.step(c, 1, evx_gpu.CHParams(dt=dt))
    assert rel_l2(c.cpu().numpy(), ch.ch_step(c0.astype(np.float64), p, bc, "spectral")) <= BOUND


@pytest.mark.parametrize("dt", [1e30, 2e37, 6e37])
def test_allen_cahn_steps(evx_gpu, dt):
    c0 = quench_field(SHAPE, 0.0, 0.01, seed=82)
    plan = evx_gpu.Plan(SHAPE, "periodic", "stencil7")
    c = torch.from_numpy(c0).cuda()
    plan.step(c, 1, evx_gpu.CHParams(dt=dt, model=evx_gpu.ALLEN_CAHN))
    ref = ch.ac_run(c0, 1, CHParams(dt=dt), "periodic", "stencil7")
    assert rel_l2(c.cpu().numpy(), ref) <= BOUND


def test_reaction_diffusion_step(evx_gpu):
    c0 = quench_field(SHAPE, 0.0, 0.01, seed=83)
    plan = evx_gpu.Plan(SHAPE, "periodic", "stencil7")
    c = torch.from_numpy(c0).cuda()
    plan.rd_step(c, 1, evx_gpu.RDParams(dt=6e37, A=2.0, D=0.1, a1=1.0, a2=0.0, a3=-1.0))
    p = rd.RDParams(dt=6e37, A=2.0, D=0.1, a0=0.0, a1=1.0, a2=0.0, a3=-1.0)
    assert rel_l2(c.cpu().numpy(), rd.rd_run(c0, 1, p, "periodic", "stencil7")) <= BOUND


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
def test_gray_scott_step(evx_gpu, bc):
    """Diffusion of everything but the mean in one step, beside a reaction of order one."""
    p = gs.GSParams(dt=0.5, Du=2e37, Dv=5e36)
    u0, v0 = quench_field(SHAPE, 0.7, 0.3, seed=84), quench_field(SHAPE, 0.2, 0.2, seed=85)
    for n in (1, 3):
        got = gpu_gs(evx_gpu, u0, v0, bc, "stencil7", n, p)
        for a, b in zip(got, gs.gs_run(u0, v0, n, p, bc, "stencil7")):
            assert np.abs(a - b).max() <= BOUND
