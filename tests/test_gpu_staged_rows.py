"""The x pass of short rows on grids of many rows, which moves its spectral rows through LDS.
A field repeated along z and y steps as the field itself does on a small grid, whose rows move directly:
each side is within 1e-5 of the exact step (relative L2, as everywhere), so the two are within 2e-5, and
after three steps within 4e-5.  Row counts that fill no workgroup (vertex-centred z and y) against the
FP64 oracle."""
import os

import numpy as np
import pytest
import torch

from oracle import ch
from paper_2507_21748_amd.inputs import quench_field
from tests.test_gpu_ch import gpu_run, rel_l2

pytestmark = pytest.mark.gpu

ch.WORKERS = min(16, os.cpu_count() or 1)

P, Z, D, V = "periodic", "zero_flux", "dirichlet", "zero_flux_vertex"
# one, two and four lanes a row; the vertex-centred rows are read and stored point by point
ROWS = [(8, P), (12, P), (16, P), (20, P), (24, P), (40, P), (48, P), (80, P), (32, P), (64, P),
        (96, P), (160, P), (9, V), (21, V), (25, V), (49, V), (8, Z), (12, D), (16, Z), (20, Z),
        (24, D), (32, Z), (40, Z), (48, Z), (80, D)]


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("nx,bc", ROWS)
def test_repeated_field(evx_gpu, nx, bc):
    evx = evx_gpu
    print(f"staged rows {nx} {bc}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(93)
    shape, tile = (32, 64, nx), (8, 8, 1)
    c0 = torch.rand(shape, generator=g, device="cuda").mul_(0.4).add_(0.3)
    ops = evx.OP_STEP | evx.OP_VAR_MOBILITY
    plans = [evx.Plan(s, (P, P, bc), "stencil7", ops=ops)
             for s in (shape, tuple(n * k for n, k in zip(shape, tile)))]

    def run(call, n, bound):
        a, b = (call(plan, c) for plan, c in zip(plans, (c0.clone(), c0.repeat(tile))))
        assert _rel(b, a.repeat(tile)) <= bound * (2 if n > 1 else 1)

    for n in (1, 3):
        run(lambda plan, c: plan.step(c, n, evx.CHParams(dt=0.5)), n, 2e-5)
        run(lambda plan, c: plan.rd_step(c, n, evx.RDParams(dt=0.2, a1=1.0, a2=0.0, a3=-1.0)), n, 2e-5)
        if bc in (P, Z):
            run(lambda plan, c: plan.vm_step(c, n, evx.VMParams(dt=0.05)), n, 2e-5)
    # recorded fields are those of the steps, to the bit
    for plan, c in zip(plans, (c0.clone(), c0.repeat(tile))):
        traj = torch.empty((2, *c.shape), device="cuda")
        plan.begin(c)
        plan.advance_record(2, evx.CHParams(dt=0.5), traj)
        one = torch.empty_like(c)
        plan.begin(c)
        plan.advance(1, evx.CHParams(dt=0.5))
        plan.end(one)
        assert torch.equal(traj[1], one)


@pytest.mark.parametrize("shape,bc", [((129, 257, 16), P), ((129, 257, 24), P), ((129, 257, 80), P),
                                      ((257, 513, 12), Z), ((257, 513, 20), D)])
def test_ragged_last_workgroup(evx_gpu, shape, bc):
    print(f"staged rows {shape} {bc}", flush=True)
    p = ch.CHParams(dt=0.5)
    c0 = quench_field(shape, 0.1, 0.3, seed=94)
    assert rel_l2(gpu_run(evx_gpu, c0, (V, V, bc), "stencil7", 1, p),
                  ch.ch_step(c0.astype(np.float64), p, (V, V, bc), "stencil7")) <= 1e-5
