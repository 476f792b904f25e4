"""The passes that reuse one exchange area several times a workgroup, under the thread sanitizer and
against the FP64 oracle: the adjoint step (its z pass with the spectral work, and on a periodic x the
x pass that combines both inverse transforms), the diagnostics, Gray-Scott with and without spectral
states, the stencil on zero-flux axes and the plane pass.  Transforms of several stages along every
axis a body works on (a single-stage transform exchanges nothing), each boundary family once."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

from oracle import adjoint, ch
from oracle.ch import CHParams
from paper_2507_21748_amd.inputs import quench_field
from tests.test_emulator import _rel, _run, _vm_emulated, tsan  # noqa: F401 (fixture)
from tests.test_emulator_gs_vertex import CODE, VX, gs_emulated


def _emulate(exe, args, inputs, outputs):
    """One emulator run: arrays in, the named outputs' raw bytes back, no race reported."""
    with tempfile.TemporaryDirectory() as d:
        paths = []
        for k, a in enumerate(inputs):
            paths.append(os.path.join(d, f"in{k}"))
            a.tofile(paths[-1])
        outs = [os.path.join(d, f"out{k}") for k in range(len(outputs))]
        r = subprocess.run([exe, *args, *paths, *outs], capture_output=True, text=True, timeout=600,
                           env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))
        assert r.returncode == 0, r.stderr[-4000:]
        assert "WARNING: ThreadSanitizer" not in r.stderr, r.stderr[-4000:]
        return [np.fromfile(o, t) for o, t in zip(outs, outputs)]


GRIDS = [((24, 8, 48), "periodic", "spectral"),
         ((24, 8, 24), "zero_flux", "stencil7"),
         ((24, 24, 8), ("dirichlet", "periodic", "zero_flux"), "spectral")]


@pytest.mark.parametrize("shape,bc,scheme", GRIDS)
def test_adjoint_and_diagnostics(tsan, shape, bc, scheme):  # noqa: F811
    p = CHParams(dt=0.5, M=0.8, kappa=1.3, A=2.0)
    c = quench_field(shape, 0.1, 0.4, seed=3)
    lam = quench_field(shape, 0.0, 1.0, seed=4)
    c1 = ch.ch_step(c.astype(np.float64), p, bc, scheme)
    _, g, _, _ = adjoint.adjoint_gradients(c, c1 - lam.astype(np.float64) / 2, 1, p, bc, scheme)
    bcarg = CODE[bc] if isinstance(bc, str) else \
        1000 + 100 * CODE[bc[2]] + 10 * CODE[bc[1]] + CODE[bc[0]]
    geo = [*map(str, shape[::-1]), str(bcarg), str(int(scheme == "stencil7")), "1"]
    lo, gr = _emulate(tsan, ["adj", *geo, repr(p.dt), repr(p.M), repr(p.kappa), repr(p.A)],
                      [c, lam], [np.float32, np.float64])
    assert _rel(lo.reshape(shape), g) <= 1e-6
    assert np.isfinite(gr).all()  # (their values: test_emulated_adjoint_step_and_diagnostics)
    o, = _emulate(tsan, ["diag", *geo, repr(p.kappa)], [c], [np.float64])
    assert abs(o[0] - ch.mass(c.astype(np.float64))) <= 1e-9 * c.size
    assert abs(o[1] / ch.energy(c.astype(np.float64), p, bc, scheme) - 1) <= 1e-6


@pytest.mark.parametrize("shape,bc", [((24, 8, 48), "periodic"), ((24, 8, 24), "zero_flux"),
                                      ((24, 8, 24), "dirichlet"),
                                      ((8, 9, 25), ("zero_flux", VX, VX))])
def test_gray_scott(tsan, shape, bc):  # noqa: F811
    got, ref = gs_emulated(tsan, shape, bc, "spectral", 2)
    for a, b in zip(got, ref):
        assert _rel(a, b) <= 1e-6


def test_stencil_on_zero_flux_axes(tsan):  # noqa: F811
    out, ref, _ = _vm_emulated(tsan, (12, 24, 24), "zero_flux", "stencil7")
    assert _rel(out, ref) <= 1e-6


def test_plane_pass(tsan):  # noqa: F811
    p = CHParams(dt=0.5)
    c0 = quench_field((8, 32, 32), 0.1, 0.3, seed=15)
    got = _run(tsan, (8, 32, 32), "periodic", "spectral", 1, p, c0)
    assert _rel(got, ch.ch_step(c0.astype(np.float64), p, "periodic", "spectral")) <= 1e-6
