"""Gray-Scott on grids with a vertex-centred z and a Dirichlet axis, in the host emulator: the species'
spectral states are then read mirrored by one lane and stored by another, so the z pass has to keep
the two apart.  Z lengths of several transform stages (25 and 33 points transform 48 and 64), where
the mirrored rows belong to other lanes.  The address sanitizer's build holds the result against the
FP64 oracle, the thread sanitizer's reports any unordered pair of accesses."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

from oracle import gray_scott as gs
from paper_2507_21748_amd.inputs import quench_field
from tests.test_emulator import _build, _rel

CODE = {"periodic": 0, "zero_flux": 1, "dirichlet": 2, "zero_flux_vertex": 3}
VX = "zero_flux_vertex"


def gs_emulated(exe, shape, bc, scheme, nsteps):
    """nsteps of the emulated schedule and of the oracle: ((u, v), (u, v))."""
    p = gs.GSParams(dt=0.8)
    u0 = quench_field(shape, 0.7, 0.3, seed=31)
    v0 = quench_field(shape, 0.2, 0.2, seed=32)
    nz, ny, nx = shape
    bcarg = CODE[bc] if isinstance(bc, str) else \
        1000 + 100 * CODE[bc[2]] + 10 * CODE[bc[1]] + CODE[bc[0]]
    with tempfile.TemporaryDirectory() as d:
        path = {k: os.path.join(d, k) for k in ("u", "v", "uo", "vo")}
        u0.tofile(path["u"])
        v0.tofile(path["v"])
        r = subprocess.run([exe, "gs", str(nx), str(ny), str(nz), str(bcarg),
                            str(int(scheme == "stencil7")), "1.0", repr(p.dt), repr(p.Du),
                            repr(p.Dv), repr(p.F), repr(p.k), str(nsteps), *path.values()],
                           capture_output=True, text=True, timeout=600,
                           env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1",
                                    ASAN_OPTIONS="detect_leaks=0"))
        assert r.returncode == 0, r.stderr[-4000:]
        assert "WARNING: ThreadSanitizer" not in r.stderr, r.stderr[-4000:]
        out = [np.fromfile(path[k], np.float32).reshape(shape) for k in ("uo", "vo")]
    return out, gs.gs_run(u0, v0, nsteps, p, bc, scheme)


@pytest.mark.parametrize("kind", ["asan", "tsan"])
@pytest.mark.parametrize("shape,bc", [((25, 8, 8), (VX, "periodic", "dirichlet")),
                                      ((33, 8, 16), (VX, "dirichlet", "periodic")),
                                      ((9, 9, 8), (VX, VX, "dirichlet"))])
def test_states_on_a_vertex_z(kind, shape, bc):
    got, ref = gs_emulated(_build(kind), shape, bc, "stencil7", 2)
    for a, b in zip(got, ref):
        assert _rel(a, b) <= 1e-6


@pytest.mark.parametrize("kind", ["asan", "tsan"])
def test_one_step(kind):
    """A call of one step takes its reactions from the real fields."""
    got, ref = gs_emulated(_build(kind), (25, 8, 8), (VX, "periodic", "dirichlet"), "stencil7", 1)
    for a, b in zip(got, ref):
        assert _rel(a, b) <= 1e-6
