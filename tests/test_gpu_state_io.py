"""State to and from the host through the pinned buffers: every subset of the
arrays md_get_state copies, one run of atoms or several (62^3 = 238 328 atoms
with positions, velocities and forces are more than one 16 MiB buffer), sizes
that fill no whole workgroup, the caller's order kept through sorts."""
import ctypes as C

import numpy as np
import pytest

from paper_0911_5631_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    yield


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("edge", [6, 17, 62])
def test_state_round_trip_and_subsets(edge, precision):
    from paper_0911_5631_amd import _lib as L
    from paper_0911_5631_amd.md import System
    pos, box = I.sc_lattice(edge, 0.7)
    pos = I.jitter(pos, box, 0.05, 2)
    vel = I.random_velocities(len(pos), 1.0, 3)
    pos, vel = I.shuffled(pos, vel, 4)
    s = System(pos, vel, box, shell=0.4, precision=precision)
    p, v, f, step = s.get_state()
    assert step == 0 and np.array_equal(p, pos) and np.array_equal(v, vel)
    s.step(40)
    p, v, f, step = s.get_state()
    assert step == 40
    n = len(pos)
    for what in range(8):
        out = [np.full((n, 3), np.nan) if what >> k & 1 else None for k in range(3)]
        k = C.c_int64(-1)
        ptr = [None if a is None else a.ctypes.data_as(C.POINTER(C.c_double)) for a in out]
        assert L.lib().md_get_state(s._h, *ptr, C.byref(k)) == 0 and k.value == 40
        for a, ref in zip(out, (p, v, f)):
            assert a is None or np.array_equal(a, ref)
    u, w = s.atom_energies()
    pr = s.props()
    assert abs(0.5 * u.sum() - pr["pe"]) <= 1e-6 * n and abs(0.5 * w.sum() - pr["virial"]) <= 1e-5 * n
    # the held state of the next step of another system
    s.set_state(p, v)
    p2, v2, f2, _ = s.get_state()
    d = p2 - p
    assert np.array_equal(v2, v) and np.all((d == 0) | (np.abs(np.abs(d) - box) < 1e-12 * box))
    s.close()
