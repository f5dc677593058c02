"""Errors that arise while a launch takes many steps: every workgroup of it
stops at the same step, so a repairable one (cell rows that outgrow their
overflow list of 4 096 atoms while a crystal of four atoms a cell melts) is
repaired and the run resumed, and a lasting one is reported with the steps
that were completed, as in launches of one step (selected by a sort split)."""
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
@pytest.mark.parametrize("steps,prm", [
    (200, dict(shell=0.55)),                     # rebuilds now and then
    (600, dict(r_cut=1.69, shell=0.0)),          # bins every step (and melts later)
])
def test_cell_rows_overflow_in_a_run(steps, prm, precision):
    from paper_0911_5631_amd.md import System
    pos, L = I.fcc_lattice(30, 0.8)                                  # 30 cells an edge
    vel = I.random_velocities(len(pos), 1.0, 5)
    out = []
    for two in (False, True):
        s = System(pos, vel, L, cell_cap=4, precision=precision, **prm)
        assert s.props()["cells_per_edge"] == 30 and s.props()["max_cell"] == 4
        if two:
            s.configure(sort_split=1)
        for n in (60, steps - 60):
            s.step(n)
        p, v, f, step = s.get_state()
        out.append((p, v, f, step, s.props()))
        cells = np.bincount(s.cells(), minlength=30 ** 3)
        assert np.maximum(cells - 4, 0).sum() > 4096
        s.close()
    a, b = out
    assert a[3] == b[3] == steps and a[4] == b[4]
    assert all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3]))


@pytest.mark.parametrize("shell", [0.4, 0.0])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_lasting_error_in_a_run(precision, shell):
    """A time step far too long: the atoms leave the box within 40 steps."""
    from paper_0911_5631_amd import _lib as L
    from paper_0911_5631_amd.md import System
    pos, box = I.fcc_lattice(9, 0.8)
    vel = I.random_velocities(len(pos), 5.0, 5)
    out = []
    for two in (False, True):
        s = System(pos, vel, box, shell=shell, dt=0.015, precision=precision)
        if two:
            s.configure(sort_split=1)
        s.step(200)
        p = L.md_props_t()
        st = L.lib().md_props(s._h, C.byref(p))
        out.append((st, p.step, p.n_rebuilds))
        s.close()
    assert out[0] == out[1]
    assert out[0][0] in (-6, -7) and 0 < out[0][1] < 200
