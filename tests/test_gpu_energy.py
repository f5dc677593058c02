"""Steps that sum energies against steps that do not.

Outside a block only the last step of a call sums energies and virials: its
list loop reads the entries again and is compiled apart from that of the
other steps.  A traced system sums them at every step, with one loop.  Both
add the same pairs in the same order, so the state, every atom's energy and
virial and the properties at the end of each call must be the same bit for
bit: lists that fit the held entries, longer ones, ones cut short, calls of
one step and of several, one launch per step and many.
"""
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


@pytest.mark.parametrize("two_launches", [False, True])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("edge,rho,prm", [
    (9, 0.8, dict(shell=0.4)),                    # ~12 entries, a ragged last tile
    (12, 0.38, dict(shell=0.8, r_cut=3.0)),       # ~90 entries
    (9, 0.8, dict(shell=0.4, nebr_cap=9)),        # most lists overflow
])
def test_last_step_sums_what_a_traced_step_sums(edge, rho, prm, precision, two_launches):
    from paper_0911_5631_amd.md import System
    pos, L = I.sc_lattice(edge, rho)
    pos = I.jitter(pos, L, 0.06, edge)
    vel = I.random_velocities(len(pos), 1.0, edge + 1)
    out = []
    for trace in (False, True):
        s = System(pos, vel, L, precision=precision, trace=trace, **prm)
        if two_launches:
            s.configure(sort_split=1)
        got = []
        for n in (1, 2, 37, 1):
            s.step(n)
            pr = s.props()
            got += [*s.get_state()[:3], *s.atom_energies(), pr["ke"], pr["pe"], pr["virial"],
                    pr["n_pairs"]]
        s.close()
        out.append(got)
    assert all(np.array_equal(a, b) for a, b in zip(*out))
