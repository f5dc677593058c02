"""The traversal over packed positions against the general one.

A rebuild (or a cell step) first tests 16-bit packed positions and then the
few candidates that pass exactly; a system whose cell-layer rows have no room
for the packed array (here: cell_cap = 1, the surplus in the overflow list)
takes the general traversal instead.  Both visit the same candidates in the
same order, so pairs (in list order), forces and trajectories must be the
same bit for bit: at the smallest grid (3 cells per edge, every lane at an
x-edge), rows of more than 32 candidates (several groups of bits), tiles with
one atom or a full one, each precision, with and without a list.
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


def _start(lattice, edge, rho, seed):
    pos, L = (I.fcc_lattice if lattice == "fcc" else I.sc_lattice)(edge, rho)
    pos = I.jitter(pos, L, 0.08, seed)
    return pos, I.random_velocities(len(pos), 1.0, seed + 1), L


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("lattice,edge,rho,prm", [
    ("fcc", 3, 0.8, dict(shell=0.4)),                # 108 atoms, 3 cells per edge
    ("fcc", 4, 0.8, dict(shell=0.5)),                # 256 atoms: one full tile
    ("sc", 13, 0.8, dict(shell=0.4)),                # 2 197 atoms, a ragged last tile
    ("fcc", 8, 0.9, dict(shell=0.0)),                # cell method
    ("sc", 11, 0.38, dict(shell=0.8, r_cut=2.5)),    # ~60 candidates per row
    ("sc", 12, 0.38, dict(shell=0.4, r_cut=3.0)),    # ~80 candidates per row
])
def test_packed_traversal_equals_the_general_one(lattice, edge, rho, prm, precision):
    from paper_0911_5631_amd.md import System
    pos, vel, L = _start(lattice, edge, rho, 5 + edge)
    out = []
    for cap in (0, 1):
        s = System(pos, vel, L, precision=precision, cell_cap=cap, **prm)
        f0 = s.get_state()[2]
        pairs = s.pairs() if prm["shell"] > 0 else (np.zeros(0), np.zeros(0))
        s.step(90)
        p, v, f, step = s.get_state()
        pr = s.props()
        s.close()
        assert step == 90
        out.append((f0, *pairs, p, v, f, pr["pe"], pr["virial"], pr["n_rebuilds"], pr["n_pairs"]))
    assert all(np.array_equal(a, b) for a, b in zip(*out))


def test_list_overflow_after_the_packed_test():
    """Atoms with more nearly-near candidates than the list holds are listed
    again exactly; the trajectory equals that of a list with room."""
    from paper_0911_5631_amd.md import System
    pos, vel, L = _start("fcc", 6, 0.85, 31)
    ref = None
    for cap in (48, 12, 5):
        s = System(pos, vel, L, shell=0.4, nebr_cap=cap)
        s.step(60)
        p, v, f, _ = s.get_state()
        pr = s.props()
        s.close()
        got = (p, v, f, pr["pe"], pr["n_pairs"], pr["max_nebr"])
        if ref is None:
            ref = got
        assert all(np.array_equal(a, b) for a, b in zip(ref, got)), cap
