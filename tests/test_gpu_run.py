"""Steps taken several per launch (a single system whose tiles are all
resident) against steps of two launches each.

A launch configuration with a sort split of its own selects the separate
launches; neither may change anything: positions, velocities, forces,
properties, rebuild and late-binning counts, block means and traces equal bit
for bit, over every kind of system (whole-system window, no window, LDS
window; list, cell method; both precisions; overflowing lists and cell rows;
storage order kept; mixtures), over several calls, and while two systems step
at once from two threads on streams of their own (whose launches then find
only part of their workgroups running).
"""
import threading

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


def _fluid(lattice, edge, rho=0.8, seed=3):
    pos, L = (I.fcc_lattice if lattice == "fcc" else I.sc_lattice)(edge, rho)
    pos = I.jitter(pos, L, 0.06, seed)
    return pos, I.random_velocities(len(pos), 1.0, seed + 1), L


def _steps(s, calls, two_launches, species=None):
    if two_launches:
        s.configure(sort_split=1)
    if species is not None:
        s.set_species(*species)
    for n in calls:
        s.step(n)
    p, v, f, step = s.get_state()
    return [p, v, f, step, s.props()]


def _same(a, b):
    assert all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3]))
    assert a[3] == b[3] and a[4] == b[4]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("lattice,edge,prm", [
    ("fcc", 4, dict(shell=0.4)),                          # one tile
    ("fcc", 6, dict(shell=0.4)),                          # the system is its window
    ("fcc", 8, dict(shell=0.4)),                          # no window
    ("sc", 27, dict(shell=0.3)),                          # ragged last tile
    ("fcc", 8, dict(shell=0.0)),                          # cell method
    ("fcc", 10, dict(shell=0.4, reorder=False)),
    ("fcc", 10, dict(shell=0.4, reorder_interval=30)),
    ("fcc", 10, dict(shell=0.4, window=False)),
    ("fcc", 9, dict(shell=0.4, nebr_cap=8)),              # overflowing lists
    ("sc", 16, dict(shell=0.4, cell_cap=1)),              # overflowing cell rows
])
def test_run_equals_separate_launches(lattice, edge, prm, precision):
    from paper_0911_5631_amd.md import System
    pos, vel, L = _fluid(lattice, edge)
    calls = (1, 37, 300)
    out = []
    for two in (False, True):
        s = System(pos, vel, L, precision=precision, **prm)
        out.append(_steps(s, calls, two))
        s.close()
    _same(*out)
    assert out[0][3] == sum(calls)


def test_late_binning_in_a_run():
    """The rule firing where binning ahead would have missed it is counted
    alike (a lattice nearly at rest with one pair pushed together)."""
    from paper_0911_5631_amd.md import System
    pos, L = I.sc_lattice(16, 0.5)
    rng = np.random.Generator(np.random.PCG64(61))
    vel = rng.uniform(-0.005, 0.005, pos.shape)
    vel -= vel.mean(0)
    d = pos[1] - pos[0]
    d -= L * np.round(d / L)
    pos[0] = pos[1] - d / np.linalg.norm(d) * 0.9
    out = []
    for two in (False, True):
        s = System(pos, vel, L, shell=0.004)
        out.append(_steps(s, (40, 24), two))
        s.close()
    _same(*out)
    assert out[0][4]["n_late_bins"] >= 1


def test_mixture_block_and_trace_in_a_run():
    from paper_0911_5631_amd.md import System
    pos, vel, L = _fluid("fcc", 11, 0.7)
    sp = (np.random.Generator(np.random.PCG64(4)).permutation(len(pos)) % 2).astype(np.int32)
    tabs = I.binary_wca()
    out, more = [], []
    for two in (False, True):
        s = System(pos, vel, L, shell=0.4, r_cut=float(tabs[2].max()))
        out.append(_steps(s, (3, 150), two, (sp, *tabs)))
        s.close()
        s = System(pos, vel, L, shell=0.4, trace=True)
        if two:
            s.configure(sort_split=1)
        s.step(90)
        s.block_begin()
        s.step(75)
        b = s.block_end()
        more.append((s.trace(1, 165), b, s.get_state()[0]))
        s.close()
    _same(*out)
    assert np.array_equal(more[0][0], more[1][0]) and more[0][1] == more[1][1]
    assert np.array_equal(more[0][2], more[1][2])


def test_two_systems_at_once():
    import torch
    from paper_0911_5631_amd.md import System
    starts = [_fluid("fcc", 36, seed=s) for s in (5, 9)]      # 729 tiles each
    ref = []
    for pos, vel, L in starts:
        s = System(pos, vel, L, shell=0.4)
        ref.append(_steps(s, (400,), False))
        s.close()
    systems = [System(pos, vel, L, shell=0.4, stream=torch.cuda.Stream())
               for pos, vel, L in starts]
    got = [None, None]

    def work(k):
        torch.cuda.set_device(0)
        got[k] = _steps(systems[k], (130, 270), False)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in systems:
        s.close()
    for k in range(2):
        _same(ref[k], got[k])


def test_batch_run_equals_separate_launches():
    """A batch whose replicas are stepped by seats (more tiles than workgroups
    resident at once, both precisions, replicas that finish in between)
    against the same batch in separate launches."""
    from paper_0911_5631_amd.md import Batch
    systems = I.replica_batch(n_replicas=40, k_lo=6, k_hi=20, steps=0, seed=12)
    out = []
    for two in (False, True):
        b = Batch(1 << 33, 48, 32)
        slots = [b.admit(s.pos, s.vel, s.box, 70 + 13 * k, shell=s.shell,
                         precision="fp64" if k % 5 == 4 else "fp32")
                 for k, s in enumerate(systems)]
        if two:
            b.configure(steps_per_run=32, sort_split=1)
        for _ in range(4):
            b.run()
        done = b.poll()
        out.append(([b.get_state(s) for s in slots], [b.props(s) for s in slots], done))
        b.close()
    for (p, v, n), (q, w, m) in zip(out[0][0], out[1][0]):
        assert n == m and np.array_equal(p, q) and np.array_equal(v, w)
    assert out[0][1] == out[1][1] and out[0][2] == out[1][2]
