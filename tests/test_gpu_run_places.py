"""Launches of many steps that not all workgroups come to (as when other work
fills the chip): those that take part step several tiles each and hold none of
them from step to step.  MD_RUN_WORKGROUPS admits at most so many to the roll
call; whatever the number, every result equals the whole launch's bit for bit:
list and cell method, both precisions, overflowing lists, storage order kept,
mixtures, blocks, traces, batches, and a launch that stops at an error."""
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


def _fluid(edge, seed, rho=0.8):
    pos, L = I.fcc_lattice(edge, rho)
    pos = I.jitter(pos, L, 0.06, seed)
    return pos, I.random_velocities(len(pos), 1.0, seed + 1), L


def _limit(monkeypatch, places):
    if places:
        monkeypatch.setenv("MD_RUN_WORKGROUPS", str(places))
    else:
        monkeypatch.delenv("MD_RUN_WORKGROUPS", raising=False)


# 54 tiles, 56 workgroups: more than one of the 32 groups that count them has
# two members; 1: no barrier partner, 31-33: groups of one, 55: one missing
@pytest.mark.parametrize("places", [1, 5, 31, 33, 55])
@pytest.mark.parametrize("prm", [
    dict(shell=0.4), dict(shell=0.4, precision="fp64"), dict(shell=0.0),
    dict(shell=0.4, nebr_cap=8), dict(shell=0.4, reorder_interval=30),
])
def test_fewer_workgroups_than_tiles(places, prm, monkeypatch):
    from paper_0911_5631_amd.md import System
    pos, vel, L = _fluid(15, 3)
    out = []
    for lim in (0, places):
        _limit(monkeypatch, lim)
        s = System(pos, vel, L, trace=True, **prm)
        for n in (1, 37, 70):
            s.step(n)
        s.block_begin()
        s.step(40)
        b = s.block_end()
        out.append((*s.get_state(), s.props(), b, s.trace(1, 148)))
        s.close()
    a, b = out
    assert all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3]))
    assert a[3] == b[3] == 148 and a[4] == b[4] and a[5] == b[5] and np.array_equal(a[6], b[6])


@pytest.mark.parametrize("places", [3, 20])
def test_mixture_and_batch(places, monkeypatch):
    from paper_0911_5631_amd.md import Batch, System
    pos, vel, L = _fluid(11, 5, 0.7)
    sp = (np.random.Generator(np.random.PCG64(4)).permutation(len(pos)) % 2).astype(np.int32)
    tabs = I.binary_wca()
    systems = I.replica_batch(n_replicas=12, k_lo=6, k_hi=16, steps=0, seed=12)
    out = []
    for lim in (0, places):
        _limit(monkeypatch, lim)
        s = System(pos, vel, L, shell=0.4, r_cut=float(tabs[2].max()))
        s.set_species(sp, *tabs)
        s.step(120)
        got = [(*s.get_state()[:3], s.props())]
        s.close()
        b = Batch(1 << 33, 16, 32)
        slots = [b.admit(q.pos, q.vel, q.box, 90 + k, shell=q.shell,
                         precision="fp64" if k % 3 == 2 else "fp32")
                 for k, q in enumerate(systems)]
        for _ in range(4):
            b.run()
        assert sorted(b.poll()) == sorted(slots)
        got += [(*b.get_state(s)[:2], np.zeros(0), b.props(s)) for s in slots]
        b.close()
        out.append(got)
    for x, y in zip(*out):
        assert all(np.array_equal(p, q) for p, q in zip(x[:3], y[:3])) and x[3] == y[3]


@pytest.mark.parametrize("places", [1, 3])
def test_error_in_a_partial_run(places, monkeypatch):
    from paper_0911_5631_amd import _lib as L
    from paper_0911_5631_amd.md import System
    pos, box = I.fcc_lattice(9, 0.8)
    vel = I.random_velocities(len(pos), 5.0, 5)
    out = []
    for lim in (0, places):
        _limit(monkeypatch, lim)
        s = System(pos, vel, box, shell=0.4, dt=0.015)
        s.step(200)
        p = L.md_props_t()
        out.append((L.lib().md_props(s._h, C.byref(p)), p.step, p.n_rebuilds))
        s.close()
    assert out[0] == out[1] and out[0][0] in (-6, -7) and 0 < out[0][1] < 200


def test_systems_and_a_batch_at_once():
    """From three threads on streams of their own, more tiles than the chip
    holds: whichever launches find room, every result is that of a run alone."""
    import threading

    import torch
    from paper_0911_5631_amd.md import Batch, System
    big = [_fluid(40, 7), _fluid(36, 8)]                       # 1 000 and 729 tiles
    small = I.replica_batch(n_replicas=24, k_lo=6, k_hi=20, steps=0, seed=3)

    def system(start, stream):
        s = System(*start, shell=0.4, stream=stream)
        for n in (150, 150):
            s.step(n)
        out = (*s.get_state(), s.props())
        s.close()
        return [out]

    def batch(stream):
        b = Batch(1 << 33, 24, 64, stream=stream)
        slots = [b.admit(q.pos, q.vel, q.box, 300, shell=q.shell) for q in small]
        for _ in range(5):
            b.run()
        b.poll()
        out = [(*b.get_state(s), b.props(s)) for s in slots]
        b.close()
        return out

    jobs = [lambda st: system(big[0], st), lambda st: system(big[1], st), batch]
    alone = [job(torch.cuda.Stream()) for job in jobs]
    got = [None] * 3

    def work(k):
        torch.cuda.set_device(0)
        got[k] = jobs[k](torch.cuda.Stream())

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, g in zip(alone, got):
        for x, y in zip(a, g):
            assert all(np.array_equal(p, q) for p, q in zip(x[:-2], y[:-2])) and x[-2:] == y[-2:]
