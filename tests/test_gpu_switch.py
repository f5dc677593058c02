"""A batch that changes, while its systems are in mid-run, between taking many
steps per launch and taking each step in launches of its own: by its launch
configuration, and because a system of more tiles than the chip holds at once
is admitted and released.  Every system equals its run alone bit for bit, late
binnings counted alike, whether its next positions were binned ahead by the
run before or not."""
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


def _jump():
    """The maximum speed jumps in one step, so a rebuild is not foreseen."""
    pos, L = I.sc_lattice(12, 0.5)
    rng = np.random.Generator(np.random.PCG64(61))
    vel = rng.uniform(-0.005, 0.005, pos.shape)
    vel -= vel.mean(0)
    d = pos[1] - pos[0]
    d -= L * np.round(d / L)
    pos[0] = pos[1] - d / np.linalg.norm(d) * 0.9
    return pos, vel, L


def _systems(steps):
    kinds = [dict(shell=0.4), dict(shell=0.3, precision="fp64"), dict(shell=0.0),
             dict(shell=0.4, reorder_interval=30), dict(shell=0.4, reorder=False),
             dict(shell=0.2, nebr_cap=8), dict(shell=0.0, precision="fp64")]
    out = [(*_fluid(5 + k % 4, 10 * k), steps + 7 * k, kinds[k % len(kinds)]) for k in range(21)]
    return out + [(*_jump(), steps, dict(shell=0.004))]


def _alone(pos, vel, L, steps, prm):
    from paper_0911_5631_amd.md import System
    s = System(pos, vel, L, **prm)
    s.step(steps)
    p, v, _, n = s.get_state()
    pr = s.props()
    s.close()
    return p, v, n, pr


def _check(got, sys_):
    p, v, n, pr = _alone(*sys_)
    assert got[2] == n
    assert np.array_equal(got[0], p) and np.array_equal(got[1], v)
    assert got[3] == pr


@pytest.mark.parametrize("trace", [False, True])
@pytest.mark.parametrize("spr", [1, 5, 16])
def test_batch_switched_between_runs_equals_solo(spr, trace):
    from paper_0911_5631_amd.md import Batch
    steps = 90
    systems = _systems(steps)
    b = Batch(1 << 32, 32, spr)
    slot = [b.admit(p, v, L, n, trace=trace, **prm) for p, v, L, n, prm in systems]
    left, out, runs = set(slot), {}, 0
    while left:
        # two runs each way, then one each way, ...
        b.configure(steps_per_run=spr, sort_split=1 if runs % 5 in (1, 3, 4) else 0)
        b.run()
        if runs % 3 == 0:
            b.get_state(slot[runs % len(slot)])
        for s in b.poll():
            if s in left:
                out[s] = (*b.get_state(s), b.props(s))
                left.discard(s)
        runs += 1
        assert runs < 1000
    b.close()
    for k, sys_ in enumerate(systems):
        _check(out[slot[k]], sys_)
    assert out[slot[-1]][3]["n_late_bins"] >= 1


def test_large_system_admitted_and_released_in_mid_run():
    from paper_0911_5631_amd.md import Batch
    systems = _systems(200)
    big = (*_fluid(41, 99), 48, dict(shell=0.4))       # 275 684 atoms: 1 077 tiles
    b = Batch(1 << 33, 32, 16)
    slot = [b.admit(p, v, L, n, **prm) for p, v, L, n, prm in systems]
    left, out, runs, sbig, done_big = set(slot), {}, 0, None, None
    while left:
        if runs == 3:
            p, v, L, n, prm = big
            sbig = b.admit(p, v, L, n, **prm)
        b.run()
        b.get_state(slot[runs % len(slot)])
        for s in b.poll():
            if s in left:
                out[s] = (*b.get_state(s), b.props(s))
                left.discard(s)
            elif s == sbig and done_big is None:
                done_big = (*b.get_state(s), b.props(s))
                b.release(s)
        runs += 1
        assert runs < 100
    b.close()
    assert done_big is not None and runs > 8
    for k, sys_ in enumerate(systems):
        _check(out[slot[k]], sys_)
    _check(done_big, big)
