"""The autotuner's choice between many steps per launch and launches of a step
on the CPU: a batch is offered both, a batch that names no candidates of its
own is tuned as before, and a system's candidates that come to one
configuration are timed once."""
from paper_0911_5631_amd import tune
from paper_0911_5631_amd.md import Batch


class Clock:
    t = 0.0

    def __call__(self):
        return self.t


class SimBatch:
    def __init__(self, clock, zero_ns):
        self.clock, self.zero_ns, self.done, self.config = clock, zero_ns, 0, None

    def configure(self, **c):
        self.config = c
        return dict(c)

    def run(self):
        k = self.config["steps_per_run"]
        ns = 0.1 if self.config["grid"] else self.zero_ns
        self.done += k
        self.clock.t += 20e-6 + 1e5 * k * ns * 1e-9

    def poll(self):
        return []

    def progress(self):
        return 100000 * self.done, 1, 10 ** 6 - self.done


def test_batches_are_offered_many_steps_per_launch():
    assert Batch.launch_candidates is tune.BATCH_CANDIDATES
    zero = [c for c in tune.BATCH_CANDIDATES
            if not (c["grid"] or c["sort_grid"] or c["sort_split"])]
    assert zero and set(map(str, tune.DEFAULT_CANDIDATES)) <= set(map(str, tune.BATCH_CANDIDATES))
    for zero_ns, want in ((0.05, True), (0.2, False)):
        clock = Clock()
        b = SimBatch(clock, zero_ns)
        b.launch_candidates = tune.BATCH_CANDIDATES
        best = tune.autotune(b, clock=clock)["best"]
        assert (best["grid"] == 0) == want and best["steps_per_run"] == 64
        assert b.config == {k: best[k] for k in tune.KNOBS}


def test_candidates_are_the_callers_or_the_default():
    clock = Clock()
    got = tune.autotune(SimBatch(clock, 0.05), clock=clock)
    assert len(got["trials"]) == len(tune.DEFAULT_CANDIDATES)
    mine = ({"steps_per_run": 8, "grid": 64},)
    b = SimBatch(clock, 0.05)
    b.launch_candidates = tune.BATCH_CANDIDATES
    assert len(tune.autotune(b, candidates=mine, clock=clock)["trials"]) == 1


def test_equal_configurations_of_a_system_are_timed_once():
    clock = Clock()

    class Sim:
        steps = []

        def configure(self, **c):
            self.c = dict(c)
            if not (c["grid"] or c["sort_grid"] or c["sort_split"]):
                self.c = dict.fromkeys(c, 0)
            return self.c

        def step(self, n):
            self.steps.append((tuple(self.c.values()), n))
            clock.t += n * (2e-5 if self.c["grid"] or self.c["sort_grid"] else 1e-5)

        def props(self):
            pass

    s = Sim()
    out = tune.autotune_system(s, 10000, steps=100, clock=clock)
    skipped = [t for t in out["trials"] if "skipped" in t]
    same = [c for c in tune.SINGLE_CANDIDATES
            if not (c["grid"] or c["sort_grid"] or c["sort_split"])]
    assert len(out["trials"]) == len(tune.SINGLE_CANDIDATES) and len(skipped) == len(same) - 1
    assert sum(n for c, n in s.steps if c == (0,) * 5) == 164
    assert out["best"]["grid"] == 0 and out["best"]["sort_grid"] == 0
