"""A batch whose allocator refuses a table while a system is admitted: the
admission fails with MD_ERR_OOM, and the systems already there go on, equal to
their runs alone."""
from types import SimpleNamespace

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


# after the system's three blocks: atom tiles, cell tiles, seats
@pytest.mark.parametrize("refused", [4, 5, 6])
def test_admission_with_a_refused_table(refused):
    import torch
    from paper_0911_5631_amd._lib import MDError
    from paper_0911_5631_amd.md import Batch, System

    def start(edge, seed):
        pos, L = I.fcc_lattice(edge, 0.8)
        return I.jitter(pos, L, 0.06, seed), I.random_velocities(len(pos), 1.0, seed), L

    small, large = start(6, 3), start(16, 4)
    b = Batch(1 << 32, 8, 16)
    slot = b.admit(*small, 100, shell=0.4)
    b.run()
    count = [0]

    def alloc(nbytes, device, stream):
        count[0] += 1
        if count[0] >= refused:
            raise MemoryError
        return torch.cuda.caching_allocator_alloc(nbytes, device, stream)

    b._alloc._torch = SimpleNamespace(cuda=SimpleNamespace(
        caching_allocator_alloc=alloc,
        caching_allocator_delete=torch.cuda.caching_allocator_delete))
    with pytest.raises(MDError) as err:
        b.admit(*large, 50, shell=0.4)
    assert err.value.code == -3 and count[0] >= refused
    b.run()
    b._alloc._torch = torch
    other = b.admit(*large, 50, shell=0.4)
    done = {}
    for _ in range(20):
        b.run()
        for s in b.poll():
            done.setdefault(s, b.get_state(s))
    b.close()
    for s, (pos, vel, L), n in ((slot, small, 100), (other, large, 50)):
        ref = System(pos, vel, L, shell=0.4)
        ref.step(n)
        p, v, _, k = ref.get_state()
        ref.close()
        assert done[s][2] == k == n
        assert np.array_equal(done[s][0], p) and np.array_equal(done[s][1], v)
