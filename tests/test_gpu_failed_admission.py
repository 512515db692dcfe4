"""An admission that runs out of device memory leaves the batch as it was.

The context's allocator refuses one request of islf_batch_add (the first, the
second, ...): the call reports ENOMEM, and the replicas that were there go on
exactly, read back by every means, through sweeps, a retirement and a later
admission that succeeds.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import oracle as O  # noqa: E402
from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import config1, oracle_trajectory  # noqa: E402

N = 16   # the tables' first size: the next admission grows them and the live list


class Refusing(islf._TorchAllocator):
    def __init__(self, *a):
        super().__init__(*a)
        self.refuse = 0   # requests until one is refused (0: none)
        give = self.alloc

        def alloc(nbytes, user):
            self.refuse -= 1
            return None if self.refuse == 0 else give(nbytes, user)

        self.alloc = islf._ALLOC_FN(alloc)


def film(r):
    return config1(Lx=2 + r % 4, Ly=6 + r % 5, Lz=8 + 2 * (r % 3), beta=0.2 + 0.02 * r, replica=r)


def check(ctx, n, skip=(), means=True):
    m = ctx.means(0, n) if means else None
    for r in range(N):
        if r in skip:
            continue
        _, rec, s = oracle_trajectory(film(r), n)
        om = [O.mean(rec, k) for k in range(4)]
        assert np.array_equal(ctx.replica_means(r, 0, n)[1:], om), r
        assert m is None or np.array_equal(m[r, 1:], om), r
        assert np.array_equal(ctx.measure(r, 0, n), rec) and np.array_equal(ctx.get_spins(r), s), r


@pytest.mark.parametrize("mode", [islf.EXEC_PLAIN, islf.EXEC_BATCHED])
@pytest.mark.parametrize("nth", [1, 2, 3, 4])   # the tables' growth; the replica's block; the live list
def test_batch_goes_on_after_a_refused_admission(monkeypatch, nth, mode):
    monkeypatch.setattr(islf, "_TorchAllocator", Refusing)
    with islf.Context([islf.Replica(**film(r)) for r in range(N)], spin_format=islf.BITPACK, obs_capacity=32,
                      exec_mode=mode) as ctx:
        ctx.sweep(4)
        ctx._alloc.refuse = nth
        with pytest.raises(islf.IslfError) as e:
            ctx.add(islf.Replica(**film(N)))
        assert e.value.status == islf.ENOMEM
        ctx._alloc.refuse = 0
        check(ctx, 4)
        ctx.sweep(3)
        check(ctx, 7)
        ctx.retire(5)
        ctx.sweep(2)
        check(ctx, 9, skip=(5,))
        more = [ctx.add(islf.Replica(**film(N + k))) for k in range(2)]
        ctx.sweep(3)
        check(ctx, 12, skip=(5,), means=False)   # (the new ones have 3 records)
        for k, slot in enumerate(more):
            _, rec, s = oracle_trajectory(film(N + k), 3)
            assert np.array_equal(ctx.measure(slot, 0, 3), rec) and np.array_equal(ctx.get_spins(slot), s)
