"""Device memory that the resident form holds beside the replicas."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import config1, oracle_trajectory  # noqa: E402


@pytest.mark.parametrize("mode", [islf.EXEC_PLAIN, islf.EXEC_BATCHED])
@pytest.mark.parametrize("shape,n", [((12, 24, 24), 2), ((24, 130, 140), 2)])
def test_longer_runs_take_no_more_memory(shape, n, mode):
    # a plan's memory is had when it is built: runs of any length after that, and between replays of a
    # captured graph, allocate nothing
    ps = [config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], replica=r) for r in range(n)]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=islf.BITPACK, obs_capacity=64,
                      exec_mode=mode) as ctx:
        ctx.sweep(8)
        held, calls, done = ctx.device_bytes(), ctx._alloc.calls, 8
        for k in (9, 10, 11, 12, 13, 300):
            ctx.sweep(k)
            done += k
            assert ctx.device_bytes() == held and ctx._alloc.calls == calls, k
        ctx.capture(20)
        ctx.sweep(30)
        ctx.replay(2)
        assert ctx.device_bytes() == held and ctx._alloc.calls == calls
        done += 70
        for r, p in enumerate(ps):
            _, rec, s = oracle_trajectory(p, done)
            assert np.array_equal(ctx.measure(r, done - 60, 60), rec[-60:])
            assert np.array_equal(ctx.get_spins(r), s)


@pytest.mark.parametrize("mode", [islf.EXEC_PLAIN, islf.EXEC_BATCHED])
def test_plans_are_bounded(mode):
    # plans of the plain form, one a film: beyond 32 MiB the films go to the launch chain, with the same results
    n, shape = 18, (100, 60, 1200)
    ps = [config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], replica=r, init=islf.INIT_UP, beta=0.3) for r in range(n)]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=islf.BITPACK, obs_capacity=8,
                      exec_mode=mode) as ctx:
        total, replicas = ctx.device_bytes()
        ctx.sweep(6)
        held, _ = ctx.device_bytes()
        assert held - total <= 33 << 20    # (and the chain's own plan)
        ctx.sweep_count(0)
        got = [(ctx.measure(r, 0, 6), ctx.get_spins(r)) for r in (0, n - 1)]
    for (rec, s), r in zip(got, (0, n - 1)):
        _, want, sw = oracle_trajectory(ps[r], 6)
        assert np.array_equal(rec, want) and np.array_equal(s, sw)
