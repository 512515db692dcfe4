"""Several contexts that sweep at the same time on one device.

Workgroups of a cluster launch wait for each other, so no two launches that do
not fit side by side may be in flight, nor a launch chain beside one: runs that
meet go in turn, or take the launch chain where that is the faster way to
share.  No launch is called off, and the chains are the same as alone.
"""
import ctypes as C
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import config1, oracle_trajectory  # noqa: E402


def runs(ctx):
    v = (C.c_uint64 * 4)()
    assert islf.lib().islf_testing_runs(ctx._h, v) == islf.OK
    return dict(zip(("cluster", "chain", "aborts", "apart"), v))


def film(shape, r=0, **over):
    return config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], replica=r, **over)


def context(p, fmt=islf.BITPACK, **kw):
    return islf.Context([islf.Replica(**q) for q in p], spin_format=fmt, obs_capacity=64, **kw)


BIG = (88, 504, 504)     # its shares take most CUs; about 16 us a sweep


def test_clusters_that_meet_go_in_turn():
    # int8: the resident form in turn beats two chains
    with context([film(BIG)], islf.INT8) as a, context([film(BIG, 1)], islf.INT8) as b:
        a.sweep(3000)
        b.sweep(20)
        a.sweep(20)
        b.sweep(20)
        assert b.sweep_count(0) == 40 and a.sweep_count(0) == 3020
        for c in (a, b):
            assert runs(c) == dict(cluster=2, chain=0, aborts=0, apart=0)


def test_single_chains_that_meet_share_the_device():
    # one bit-packed film each: two chains side by side are faster than the resident form in turn
    with context([film(BIG)]) as a, context([film(BIG, 1)]) as b:
        a.sweep(20)
        a.sweep_count(0)
        b.sweep(20)            # one after the other: nothing meets
        b.sweep_count(0)
        assert runs(a)["cluster"] == runs(b)["cluster"] == 1 and runs(b)["chain"] == 0
        a.sweep(3000)          # 50 ms of clusters in flight
        b.sweep(20)
        ra, rb = runs(a), runs(b)
        assert ra["cluster"] == 2 and rb["cluster"] == 1 and rb["chain"] == 1 and ra["apart"] > 0 and rb["apart"] > 0
        assert b.sweep_count(0) == 40 and a.sweep_count(0) == 3020   # (b's run came behind a's)
        for k in range(rb["apart"]):
            b.sweep(1)
        b.sweep(20)
        assert runs(b)["cluster"] == 2 and runs(b)["apart"] == 0
        assert runs(a)["aborts"] == runs(b)["aborts"] == 0


def test_a_new_context_comes_behind_the_clusters_of_one_that_was_alone():
    with context([film(BIG)], islf.INT8) as a:
        a.sweep(2000)
        with context([film(BIG, 1)], islf.INT8) as b:
            b.sweep(500)
            a.sweep(20)
            b.sweep(20)
            assert a.sweep_count(0) == 2020 and b.sweep_count(0) == 520
            for c in (a, b):
                assert runs(c) == dict(cluster=2, chain=0, aborts=0, apart=0)


@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_meeting_a_stream_that_its_caller_captures(mode):
    # no event can be recorded there: the run waits on the host, and the caller's graph is what it recorded
    x = torch.zeros(64, device="cuda")
    with context([film(BIG)], islf.INT8) as a, context([film(BIG, 1)], islf.INT8) as b:
        b.sweep(20)
        a.sweep(20)
        b.sweep_count(0)
        a.sweep_count(0)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        a.sweep(1500)
        with torch.cuda.stream(a.stream):
            g.capture_begin(capture_error_mode=mode)
            x.add_(1.0)
            b.sweep(20)
            x.add_(1.0)
            g.capture_end()
        for k in range(3):
            g.replay()
            b.sweep(20)
        torch.cuda.synchronize()
        assert (x == 6.0).all()
        assert a.sweep_count(0) == 1520 and b.sweep_count(0) == 100
        assert runs(a) == dict(cluster=2, chain=0, aborts=0, apart=0)
        assert runs(b) == dict(cluster=5, chain=0, aborts=0, apart=0)
        got = b.measure(0, 40, 60), b.get_spins(0)
    with context([film(BIG, 1)], islf.INT8) as c:
        c.set_groups(1)
        c.sweep(100)
        assert np.array_equal(got[0], c.measure(0, 40, 60)) and np.array_equal(got[1], c.get_spins(0))


def test_clusters_meet_a_chain():
    with context([film(BIG)]) as a, context([film(BIG, 1)]) as b:
        b.set_groups(1)        # b's runs are chains
        b.sweep(1000)
        a.sweep(20)
        assert runs(a)["cluster"] == 0 and runs(a)["chain"] == 1
        a.sweep_count(0)
        # a chain from before there was another context: in flight until its context is read
        b.sweep_count(0)
    with context([film(BIG)]) as b:
        b.set_groups(1)
        b.sweep(10)
        with context([film(BIG, 1)]) as a:
            a.sweep(20)
            assert runs(a)["cluster"] == 0
            b.sweep_count(0)
            a.sweep_count(0)


def test_small_clusters_go_side_by_side():
    shape = (24, 130, 140)
    with context([film(shape)]) as a, context([film(shape, 1)]) as b:
        a.sweep(5000)
        b.sweep(50)
        assert runs(a)["cluster"] == runs(b)["cluster"] == 1
        assert runs(a)["apart"] == runs(b)["apart"] == 0
        b.sweep_count(0)
        a.sweep_count(0)
        assert runs(a)["aborts"] == runs(b)["aborts"] == 0


@pytest.mark.parametrize("mode", [islf.EXEC_PLAIN, islf.EXEC_BATCHED, islf.EXEC_PERSISTENT])
def test_replays_that_meet(mode):
    # a graph of cluster launches is replayed as a chain beside another context's chain, and in turn with its clusters
    shape = (60, 120, 120)
    ps = [film(shape, r) for r in range(2)]
    with context([film(BIG, 8)]) as other, context([film(BIG, 9)], islf.INT8) as big, \
            context(ps, islf.INT8, exec_mode=mode) as a:
        a.capture(6)
        other.set_groups(1)
        other.sweep(2000)
        a.replay(2)
        a.sweep(3)
        assert runs(a)["cluster"] == 0 and runs(a)["chain"] == 2
        other.sweep_count(0)
        a.sweep_count(0)
        big.sweep(1500)
        a.replay(2)
        a.sweep(3)
        in_turn = mode != islf.EXEC_PLAIN     # (plain runs leave the device idle between launches)
        assert runs(a)["cluster"] == (2 if in_turn else 0), runs(a)
        big.sweep_count(0)
        for i in range(2):
            _, rec, s = oracle_trajectory(ps[i], 30)
            assert np.array_equal(a.measure(i, 0, 30), rec) and np.array_equal(a.get_spins(i), s)
        assert all(runs(c)["aborts"] == 0 for c in (other, big, a))


def test_runs_that_joined_a_chain_do_not_keep_others_on_it():
    with context([film(BIG)], islf.INT8) as a, context([film(BIG, 1)], islf.INT8) as b:
        assert islf.lib().islf_testing_abort_resident(a._h) == islf.OK
        a.sweep(10)                    # called off: a keeps to the chain for 256 runs
        a.sweep_count(0)
        for _ in range(255):
            a.sweep(10)
        assert runs(a) == dict(cluster=1, chain=255, aborts=1, apart=1)
        a.sweep(300)                   # the last of them, 7 ms
        b.sweep(1500)                  # joins it: 36 ms on the chain
        assert runs(b) == dict(cluster=0, chain=1, aborts=0, apart=0)
        a.sweep(20)                    # behind b's run, resident again
        assert runs(a) == dict(cluster=2, chain=256, aborts=1, apart=0)
        n = a.sweep_count(0)
        assert n == 2880 and b.sweep_count(0) == 1500
        b.sweep(20)
        assert runs(b)["cluster"] == 1
        got = a.measure(0, n - 60, 60), a.get_spins(0)
    with context([film(BIG)], islf.INT8) as c:
        c.set_groups(1)
        c.sweep(n)
        assert np.array_equal(got[0], c.measure(0, n - 60, 60)) and np.array_equal(got[1], c.get_spins(0))


def test_a_called_off_launch_keeps_to_the_chain():
    with context([film((24, 130, 140))]) as a:
        a.sweep(6)
        assert islf.lib().islf_testing_abort_resident(a._h) == islf.OK
        a.sweep(6)
        a.sweep_count(0)
        a.sweep(6)
        r = runs(a)
        assert r["aborts"] == 1 and r["cluster"] == 2 and r["chain"] == 1
        _, rec, s = oracle_trajectory(film((24, 130, 140)), 18)
        assert np.array_equal(a.measure(0, 0, 18), rec) and np.array_equal(a.get_spins(0), s)


@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
def test_four_contexts_on_threads(fmt):
    shape, turns, k = (50, 200, 200), 12, 10
    ps = [[film(shape, 2 * c + r) for r in range(2)] for c in range(4)]
    want = []
    for p in ps:
        with context(p, fmt) as ctx:
            ctx.set_groups(1)      # alone, on the chain
            ctx.sweep(turns * k)
            want.append([(ctx.measure(r, turns * k - 60, 60), ctx.get_spins(r)) for r in range(2)])
    ctxs = [context(p, fmt) for p in ps]
    got = [None] * 4
    start = threading.Barrier(4)

    def work(i):
        start.wait()
        for t in range(turns):
            ctxs[i].sweep(k)
            if t % 4 == i:
                ctxs[i].sweep_count(0)
        got[i] = [(ctxs[i].measure(r, turns * k - 60, 60), ctxs[i].get_spins(r)) for r in range(2)]

    th = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for i in range(4):
        assert runs(ctxs[i])["aborts"] == 0
        for (rec, s), (rec0, s0) in zip(got[i], want[i]):
            assert np.array_equal(rec, rec0) and np.array_equal(s, s0), i
    for c in ctxs:
        c.close()


def test_beside_other_work_on_the_device():
    # work that the library does not see: whichever way a launch goes, the chain is the same
    p = film((24, 130, 140), 3)
    x = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    with context([p]) as a:
        a.sweep(2)
        a.sweep_count(0)
        with torch.cuda.stream(side):
            for _ in range(60):
                y = x @ x
        for _ in range(10):
            a.sweep(2)
        got = a.measure(0, 0, 22), a.get_spins(0)
        side.synchronize()
        del y
    _, rec, s = oracle_trajectory(p, 22)
    assert np.array_equal(got[0], rec) and np.array_equal(got[1], s)
