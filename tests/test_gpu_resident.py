"""The resident form (spins in LDS for a whole launch) against the oracle.

Runs of several sweeps in the default configuration take it: small films one
four-site group per lane, larger ones word by word, in one workgroup or cut
along y into shares that exchange edge rows.  Records and spins must equal the
oracle's exactly.
"""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import oracle as O  # noqa: E402
from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import config1, oracle_trajectory  # noqa: E402


def check(ctx, ps, n, first=0):
    recs = [ctx.measure(i, first, n - first) for i in range(len(ps))]
    spins = [ctx.get_spins(i) for i in range(len(ps))]
    for i, p in enumerate(ps):
        _, o_rec, o_s = oracle_trajectory(p, n)
        assert np.array_equal(recs[i], np.asarray(o_rec)[first:]), i
        assert np.array_equal(spins[i], o_s), i


SHAPES = [
    (1, 2, 2), (2, 2, 4), (1, 3, 64), (3, 4, 66), (5, 7, 62),            # tiny: one row beside the seam, one layer
    (12, 24, 24), (8, 12, 12), (16, 16, 64), (7, 43, 58),                # one lane per group, up to the last lane
    (30, 40, 64), (30, 41, 62), (9, 60, 128), (13, 33, 130),             # words, one workgroup
    (20, 64, 76), (16, 150, 130), (40, 120, 120), (21, 333, 66),         # shares along y
    (61, 50, 70), (80, 200, 160), (37, 24, 190), (90, 9, 250),           # and along x
]


@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_and_boundaries(fmt, shape):
    ps = [config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], ybc=ybc, beta=b, H=H, replica=i)
          for i, (ybc, b, H) in enumerate(((O.GAPBC, 1 / 3, 0.0), (O.APBC, 0.6, 0.3), (O.PBC, 3.0, 0.0)))]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=fmt, obs_capacity=32) as ctx:
        ctx.sweep(3)
        ctx.sweep(6)
        check(ctx, ps, 9)


@pytest.mark.parametrize("mode", [islf.EXEC_PLAIN, islf.EXEC_BATCHED, islf.EXEC_PERSISTENT])
@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
def test_mixed_batch_in_every_form(mode, fmt):
    # clusters and single-workgroup films in one launch, graph replays between eager runs
    ps = [config1(Lx=24, Ly=130, Lz=140, replica=0), config1(replica=1), config1(Lx=6, Ly=9, Lz=30, beta=4.0, replica=2),
          config1(Lx=31, Ly=57, Lz=64, h1=0.2, hn=0.4, replica=3), config1(Lx=1, Ly=80, Lz=130, replica=4)]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=fmt, obs_capacity=64, exec_mode=mode) as ctx:
        ctx.capture(4)
        ctx.replay(2)
        ctx.sweep(5)
        ctx.replay(1)
        ctx.sweep(12)
        ctx.replay(1)
        check(ctx, ps, 33)


def test_more_sweeps_than_a_launch_and_the_ring():
    p = config1(Lx=4, Ly=6, Lz=10)
    n = 600
    with islf.Context([islf.Replica(**p)], spin_format=islf.BITPACK, obs_capacity=100) as ctx:
        ctx.sweep(n)
        check(ctx, [p], n, first=n - 99)


def test_launch_chain_and_resident_runs_alternate():
    ps = [config1(Lx=18, Ly=70, Lz=96, replica=i) for i in range(3)]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=islf.INT8, obs_capacity=64) as ctx:
        ctx.sweep(5)
        ctx.set_groups(2)          # a chosen configuration asks for the launch chain
        ctx.sweep(4)
        ctx.set_groups(0)
        ctx.sweep(6)
        slot = ctx.add(islf.Replica(**config1(Lx=5, Ly=8, Lz=12, replica=9)))
        ctx.sweep(7)
        check(ctx, ps, 22)
        _, rec, s = oracle_trajectory(config1(Lx=5, Ly=8, Lz=12, replica=9), 7)
        assert np.array_equal(ctx.measure(slot, 0, 7), rec) and np.array_equal(ctx.get_spins(slot), s)


@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
def test_aborted_launch_is_swept_by_the_closing_kernel(fmt):
    # the state word is set from the host, so that the launch finds itself
    # aborted: its clusters leave at once and the closing kernel sweeps them
    ps = [config1(Lx=24, Ly=130, Lz=140, beta=0.4, replica=0), config1(replica=1)]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=fmt, obs_capacity=32) as ctx:
        ctx.sweep(6)
        assert islf.lib().islf_testing_abort_resident(ctx._h) == islf.OK
        ctx.sweep(6)
        ctx.sweep(6)
        check(ctx, ps, 18)


def test_contexts_on_two_threads():
    ps = [config1(Lx=40, Ly=120, Lz=120, seed=100 + k, replica=k) for k in range(2)]
    out = [None, None]

    def work(k):
        with islf.Context([islf.Replica(**ps[k])], spin_format=islf.BITPACK, obs_capacity=64) as ctx:
            for _ in range(5):
                ctx.sweep(8)
            out[k] = (ctx.measure(0, 0, 40), ctx.get_spins(0))

    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for k in range(2):
        _, rec, s = oracle_trajectory(ps[k], 40)
        assert np.array_equal(out[k][0], rec) and np.array_equal(out[k][1], s), k


@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
@pytest.mark.parametrize("shape", [(25, 76, 76), (24, 40, 94), (30, 60, 126), (14, 90, 42), (60, 40, 300),
                                   (120, 12, 200)])
def test_few_words_a_stage(fmt, shape):
    # four lanes to a word: partial words of 2 to 8 groups, rows without a whole word, cuts along y and along x;
    # the four-site table, a bulk field, and moves that are never accepted
    ps = [config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], ybc=ybc, beta=b, H=H, replica=i)
          for i, (ybc, b, H) in enumerate(((O.GAPBC, 1 / 3, 0.0), (O.APBC, 0.6, 0.3), (O.PBC, 40.0, 0.1)))]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=fmt, obs_capacity=32) as ctx:
        ctx.sweep(2)
        ctx.sweep(5)
        check(ctx, ps, 7)
