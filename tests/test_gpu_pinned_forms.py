"""Every execution form against the oracle, each chosen so that it is the one that runs.

In the default configuration most batches take the resident form whatever the
execution form, so the launch chain (in groups, and one lattice per launch) and
the persistent kernel with either barrier are asked for here, and the library's
own count of runs says that they ran.
"""
import ctypes as C
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import oracle as O  # noqa: E402
from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import SEED, config1, oracle_trajectory, parallel_map, random_shape  # noqa: E402

FORMATS = [islf.INT8, islf.BITPACK]
FORMS = {
    "plain": (islf.EXEC_PLAIN, lambda c: c.set_grid(c.get_grid())),
    "one chain": (islf.EXEC_BATCHED, lambda c: c.set_groups(1)),
    "three groups": (islf.EXEC_BATCHED, lambda c: c.set_groups(3)),
    "grid barriers": (islf.EXEC_PERSISTENT, lambda c: c.set_barriers(islf.BARRIER_GRID)),
    "team barriers": (islf.EXEC_PERSISTENT, lambda c: c.set_barriers(islf.BARRIER_TEAM)),
    "resident": (islf.EXEC_BATCHED, lambda c: None),
    "resident persistent": (islf.EXEC_PERSISTENT, lambda c: None),
}


def chain_runs(ctx):
    v = (C.c_uint64 * 4)()
    assert islf.lib().islf_testing_runs(ctx._h, v) == islf.OK
    return v[1]


def context(ps, fmt, form, cap):
    mode, choose = FORMS[form]
    ctx = islf.Context([islf.Replica(**p) for p in ps], spin_format=fmt, obs_capacity=cap, exec_mode=mode)
    choose(ctx)
    return ctx


def films():
    ps = [config1(replica=0),
          config1(Lx=5, Ly=7, Lz=18, ybc=O.PBC, beta=0.25, h1=0.3, hn=-0.7, replica=1),
          config1(Lx=1, Ly=2, Lz=2, beta=0.4, replica=2),
          config1(Lx=3, Ly=9, Lz=66, ybc=O.APBC, beta=0.5, H=0.05, seed=7, replica=3),
          config1(Lx=4, Ly=6, Lz=130, beta=float("inf"), h1=0.0, hn=0.0, replica=4)]
    rng = np.random.default_rng(SEED + 5)
    for k in range(12):
        Lx, Ly, Lz = random_shape(rng)
        ps.append(dict(Lx=Lx, Ly=Ly, Lz=Lz, ybc=k % 3, J=float(rng.choice([1.0, 0.7])),
                       beta=float(rng.choice([0.0, 0.1, 0.25, 1 / 3, 0.6, 2.0])), H=float(rng.choice([0.0, 0.1])),
                       h1=float(rng.uniform(-1, 1)), hn=float(rng.uniform(-1, 1)), seed=int(rng.integers(0, 2**63)),
                       replica=10 + k, init=k % 3))
    return ps


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("fmt", FORMATS)
def test_small_films(fmt, form):
    ps, n = films(), 24
    with context(ps, fmt, form, 32) as ctx:
        ctx.sweep(10)
        ctx.capture(7)
        ctx.replay(2)
        assert (chain_runs(ctx) == 0) == form.startswith("resident")
        recs = [ctx.measure(i, 0, n) for i in range(len(ps))]
        spins = [ctx.get_spins(i) for i in range(len(ps))]
    for i, (_, rec, s) in enumerate(parallel_map(lambda p: oracle_trajectory(p, n), ps)):
        assert np.array_equal(recs[i], rec) and np.array_equal(spins[i], s), ps[i]


@pytest.mark.parametrize("form", ["grid barriers", "team barriers", "resident persistent", "resident"])
@pytest.mark.parametrize("fmt", FORMATS)
def test_failed_launch(fmt, form):
    # the error word is raised from the host before the launch: with barriers every block stops at its first one
    # and leaves; the resident forms (films cut into shares) leave at once or run on, and are marked failed alike
    ps = [config1(Lx=24, Ly=130, Lz=140, replica=0), config1(Lx=6, Ly=10, Lz=16, beta=0.4, seed=77, replica=1)]
    with context(ps, fmt, form, 64) as ctx:
        ctx.sweep(6)
        assert ctx.sweep_count(0) == 6
        assert (chain_runs(ctx) == 0) == form.startswith("resident")
        assert islf.lib().islf_testing_raise_barrier_error(ctx._h) == islf.OK
        ctx.sweep(6)
        with pytest.raises(islf.IslfError) as e:
            ctx.measure(0, 0, 3)
        assert e.value.status == islf.EDEVICE
        for call in (lambda: ctx.measure(0, 0, 3), lambda: ctx.get_spins(1), lambda: ctx.sweep(1),
                     lambda: ctx.means(0, 3), lambda: ctx.capture(2)):
            with pytest.raises(islf.IslfError) as e:
                call()
            assert e.value.status == islf.ESTATE
        rng = np.random.default_rng(5)
        starts = [rng.choice(np.array([-1, 1], dtype=np.int8), size=islf.Replica(**p).N) for p in ps]
        for i, s in enumerate(starts):
            ctx.set_spins(i, s)
        ctx.sweep(6)
        recs = [ctx.measure(i, 0, 6) for i in range(2)]
        spins = [ctx.get_spins(i) for i in range(2)]
    for i, p in enumerate(ps):
        _, rec, s = oracle_trajectory(p, 6, spins=starts[i])
        assert np.array_equal(recs[i], rec) and np.array_equal(spins[i], s), i


PAPER = [config1(Lx=160, Ly=480, Lz=600, beta=1.0 / T, h1=0.55, hn=-0.55, seed=SEED + i, replica=i)
         for i, T in enumerate((2.0, 3.0, 4.0))]


@pytest.fixture(scope="module")
def paper_oracle():
    """Six sweeps of each film, one thread per film, beside the GPU work."""
    out = [None] * len(PAPER)

    def work(i):
        out[i] = oracle_trajectory(PAPER[i], 6)

    th = [threading.Thread(target=work, args=(i,)) for i in range(len(PAPER))]
    for t in th:
        t.start()
    yield th, out


@pytest.fixture(scope="module")
def long_runs():
    """120 sweeps of the three films in every form and format: records and spins."""
    res = {}
    for fmt in FORMATS:
        for form in ("three groups", "grid barriers", "team barriers", "resident persistent"):
            with context(PAPER, fmt, form, 128) as ctx:
                ctx.sweep(6)
                six = [(ctx.measure(i, 0, 6), ctx.get_spins(i)) for i in range(3)]
                ctx.capture(38)
                ctx.replay(3)
                assert (chain_runs(ctx) == 0) == form.startswith("resident")
                last = [(ctx.measure(i, 0, 120), ctx.get_spins(i), ctx.recompute(i)) for i in range(3)]
            res[fmt, form] = six, last
    return res


def test_paper_films_over_six_sweeps(paper_oracle, long_runs):
    th, out = paper_oracle
    for t in th:
        t.join()
    for key, (six, _) in long_runs.items():
        for (rec, s), (_, orec, os) in zip(six, out):
            assert np.array_equal(rec, orec) and np.array_equal(s, os), key


def test_paper_films_agree_over_120_sweeps(long_runs):
    ref = long_runs[islf.BITPACK, "three groups"][1]
    for key, (_, last) in long_runs.items():
        for (rec, s, rc), (rec0, s0, _) in zip(last, ref):
            assert np.array_equal(rec, rec0) and np.array_equal(s, s0) and np.array_equal(rec[-1], rc), key
