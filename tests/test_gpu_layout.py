"""Spins in and out of the internal formats, and their observables, exactly.

Rows of every alignment of the host layout (Lz = 16k, 4k, 2k), rows that end
inside an int8 column and inside a bit-packed word, one plane, two rows, and a
film of more lanes than a launch: the spins read back are those set, and the
recomputed (B, M, M1, Mn) are those of an int64 sum over the lattice.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import SEED, config1  # noqa: E402

PBC, APBC, GAPBC = 0, 1, 2
SHAPES = [(1, 2, 2), (3, 2, 4), (2, 5, 6), (4, 3, 14), (3, 5, 16), (2, 7, 18), (5, 4, 30), (3, 3, 32), (2, 3, 34),
          (4, 6, 62), (3, 2, 64), (2, 5, 66), (1, 9, 128), (3, 4, 130), (2, 3, 200), (6, 50, 1000)]


def sums(s, ybc):
    s = s.astype(np.int64)
    up = np.roll(s, -1, axis=1)
    if ybc != PBC:
        first = s[::-1, 0] if ybc == GAPBC else s[:, 0]
        up[:, -1] = -first
    B = (s * np.roll(s, -1, axis=2)).sum() + (s * up).sum() + (s[:-1] * s[1:]).sum()
    return int(B), int(s.sum()), int(s[0].sum()), int(s[-1].sum())


@pytest.mark.parametrize("ybc", [PBC, APBC, GAPBC])
@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
def test_spins_and_observables_round_trip(fmt, ybc):
    rng = np.random.default_rng(SEED + 31)
    reps = [islf.Replica(**config1(Lx=x, Ly=y, Lz=z, seed=SEED, replica=i, ybc=ybc)) for i, (x, y, z) in
            enumerate(SHAPES)]
    want = [(2 * rng.integers(0, 2, size=s) - 1).astype(np.int8) for s in SHAPES]
    with islf.Context(reps, spin_format=fmt, obs_capacity=4) as ctx:
        for r, s in enumerate(want):
            ctx.set_spins(r, s)
        for r, s in enumerate(want):
            assert np.array_equal(np.asarray(ctx.get_spins(r)).reshape(s.shape), s), SHAPES[r]
            assert tuple(ctx.recompute(r)) == sums(s, ybc), SHAPES[r]
        # the running observables start from the same sums: one sweep's record is the lattice's own
        ctx.sweep(1)
        for r in range(len(SHAPES)):
            assert tuple(ctx.measure(r, 0, 1)[0]) == tuple(ctx.recompute(r)), SHAPES[r]


@pytest.mark.parametrize("shape", [(2, 8, 4096), (2, 8, 4098), (37, 251, 226), (3, 2, 700002), (44, 252, 504)])
@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
def test_spins_in_windows(fmt, shape):
    """64 KiB (one piece), just over it, and several windows with rows across their ends, with and without helpers."""
    rng = np.random.default_rng(SEED + 32)
    a, b = [(2 * rng.integers(0, 2, size=shape) - 1).astype(np.int8) for _ in range(2)]
    p = config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], seed=SEED, replica=0, ybc=GAPBC)
    with islf.Context([islf.Replica(**p)], spin_format=fmt, obs_capacity=4) as ctx:
        ctx.set_spins(0, a)
        b[-1, -1, -1] = 0
        with pytest.raises(islf.IslfError) as e:   # refused whole: the last byte is no spin
            ctx.set_spins(0, b)
        assert e.value.status == islf.EINVAL
        assert np.array_equal(ctx.get_spins(0).reshape(shape), a)
        assert tuple(ctx.recompute(0)) == sums(a, GAPBC)
        b[-1, -1, -1] = 1
        ctx.set_spins(0, b)
        assert np.array_equal(ctx.get_spins(0).reshape(shape), b)
        assert tuple(ctx.recompute(0)) == sums(b, GAPBC)


@pytest.mark.parametrize("count", [2048, 2049, 8192, 8193])
def test_records_at_the_edges_of_the_result_buffer(count):
    """Records and energies around the sizes at which they come in one piece, from a ring that has wrapped."""
    p = config1(Lx=2, Ly=4, Lz=4, seed=SEED, replica=0)
    cap, n = 9000, 13000
    with islf.Context([islf.Replica(**p)], spin_format=islf.INT8, obs_capacity=cap) as ctx:
        ctx.sweep(n)
        first = n - count - 3
        one = np.concatenate([ctx.measure(0, k, min(1000, n - k)) for k in range(n - cap, n, 1000)])
        assert np.array_equal(ctx.measure(0, first, count), one[first - (n - cap):][:count])
        E = ctx.energy(0, first, count)
        r = one[first - (n - cap):][:count].astype(np.float64)
        e = -p["J"] * r[:, 0]
        for k, h in enumerate(("H", "h1", "hn")):
            e = e - p[h] * r[:, k + 1]
        assert np.array_equal(E, e)
