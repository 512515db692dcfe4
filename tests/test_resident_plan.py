"""Plans of the resident form, checked on the host (no GPU).

Every row of every plane of every film is updated by one share, in one of its
row sets; every chunk of a set is updated once in each of its phases, row 0
after the other rows; a share's edge words have a mailbox of their own in the
share that holds the row or plane beside them.
"""
import ctypes as C
import os

import numpy as np
import pytest

from paper_1411_5588_amd import islf

HAS_Y, HAS_OUTER, HAS_INNER = 1, 2, 4
WORDS, GROUPS, FINE = 0, 1, 2


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(islf.LIB_PATH):
        from paper_1411_5588_amd import build
        build.build()


def plan(shapes, fmt, cus=256):
    descs = (islf.ReplicaDesc * len(shapes))()
    for d, (x, y, z) in zip(descs, shapes):
        d.Lx, d.Ly, d.Lz, d.ybc, d.J, d.beta = x, y, z, 2, 1.0, 0.3
    n = C.c_int64()
    call = islf.lib().islf_testing_resident_plan
    assert call(C.cast(descs, C.c_void_p), len(shapes), fmt, cus, None, 0, C.cast(C.byref(n), C.c_void_p)) == islf.OK
    if n.value == 0:
        return None
    v = np.zeros(n.value, dtype=np.int32)
    assert call(C.cast(descs, C.c_void_p), len(shapes), fmt, cus, v.ctypes.data_as(C.c_void_p), n.value,
                C.cast(C.byref(n), C.c_void_p)) == islf.OK
    it = iter(v.tolist())
    get = lambda k: [next(it) for _ in range(k)]  # noqa: E731
    form, grid, njobs, mbox = get(4)
    jobs = []
    for _ in range(njobs):
        j = dict(zip(("rep", "P", "id", "wg", "R", "Wq", "Wf", "ng", "has", "at", "slot", "dn", "up", "outer", "inner"),
                     get(15)))
        j["planes"] = get(get(1)[0])
        j["sets"] = []
        for _ in range(4):
            j["sets"].append((get(get(1)[0]), *get(2)))
        j["stages"] = [([get(4) for _ in range(3)], *get(2)) for _ in range(get(1)[0])]
        jobs.append(j)
    assert next(it, None) is None
    return form, grid, mbox, jobs


def check(shapes, fmt, cus=256):
    got = plan(shapes, fmt, cus)
    if got is None:
        return None
    form, grid, mbox, jobs = got
    assert grid <= cus and sorted(j["id"] for j in jobs) == list(range(len(jobs)))
    per = 16 if form == FINE else 64
    cover = [np.zeros(s[:2], dtype=int) for s in shapes]
    owner = {}
    written = np.zeros(mbox, dtype=bool)
    clusters = [j["wg"] for j in jobs if j["P"] > 1]
    assert len(set(clusters)) == len(clusters)   # all at once: one share of a cluster to a workgroup
    for j in jobs:
        rows = [y for s in j["sets"] for y in s[0]]
        assert len(rows) == j["R"] and (0 in j["sets"][3][0]) == (0 in rows) and len(j["sets"][3][0]) <= 1
        Ly = shapes[j["rep"]][1]
        if 0 in rows:   # the seam lies within the share
            assert Ly - 1 in rows and 1 in rows
        np.add.at(cover[j["rep"]], np.ix_(j["planes"], rows), 1)
        for x in j["planes"]:
            for y in rows:
                owner[j["rep"], x, y] = j
        # chunks: each once per phase, row 0 behind all others
        seen, order = {}, []
        for parts, *_ in j["stages"]:
            for k, ph, c0, c1 in parts:
                if c1 > c0:
                    seen.setdefault((k, ph), []).extend(range(c0, c1))
                    order.append((k, ph))
        for k, (ys, whole, part) in enumerate(j["sets"]):
            n = len(ys) * len(j["planes"])
            assert whole == -(-n * j["Wf"] // per) and part == (-(-n // per) if j["ng"] else 0)
            for ph in (2, 3) if k == 3 else (0, 1):
                assert sorted(seen.get((k, ph), [])) == list(range(whole + part)), (k, ph)
        if j["sets"][1][0] and (3, 2) in order:
            assert order.index((1, 1)) < order.index((3, 2)) < order.index((3, 3))
    for c in cover:
        assert (c == 1).all()
    # faces: 32-bit words of the edge rows and planes, each to its own place in the right neighbour's mailbox
    for j in jobs:
        if j["P"] == 1:
            assert j["has"] == 0
            continue
        Ly, n = shapes[j["rep"]][1], len(j["planes"])
        rows = {y for s in j["sets"] for y in s[0]}
        faces = []
        if j["has"] & HAS_Y:
            low = [y for y in rows if (y - 1) % Ly not in rows]
            high = [y for y in rows if (y + 1) % Ly not in rows]
            assert len(low) == len(high) == 1 and set(low + high) == set(j["sets"][0][0])
            x = j["planes"][0]
            faces += [(j["dn"], n * j["Wq"], owner[j["rep"], x, (low[0] - 1) % Ly]),
                      (j["up"], n * j["Wq"], owner[j["rep"], x, (high[0] + 1) % Ly])]
        y = min(rows)
        lo, hi = min(j["planes"]), max(j["planes"])
        if j["has"] & HAS_OUTER:
            assert owner[j["rep"], lo - 1, y] is owner[j["rep"], hi + 1, y]
            faces.append((j["outer"], 2 * j["R"] * j["Wq"], owner[j["rep"], lo - 1, y]))
        if j["has"] & HAS_INNER:
            inner = next(x for x in range(lo, hi) if x not in j["planes"])
            faces.append((j["inner"], 2 * j["R"] * j["Wq"], owner[j["rep"], inner, y]))
        for at, size, to in faces:
            assert to is not j and to["at"] <= at and at + size <= to["at"] + to["slot"] <= mbox
            assert not written[at:at + size].any()
            written[at:at + size] = True
    return form


@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
@pytest.mark.parametrize("shapes,form", [
    ([(12, 24, 24)], GROUPS), ([(4, 12, 24), (6, 12, 16), (8, 12, 12)] * 56, GROUPS), ([(30, 40, 64)], FINE),
    ([(25, 76, 76), (29, 90, 90), (34, 102, 102)], FINE), ([(40, 120, 120)] * 64, WORDS), ([(184, 504, 504)], WORDS),
    ([(160, 480, 600)] * 3, WORDS), ([(60, 40, 300)] * 3, FINE), ([(1, 2, 2)], GROUPS)])
def test_forms(shapes, form, fmt):
    assert check(shapes, fmt) == form


def test_a_film_beyond_the_lds_is_left_to_the_launch_chain():
    assert check([(1023, 1024, 4096)], islf.BITPACK) is None


@pytest.mark.parametrize("seed", range(40))
def test_drawn_batches(seed):
    rng = np.random.default_rng(seed)
    top = int(rng.choice([20, 60, 200]))
    shapes = [(int(rng.integers(1, 61)), int(rng.integers(2, 2 * top)), 2 * int(rng.integers(1, top)))
              for _ in range(int(rng.integers(1, 13)))]
    check(shapes, seed % 2, int(rng.choice([256, 256, 64, 19])))
