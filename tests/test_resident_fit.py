"""The LDS that plans of the resident form ask for, checked on the host (no GPU).

A share's lattice, with the halo rows and planes around it, and its tables must
fit the LDS that a launch may ask for, whatever the form the planner chose; a
launch that asks for more is refused by the runtime.
"""
import numpy as np
import pytest

from paper_1411_5588_amd import islf

from test_resident_plan import FINE, HAS_INNER, HAS_OUTER, HAS_Y, built, check, plan  # noqa: F401

LIMIT = 160 * 1024 - 11392   # a CU's LDS without the kernels' static tables


def asked(j, cut_x):
    """LDS bytes of a share: lattice, plane and column tables, mail of its faces."""
    n, R, W = len(j["planes"]), j["R"], j["Wq"]
    lattice = (n + (4 if cut_x else 2)) * (R + 2) * 8 * W
    return (lattice + 15) // 16 * 16 + 24 * n + 28 * R * W + 4 * (2 * n + (4 if cut_x else 0) * R) * W


def fits(shapes, fmt, cus=256):
    got = plan(shapes, fmt, cus)
    if got is None:
        return None
    cut = {j["rep"] for j in got[3] if j["has"] & (HAS_OUTER | HAS_INNER)}
    for j in got[3]:
        assert asked(j, j["rep"] in cut) <= LIMIT, (shapes[j["rep"]], j["R"], len(j["planes"]), j["has"] & HAS_Y)
    return got[0]


@pytest.mark.parametrize("fmt", [islf.INT8, islf.BITPACK])
@pytest.mark.parametrize("n,shape", [(128, (75, 149, 192)), (64, (32, 490, 256)), (64, (28, 1116, 124)),
                                     (85, (4, 5935, 64)), (128, (169, 205, 64))])
def test_full_workgroups(n, shape, fmt):
    # films that leave a share's workgroup next to no LDS
    fits([shape] * n, fmt)
    check([shape] * n, fmt)


@pytest.mark.parametrize("seed", range(60))
def test_drawn_full_batches(seed):
    # one or two shapes, as many films as the device's LDS holds or nearly so
    rng = np.random.default_rng(1000 + seed)
    shapes = []
    for _ in range(int(rng.integers(1, 3))):
        x, y, z = int(rng.integers(2, 180)), int(rng.integers(5, 1200)), 2 * int(rng.integers(8, 130))
        bits = x * y * 8 * (-(-z // 64))
        room = int(256 * LIMIT * rng.uniform(0.75, 1.0)) // 2
        shapes += [(x, y, z)] * max(1, min(256, room // bits))
    fits(shapes, seed % 2)
