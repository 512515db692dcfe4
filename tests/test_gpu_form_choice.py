"""Which form a run takes follows from the context as it is, not from how it got there."""
import ctypes as C
import itertools

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1411_5588_amd import islf  # noqa: E402

from _helpers import config1  # noqa: E402

FORMS = (islf.EXEC_PLAIN, islf.EXEC_BATCHED, islf.EXEC_PERSISTENT)


def takes_resident(ctx, n):
    v = C.c_int32()
    assert islf.lib().islf_testing_takes_resident(ctx._h, n, C.byref(v)) == islf.OK
    return v.value


def big(fmt, exec_mode=islf.EXEC_BATCHED, **over):
    ps = [config1(Lx=160, Ly=480, Lz=600, init=islf.INIT_UP, replica=r, **over) for r in range(3)]
    return islf.Context([islf.Replica(**p) for p in ps], spin_format=fmt, obs_capacity=64, exec_mode=exec_mode)


def test_choice_does_not_depend_on_the_forms_before():
    # three films of 46 M sites in bits: the chain of concurrent groups is the faster batched form, the
    # resident one the faster persistent form
    want = {}
    for form in FORMS:
        with big(islf.BITPACK, form) as ctx:
            want[form] = [takes_resident(ctx, n) for n in (2, 100)]
    assert want[islf.EXEC_BATCHED][1] == 0 and want[islf.EXEC_PERSISTENT][1] == 1
    for order in itertools.permutations(FORMS):
        with big(islf.BITPACK) as ctx:
            for form in order + order[:1]:
                ctx.set_exec(form)
                assert [takes_resident(ctx, n) for n in (2, 100)] == want[form], (order, form)


@pytest.mark.parametrize("mode", [islf.EXEC_BATCHED, islf.EXEC_PERSISTENT])
@pytest.mark.parametrize("shape,n", [((12, 24, 24), 1), ((20, 64, 64), 24), ((40, 120, 120), 16)])
def test_tuning_leaves_long_runs_resident(shape, n, mode):
    # trials of one or two sweeps, in which a resident launch cannot pay for itself, tune the launch chain only
    ps = [config1(Lx=shape[0], Ly=shape[1], Lz=shape[2], replica=r) for r in range(n)]
    with islf.Context([islf.Replica(**p) for p in ps], spin_format=islf.INT8, obs_capacity=64, exec_mode=mode) as ctx:
        for sweeps in (1, 2):
            assert takes_resident(ctx, 200) == 1
            ctx.autotune(sweeps=sweeps)
        assert takes_resident(ctx, 200) == 1
        ctx.set_grid(256)      # the caller's own choice asks for the chain
        assert takes_resident(ctx, 200) == 0
