"""The resident loop's plans (host code, CPU): which calls take it."""
import ctypes

import pytest

from paper_1107_2157_amd import sw

F32, F64 = 0, 1


def plan_batch(dtype, scheme, sides, cus=256):
    """(rows, waves per workgroup, workgroups, largest team, from_steps, most_steps, exact) or None."""
    n = len(sides)
    ints = ctypes.c_int * n
    out = (ctypes.c_int * 7)()
    f = sw.lib().sw_internal_plan_batch
    if not f(dtype, scheme, n, ints(*[s[0] for s in sides]), ints(*[s[1] for s in sides]), cus, out):
        return None
    return tuple(out)


# time of a call of so many steps, resident over per-step launches, measured on MI355X
MEASURED = [
    (F32, 0, [(256, 256)] * 256, {1: 1.48, 2: 1.27, 8: 0.86, 20: 0.78}),
    (F32, 0, [(1024, 1024)] * 16, {1: 1.75, 2: 1.42, 12: 0.87, 20: 0.82}),
    (F32, 0, [(512, 512)] * 60, {1: 1.38, 2: 1.19, 8: 0.85, 20: 0.80}),
    (F32, 0, [(256, 256)] * 16, {1: 0.92, 4: 0.59, 20: 0.40}),
    (F32, 0, [(64, 64)] * 32, {1: 0.50, 20: 0.21}),
    (F32, 1, [(1024, 1024)] * 4, {4: 0.85, 20: 0.63}),
    (F64, 0, [(512, 512)] * 60, {1: 1.88, 2: 1.43, 20: 0.87}),
    (F64, 0, [(512, 512)] * 8, {1: 2.11, 2: 1.66, 4: 1.32, 20: 0.83}),
    (F64, 0, [(256, 256)] * 32, {1: 1.48, 2: 1.29, 20: 0.84}),
    (F64, 1, [(512, 512)] * 16, {1: 1.42, 2: 1.33, 4: 1.15}),
    (F64, 1, [(256, 256)] * 8, {1: 0.90, 4: 0.66, 20: 0.40}),
]


@pytest.mark.parametrize("dtype,scheme,sides,ratio", MEASURED)
def test_short_batch_calls_take_the_faster_form(dtype, scheme, sides, ratio):
    """A resident call reads and writes every state once: a call of a few steps
    over many large grids is faster as per-step launches."""
    p = plan_batch(dtype, scheme, sides)
    assert p is not None
    for steps, r in ratio.items():
        if not 0.88 < r < 1.12:
            assert (steps >= p[4]) == (r < 1.0), (steps, r, p)


def plan_grid(dtype, nx, ny, cus=256):
    """(rows, waves per workgroup, workgroups, most_steps) or None."""
    out = (ctypes.c_int * 4)()
    return tuple(out) if sw.lib().sw_internal_plan_grid(dtype, nx, ny, cus, out) else None


# us per step, measured on MI355X
@pytest.mark.parametrize("dtype,scheme,sides,us", [
    (F32, 0, [(256, 256)] * 256, 54.5), (F32, 0, [(1024, 1024)] * 16, 52.3), (F32, 0, [(64, 64)] * 32, 2.9),
    (F32, 1, [(1024, 1024)] * 16, 64.0), (F64, 0, [(512, 512)] * 60, 99.0), (F64, 1, [(512, 512)] * 60, 128.5)])
def test_batch_launches_stay_far_below_the_patience(dtype, scheme, sides, us):
    """A team that does not fit at first waits for whole launches of the teams
    before it, at most one launch's time; it gives up after 5 s."""
    p = plan_batch(dtype, scheme, sides)
    assert p[5] >= 64 and p[5] * us < 0.5e6, p


@pytest.mark.parametrize("dtype,nx,ny,us", [(F32, 64, 48, 2.6), (F32, 1024, 1024, 5.9), (F32, 2048, 2048, 14.8),
                                            (F64, 128, 128, 3.0), (F64, 1024, 1024, 10.7)])
def test_grid_launches_are_short(dtype, nx, ny, us):
    """What one workgroup does alone where a team gives up is a launch, not the call."""
    p = plan_grid(dtype, nx, ny)
    assert p[3] >= 64 and p[3] * us < 0.1e6, p
