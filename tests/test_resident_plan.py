"""The resident loop's plans (host code, CPU): which calls take it."""
import ctypes

import pytest

from paper_1107_2157_amd import sw

F32, F64 = 0, 1


def plan_batch(dtype, scheme, sides, cus=256):
    """(rows, waves per workgroup, workgroups, largest team, from_steps) or None."""
    n = len(sides)
    ints = ctypes.c_int * n
    out = (ctypes.c_int * 5)()
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
