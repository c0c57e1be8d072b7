"""Limits of the resident loop: calls of several launches, teams that give up."""
import ctypes

import pytest
import torch

from paper_1107_2157_amd import ics, sw
from swtest import G, announce

pytestmark = pytest.mark.gpu


def pair(nx, ny, seed, **how):
    """A solver at its default tuning and one that takes a launch per step, at the same state."""
    a, b = sw.Solver(nx, ny, g=G, **how), sw.Solver(nx, ny, g=G, **how)
    b.set_variant(sw.VARIANT_FUSED)
    u = ics.random_state(nx, ny, seed=seed)
    a.set_state(*u)
    b.set_state(*u)
    return a, b


def batches(sides, **how):
    a, b = (sw.Batch(sides, g=G, **how) for _ in range(2))
    b.set_tuning(variant=2)
    for i, (nx, ny) in enumerate(sides):
        u = ics.random_state(nx, ny, seed=i)
        a.set_state(i, *u)
        b.set_state(i, *u)
    return a, b


def same(a, b, what):
    assert a.sync_status() == b.sync_status(), what
    assert a.state.cur == b.state.cur
    for k, (x, y) in enumerate(zip(a.get_state(halo=True), b.get_state(halo=True))):
        assert torch.equal(x, y), f"{what}: field {k} differs"


def same_batch(a, b, what):
    assert a.sync_status() == b.sync_status(), what
    for i in range(a.n):
        for x, y in zip(a.get_state(i, halo=True), b.get_state(i, halo=True)):
            assert torch.equal(x, y), f"{what}: grid {i}"


def batch_limits(a, patience, steps):
    f = sw.lib().sw_internal_batch_limits
    f.argtypes = [ctypes.c_void_p, ctypes.c_longlong, ctypes.c_int]
    f.restype = None
    f(a.handle, patience, steps)


def is_resident(a, steps):
    f = sw.lib().sw_internal_batch_resident
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    return f(a.handle, steps, None) == 1


PATIENCE = 500_000_000


@pytest.mark.parametrize("how", [dict(dtype="f32"), dict(dtype="f64", scheme=sw.SCHEME_TRANSVERSE, bc_x=sw.PERIODIC),
                                 dict(dtype="f32", cfl=0.0, dt_fixed=0.01)])
def test_call_of_several_launches(how):
    announce(f"resident call of several launches: 190x70 {how}")
    a, b = pair(190, 70, 4, **how)
    f = sw.lib().sw_internal_ctx_most_steps
    f.argtypes = [ctypes.c_void_p, ctypes.c_int]
    f.restype = None
    f(a.ctx, 3)
    for steps in (11, 3, 4, 1):                # 3 + 3 + 3 + 2, 3, 2 + 2, 1
        a.step(steps)
        b.step(steps)
        same(a, b, f"{steps} steps")


def test_batch_call_of_several_launches():
    sides = [(64, 64), (130, 130), (320, 320), (5, 40)]
    announce(f"resident batch call of several launches: {sides}")
    a, b = batches(sides, dtype="f32")
    batch_limits(a, PATIENCE, 4)
    for steps in (9, 8, 5):
        assert is_resident(a, steps)
        a.step(steps)
        b.step(steps)
        same_batch(a, b, f"{steps} steps")


def test_batch_teams_that_give_up():
    """Every team's last workgroup does the steps of its grid alone: the same bits."""
    sides = [(130, 130), (64, 48), (200, 150)]
    announce(f"resident batch given up: {sides}")
    a, b = batches(sides, dtype="f32", bc_y=sw.PERIODIC)
    batch_limits(a, -1, 64)
    for steps in (3, 4):
        assert is_resident(a, steps)
        a.step(steps)
        b.step(steps)
        same_batch(a, b, f"given up, {steps} steps")
    batch_limits(a, PATIENCE, 64)
    a.step(5)
    b.step(5)
    same_batch(a, b, "after launches that were given up")


def test_per_step_launches_after_a_team_gave_up():
    """A team that gives up shows that the device is shared: once the status
    call has seen it, calls take the per-step launches."""
    announce("per-step launches after a team gave up")
    a, b = pair(190, 70, 5, dtype="f64")
    patience = sw.lib().sw_internal_ctx_patience
    patience.argtypes = [ctypes.c_void_p, ctypes.c_longlong]
    patience.restype = None
    route = sw.lib().sw_internal_ctx_resident
    route.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    batch, ref = batches([(64, 48), (130, 130)], dtype="f32")
    a.step(2)
    batch.step(2)
    a.sync_status()
    batch.sync_status()
    assert route(a.ctx, None) == 1 and is_resident(batch, 4)
    patience(a.ctx, -1)
    batch_limits(batch, -1, 64)
    a.step(3)
    batch.step(3)
    torch.cuda.synchronize()
    patience(a.ctx, PATIENCE)
    batch_limits(batch, PATIENCE, 64)
    a.sync_status()
    batch.sync_status()
    assert route(a.ctx, None) == 0 and not is_resident(batch, 4)
    a.step(4)
    batch.step(4)
    b.step(9)
    ref.step(9)
    same(a, b, "after giving up")
    same_batch(batch, ref, "after giving up")


def test_no_memory_for_the_exchange():
    """A context or batch without memory for the exchange words is created all
    the same, and takes the per-step launches."""
    announce("no memory for the exchange words")
    deny = sw.lib().sw_internal_deny_alloc
    deny.argtypes, deny.restype = [], None
    route = sw.lib().sw_internal_ctx_resident
    route.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    deny()
    a, b = pair(190, 70, 5, dtype="f32")
    assert route(a.ctx, None) == 0
    deny()
    batch, ref = batches([(64, 48), (130, 130)], dtype="f64")
    assert not is_resident(batch, 40)
    for steps in (2, 5):
        a.step(steps)
        b.step(steps)
        same(a, b, f"{steps} steps")
        batch.step(steps)
        ref.step(steps)
        same_batch(batch, ref, f"{steps} steps")
    c, _ = pair(190, 70, 5, dtype="f32")
    assert route(c.ctx, None) == 1
