"""Which calls the tuning leaves to the resident time loop: the default's and
the autotuner's choice, also where a program saved it, tried another shape and
set it again; a shape of the caller's own is run as asked."""
import ctypes

import pytest

from paper_1107_2157_amd import ics, sw
from swtest import G, announce

pytestmark = pytest.mark.gpu


def resident(s, steps=40):
    if isinstance(s, sw.Solver):
        f = sw.lib().sw_internal_ctx_resident
        f.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        return f(s.ctx, None) == 1
    f = sw.lib().sw_internal_batch_resident
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    return f(s.handle, steps, None) == 1


def single():
    s = sw.Solver(300, 200, g=G)
    s.set_state(*ics.random_state(300, 200, seed=2))
    return s


def batch():
    b = sw.Batch([(64, 64), (130, 130), (320, 200)], g=G)
    for i, (nx, ny) in enumerate(b.shapes):
        b.set_state(i, *ics.random_state(nx, ny, seed=i))
    return b


@pytest.mark.parametrize("make", [single, batch])
def test_round_trip_of_the_default(make):
    announce(f"tuning round trip: {make.__name__}")
    s = make()
    assert resident(s)
    t = s.get_tuning()
    s.set_tuning(**t)
    assert resident(s) and s.get_tuning() == t
    other = dict(t, rows=t["rows"] * 2)
    s.set_tuning(**other)
    assert not resident(s)
    s.set_tuning(**t)
    assert resident(s)
    s.set_tuning(variant=2)              # the fused kernel, asked for
    assert not resident(s)
    s.set_tuning()
    assert resident(s)


@pytest.mark.parametrize("make", [single, batch])
def test_round_trip_of_the_autotuners_choice(make, tmp_path):
    announce(f"tuning round trip after a search: {make.__name__}")
    s = make()
    cache = str(tmp_path / "tune.txt")
    best = s.autotune(steps_per_trial=1, cache_path=cache)
    assert resident(s)
    other = dict(best, rows=100)          # neither the default's height nor one the search tries
    s.set_tuning(**other)
    assert not resident(s)
    s.set_tuning(**best)
    assert resident(s) and s.get_tuning() == best
    again = make()
    again.set_tuning(**other)
    assert not resident(again)
    assert again.autotune(steps_per_trial=1, cache_path=cache) == best     # read back
    assert resident(again)


def test_search_that_fails_leaves_the_tuning(tmp_path):
    announce("tuning search that fails")
    s = single()
    with pytest.raises(sw.SwError):
        s.autotune(steps_per_trial=0)
    assert resident(s)
    s.set_variant(sw.VARIANT_FUSED)
    with pytest.raises(sw.SwError):
        s.autotune(steps_per_trial=0)
    assert not resident(s)


@pytest.mark.parametrize("nx,ny,dtype", [(64, 48, "f32"), (700, 640, "f32"), (300, 200, "f64")])
def test_search_with_a_fixed_dt_keeps_the_faster_form(nx, ny, dtype, tmp_path):
    """Blocked launches must beat the resident loop, which is half their time
    and less at these sizes (3.7 us a step against 1.9 at 64x48)."""
    announce(f"tuning search with a fixed dt: {dtype} {nx}x{ny}")
    s = sw.Solver(nx, ny, g=G, dtype=dtype, cfl=0.0, dt_fixed=0.01)
    s.set_state(*ics.random_state(nx, ny, seed=2))
    cache = str(tmp_path / "tune.txt")
    best = s.autotune(steps_per_trial=40, cache_path=cache)
    assert best["variant"] == sw.VARIANT_FUSED and resident(s)
    again = sw.Solver(nx, ny, g=G, dtype=dtype, cfl=0.0, dt_fixed=0.01)
    assert again.autotune(steps_per_trial=40, cache_path=cache) == best and resident(again)


def test_variant_0_after_a_search():
    """Setting the variant alone leaves the other fields: the library's choice stays it."""
    announce("variant 0 after a search")
    s = single()
    best = s.autotune(steps_per_trial=1)
    s.set_variant(sw.VARIANT_AUTO)
    assert resident(s) and s.get_tuning() == best
    s.set_tuning(rows=100)               # neither the default's height nor one the search tries
    assert not resident(s)
