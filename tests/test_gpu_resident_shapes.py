"""Every instance of the resident time loop against the per-step launches, bit
for bit: each height of a wave that single grids are cut into, batches whose
waves differ in height, teams of more workgroups than a lane polls flags of at
once.  Each case states the cut that it is there for and that it takes the
resident loop."""
import ctypes
import random

import pytest
import torch

from paper_1107_2157_amd import ics, sw
from swtest import G, announce

pytestmark = pytest.mark.gpu

WALLS = [(sw.REFLECT, sw.REFLECT), (sw.PERIODIC, sw.PERIODIC), (sw.REFLECT, sw.PERIODIC), (sw.PERIODIC, sw.REFLECT)]
SCHEMES = [sw.SCHEME_PAPER, sw.SCHEME_TRANSVERSE]


def cut_of_grid(dtype, nx, ny):
    """(rows, waves per workgroup, workgroups, steps of a launch at most)"""
    out = (ctypes.c_int * 4)()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert sw.lib().sw_internal_plan_grid(int(dtype == "f64"), nx, ny, cus, out) == 1
    return tuple(out)


def cut_of_batch(dtype, scheme, sides):
    """(rows, waves per workgroup, workgroups, largest team, from_steps, steps of a launch at most, exact)"""
    n = len(sides)
    ints = ctypes.c_int * n
    out = (ctypes.c_int * 7)()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert sw.lib().sw_internal_plan_batch(int(dtype == "f64"), scheme, n, ints(*[s[0] for s in sides]),
                                           ints(*[s[1] for s in sides]), cus, out) == 1
    return tuple(out)


def resident(s, steps=1):
    if isinstance(s, sw.Solver):
        f = sw.lib().sw_internal_ctx_resident
        f.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        return f(s.ctx, None) == 1
    f = sw.lib().sw_internal_batch_resident
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    return f(s.handle, steps, None) == 1


# (nx, ny, rows of a wave, waves of a workgroup): odd heights, several strips
F32 = [(16, 16, 1, 4), (16, 1025, 2, 4), (16, 2063, 3, 4), (16, 5277, 3, 8), (65, 3079, 4, 8), (16, 4221, 5, 4),
       (63, 4111, 5, 8), (63, 5287, 6, 8), (5301, 97, 8, 8), (5352, 231, 8, 16), (5453, 129, 10, 8), (5449, 271, 10, 16),
       (5354, 161, 12, 8), (5604, 332, 12, 16), (5278, 196, 14, 8), (5338, 393, 14, 16), (5370, 449, 16, 16),
       (5349, 265, 18, 8), (5316, 292, 20, 8), (5523, 326, 22, 8), (5423, 354, 24, 8), (5414, 413, 28, 8),
       (5287, 467, 32, 8), (5420, 532, 36, 8), (5593, 587, 40, 8)]
F64 = [(16, 16, 1, 4), (16, 1033, 2, 4), (16, 5148, 3, 8), (64, 3096, 4, 8), (63, 4268, 5, 8), (63, 5228, 6, 8),
       (125, 4129, 8, 8), (125, 5514, 10, 8), (5316, 166, 12, 8), (5272, 196, 14, 8), (5309, 233, 16, 8)]


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("dtype,nx,ny,rows,nw", [("f32", *c) for c in F32] + [("f64", *c) for c in F64])
def test_each_height_of_a_wave(dtype, nx, ny, rows, nw, scheme):
    assert cut_of_grid(dtype, nx, ny)[:2] == (rows, nw)
    u = ics.random_state(nx, ny, seed=nx + ny)
    for k, (bc_x, bc_y) in enumerate(WALLS):
        if k > 1 and nx * ny > 400_000:
            break
        announce(f"resident {dtype} {nx}x{ny} scheme={scheme} bc={bc_x}{bc_y}: {rows} rows, {nw} waves")
        a, b = (sw.Solver(nx, ny, g=G, dtype=dtype, bc_x=bc_x, bc_y=bc_y, scheme=scheme) for _ in range(2))
        b.set_variant(sw.VARIANT_FUSED)
        assert resident(a) and not resident(b)
        for s in (a, b):
            s.set_state(*u)
            s.step(1)
            s.step(4)
        assert a.sync_status() == b.sync_status()
        for q in range(3):
            assert torch.equal(a.halo_view(q), b.halo_view(q)), f"field {q}, bc {bc_x}{bc_y}"


def sides_of(seed, n, lo, hi):
    rng = random.Random(seed)
    return [(rng.randint(lo, hi), rng.randint(lo, hi)) for _ in range(n)]


# batches whose waves have any number of rows up to the greatest
UNEVEN = [("f32", 56, 38, 4, 80, 4), ("f32", 167, 38, 4, 130, 6), ("f32", 179, 38, 4, 250, 8), ("f32", 369, 38, 4, 200, 10),
          ("f32", 171, 38, 4, 300, 12), ("f32", 353, 38, 4, 300, 16), ("f32", 1355, 24, 133, 400, 20),
          ("f32", 2634, 22, 50, 500, 24), ("f32", 1809, 12, 80, 800, 32), ("f32", 2966, 22, 200, 600, 40),
          ("f64", 56, 38, 4, 80, 4), ("f64", 167, 38, 4, 130, 6), ("f64", 164, 38, 4, 250, 8), ("f64", 369, 38, 4, 200, 10),
          ("f64", 171, 38, 4, 300, 12), ("f64", 2, 38, 4, 300, 16)]


def check_batch(dtype, scheme, sides, bc_x, bc_y, cut):
    a, b = (sw.Batch(sides, g=G, dtype=dtype, bc_x=bc_x, bc_y=bc_y, scheme=scheme) for _ in range(2))
    b.set_tuning(variant=2)
    for i, (nx, ny) in enumerate(sides):
        u = ics.random_state(nx, ny, seed=i)
        a.set_state(i, *u)
        b.set_state(i, *u)
    for steps in (cut[4], cut[4] + 5):
        assert resident(a, steps) and not resident(b, steps)
        a.step(steps)
        b.step(steps)
    assert a.sync_status() == b.sync_status()
    for i in range(len(sides)):
        for q in range(3):
            assert torch.equal(a.halo_view(i, q), b.halo_view(i, q)), f"grid {i}, field {q}, bc {bc_x}{bc_y}"


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("dtype,seed,n,lo,hi,rows", UNEVEN)
def test_batches_of_uneven_heights(dtype, seed, n, lo, hi, rows, scheme):
    sides = sides_of(seed, n, lo, hi)
    cut = cut_of_batch(dtype, scheme, sides)
    assert cut[0] == rows and not cut[6], cut
    for bc_x, bc_y in WALLS[:2]:
        announce(f"resident batch of {n} {dtype}, sides {lo} to {hi} scheme={scheme} bc={bc_x}{bc_y}: up to {rows} rows")
        check_batch(dtype, scheme, sides, bc_x, bc_y, cut)


@pytest.mark.parametrize("dtype,scheme,sides,team", [
    ("f32", sw.SCHEME_PAPER, [(2000, 2000), (300, 200)], 429), ("f32", sw.SCHEME_TRANSVERSE, [(1000, 2100), (60, 60)], 459),
    ("f64", sw.SCHEME_PAPER, [(1024, 1024)] * 2, 442)])
def test_teams_of_many_workgroups(dtype, scheme, sides, team):
    """More than the 256 flags that a wave polls at once."""
    cut = cut_of_batch(dtype, scheme, sides)
    assert cut[3] == team, cut
    announce(f"resident batch {dtype} {sides} scheme={scheme}: teams of up to {team} workgroups")
    check_batch(dtype, scheme, sides, sw.REFLECT, sw.PERIODIC, cut)


@pytest.mark.parametrize("sides,dtype", [([(256, 256)] * 70, "f32"), ([(512, 512)] * 30, "f32"),
                                         ([(48, 100), (300, 33), (700, 260)], "f64")])
@pytest.mark.parametrize("scheme", SCHEMES)
def test_even_batches(sides, dtype, scheme):
    """More workgroups than fit at once, with as many steps as it takes for the resident loop."""
    cut = cut_of_batch(dtype, scheme, sides)
    announce(f"resident batch of {len(sides)} {dtype} {sides[0]} scheme={scheme}, {cut[2]} workgroups")
    check_batch(dtype, scheme, sides, sw.REFLECT, sw.REFLECT, cut)
