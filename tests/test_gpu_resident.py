"""The resident time loop (every step of a call in one launch, the state in
registers) against the per-step launches of the fused kernel: the same cells,
halos, time, dt and step count, bit for bit.  A Solver left at its default
tuning takes the resident loop where the grid fits the device; one with a
launch shape set takes the per-step launches."""
import ctypes
import threading

import pytest
import torch

from paper_1107_2157_amd import ics, sw
from swtest import G, announce

pytestmark = pytest.mark.gpu


def pair(nx, ny, **how):
    a, b = sw.Solver(nx, ny, g=G, **how), sw.Solver(nx, ny, g=G, **how)
    b.set_variant(sw.VARIANT_FUSED)
    return a, b


def same(a, b, what):
    assert a.sync_status() == b.sync_status(), what
    assert a.state.cur == b.state.cur
    for k, (x, y) in enumerate(zip(a.get_state(halo=True), b.get_state(halo=True))):
        assert torch.equal(x, y), f"{what}: field {k} differs at {(x != y).nonzero()[:4].tolist()}"


# a strip is up to 62 columns; a wave up to 2, 6, 12, 16 (FP32: 24, 40) rows; a workgroup 4 to 16 waves
SHAPES = [(1, 1), (1, 7), (5, 1), (2, 2), (16, 16), (61, 3), (62, 4), (63, 5), (64, 48), (124, 9), (125, 64),
          (128, 128), (130, 257), (300, 17), (9, 1000), (700, 640), (1024, 1024), (1531, 1087)]


@pytest.mark.parametrize("scheme", [sw.SCHEME_PAPER, sw.SCHEME_TRANSVERSE])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_equals_per_step_launches(nx, ny, dtype, scheme):
    for bc_x, bc_y in ((sw.REFLECT, sw.REFLECT), (sw.PERIODIC, sw.PERIODIC), (sw.REFLECT, sw.PERIODIC),
                       (sw.PERIODIC, sw.REFLECT)):
        announce(f"resident {dtype} {nx}x{ny} scheme={scheme} bc={bc_x}{bc_y}")
        a, b = pair(nx, ny, dtype=dtype, bc_x=bc_x, bc_y=bc_y, scheme=scheme)
        u = ics.random_state(nx, ny, seed=nx + 7 * ny)
        a.set_state(*u)
        b.set_state(*u)
        for steps in (1, 2, 7):                      # several calls: odd and even, the exchange words reused
            a.step(steps)
            b.step(steps)
            same(a, b, f"{steps} steps, bc {bc_x}{bc_y}")


@pytest.mark.parametrize("scheme", [sw.SCHEME_PAPER, sw.SCHEME_TRANSVERSE])
@pytest.mark.parametrize("how", [dict(dx=0.3, dy=0.7), dict(dx=3.0, dy=0.11, cfl=0.4), dict(dx=0.3, dy=0.7, cfl=0.0, dt_fixed=1e-3)])
def test_spacings_and_fixed_dt(how, scheme):
    announce(f"resident spacings {how} scheme={scheme}")
    for dtype in ("f32", "f64"):
        a, b = pair(190, 70, dtype=dtype, bc_y=sw.PERIODIC, scheme=scheme, **how)
        u = ics.random_state(190, 70, seed=5)
        a.set_state(*u)
        b.set_state(*u)
        for steps in (1, 8):
            a.step(steps)
            b.step(steps)
            same(a, b, f"{dtype} {steps} steps")


def test_unstable_state():
    """A dry cell: both report it, and end with the same bits, NaN included."""
    announce("resident unstable 130x70 f32")
    a, b = pair(130, 70, dtype="f32")
    u = [x.clone() if torch.is_tensor(x) else x.copy() for x in ics.random_state(130, 70, seed=6)]
    u[0][30, 64] = -1.0
    for s in (a, b):
        s.set_state(*u)
        s.step(6)
        with pytest.raises(sw.Unstable):
            s.sync_status()
    for x, y in zip(a.get_state(halo=True), b.get_state(halo=True)):
        assert torch.equal(x.contiguous().view(torch.int32), y.contiguous().view(torch.int32))


BATCHES = [([(64, 64), (192, 192), (130, 130), (320, 320), (5, 40), (1, 1)], "f32"),
           ([(256, 256)] * 70, "f32"), ([(48, 100), (300, 33), (700, 260)], "f64"),
           ([(512, 512)] * 30, "f32")]


@pytest.mark.parametrize("scheme", [sw.SCHEME_PAPER, sw.SCHEME_TRANSVERSE])
@pytest.mark.parametrize("sides,dtype", BATCHES)
def test_batch_equals_per_step_launches(sides, dtype, scheme):
    for bc in (sw.REFLECT, sw.PERIODIC):
        announce(f"resident batch of {len(sides)} {dtype} {sides[0]} scheme={scheme} bc={bc}")
        a, b = (sw.Batch(sides, g=G, dtype=dtype, bc_x=bc, bc_y=bc, scheme=scheme) for _ in range(2))
        b.set_tuning(variant=2)
        for i, (nx, ny) in enumerate(sides):
            u = ics.random_state(nx, ny, seed=i)
            a.set_state(i, *u)
            b.set_state(i, *u)
        for steps in (1, 6):
            a.step(steps)
            b.step(steps)
            assert a.sync_status() == b.sync_status()
            for i in range(len(sides)):
                for x, y in zip(a.get_state(i, halo=True), b.get_state(i, halo=True)):
                    assert torch.equal(x, y), f"grid {i} after {steps} steps"


@pytest.mark.parametrize("nx,ny,dtype,scheme", [(300, 200, "f32", sw.SCHEME_PAPER), (70, 33, "f64", sw.SCHEME_TRANSVERSE)])
def test_team_that_gives_up_still_steps(nx, ny, dtype, scheme):
    """With no patience at all the team never comes together, and its last
    workgroup does the steps alone: the same bits."""
    announce(f"resident loop given up: {dtype} {nx}x{ny}")
    f = sw.lib().sw_internal_ctx_patience
    f.argtypes = [ctypes.c_void_p, ctypes.c_longlong]
    f.restype = None
    a, b = pair(nx, ny, dtype=dtype, bc_x=sw.PERIODIC, scheme=scheme)
    u = ics.random_state(nx, ny, seed=3)
    a.set_state(*u)
    b.set_state(*u)
    f(a.ctx, -1)
    for steps in (3, 4):
        a.step(steps)
        b.step(steps)
        same(a, b, f"given up, {steps} steps")
    f(a.ctx, 500_000_000)
    a.step(5)
    b.step(5)
    same(a, b, "after a launch that was given up")


def test_streams_and_threads():
    """Contexts stepped from several threads, each on a stream of its own: more
    workgroups in all than the device holds at once."""
    announce("resident loop: 4 threads x 4 streams, 700x640 f32")
    jobs = []
    for k in range(4):
        a, b = pair(700, 640, dtype="f32")
        u = ics.random_state(700, 640, seed=50 + k)
        a.set_state(*u)
        b.set_state(*u)
        jobs.append((a, b, torch.cuda.Stream()))
    torch.cuda.synchronize()

    def work(job):
        for _ in range(20):
            job[0].step(11, stream=job[2])

    threads = [threading.Thread(target=work, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for a, b, _ in jobs:
        b.step(220)
        same(a, b, "threads")
