"""The resident time loop beside other streams and threads: captures that are
under way, streams that come and go, launches of uneven size that do not fit
the device together."""
import ctypes
import threading
import time

import pytest
import torch

from paper_1107_2157_amd import ics, sw
from swtest import G, announce

pytestmark = pytest.mark.gpu


def hip():
    return ctypes.CDLL("libamdhip64.so")


def pair(nx, ny, seed, **how):
    """A solver at its default tuning and one that takes a launch per step, at the same state."""
    a, b = sw.Solver(nx, ny, g=G, **how), sw.Solver(nx, ny, g=G, **how)
    b.set_variant(sw.VARIANT_FUSED)
    u = ics.random_state(nx, ny, seed=seed)
    a.set_state(*u)
    b.set_state(*u)
    return a, b


def same(a, b, what):
    assert a.sync_status() == b.sync_status(), what
    for k, (x, y) in enumerate(zip(a.get_state(halo=True), b.get_state(halo=True))):
        assert torch.equal(x, y), f"{what}: field {k} differs"


def test_steps_beside_a_capture_of_another_thread():
    """A capture in the global mode forbids other threads some calls (to query
    an event among them) and is invalidated by them: steps make none."""
    announce("resident steps beside a capture in another thread")
    a, b = pair(300, 200, 1)
    c, _ = pair(64, 64, 2)
    own, cap = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(2):                                  # launches to be ordered behind
        a.step(5, stream=own)
    c.fill_halo(stream=cap)
    torch.cuda.synchronize()
    failed = []

    def work():
        try:
            for _ in range(4):
                a.step(3, stream=own)
        except Exception as e:                          # noqa: BLE001 (reported below)
            failed.append(e)

    h = hip()
    s, graph = ctypes.c_void_p(cap.cuda_stream), ctypes.c_void_p()
    assert h.hipStreamBeginCapture(s, 0) == 0           # global
    t = threading.Thread(target=work)
    try:
        c.fill_halo(stream=cap)
        t.start()
        t.join()
    finally:
        rc = h.hipStreamEndCapture(s, ctypes.byref(graph))
    assert not failed, failed
    assert rc == 0 and graph.value, f"capture ended with error {rc}"
    assert h.hipGraphDestroy(graph) == 0
    b.step(22)
    same(a, b, "beside a capture")


def test_streams_that_end():
    """A launch is ordered behind launches of streams that are no more."""
    announce("resident steps on streams that are destroyed")
    a, b = pair(700, 640, 3)
    h = hip()
    for k in range(6):
        s = ctypes.c_void_p()
        assert h.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        a.step(5, stream=torch.cuda.ExternalStream(s.value))
        assert h.hipStreamSynchronize(s) == 0
        assert h.hipStreamDestroy(s) == 0
    a.step(1)
    b.step(31)
    same(a, b, "streams destroyed")


def test_uneven_grids_on_many_streams():
    """Grids of very different size stepped from five threads on a stream
    each: more workgroups in all than fit, in changing company."""
    announce("resident loop: 5 threads x 5 streams, uneven grids f32")
    sizes = [(1024, 1024), (300, 200), (64, 48), (700, 640), (1500, 200)]
    jobs = [(*pair(nx, ny, 60 + k), torch.cuda.Stream()) for k, (nx, ny) in enumerate(sizes)]
    torch.cuda.synchronize()

    def work(a, stream):
        for k in range(30):
            a.step(1 + k % 7, stream=stream)

    threads = [threading.Thread(target=work, args=(a, s)) for a, _, s in jobs]
    began = time.perf_counter()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    took = time.perf_counter() - began
    for a, b, _ in jobs:
        for k in range(30):
            b.step(1 + k % 7)
        same(a, b, "uneven grids")
    assert took < 4.0, f"{took:.1f} s: a team waited out its patience (5 s)"


def test_stream_with_a_mask_of_compute_units():
    """A stream whose kernels may use half of the device takes the per-step
    launches: a team cut for the whole device would never come together."""
    announce("steps on a stream with a mask of compute units")
    a, b = pair(700, 640, 8)
    batch, ref = (sw.Batch([(256, 256)] * 16, g=G) for _ in range(2))
    ref.set_tuning(variant=2)
    u = ics.random_state(256, 256, seed=9)
    for i in range(16):
        batch.set_state(i, *u)
        ref.set_state(i, *u)
    h = hip()
    words = (torch.cuda.get_device_properties(0).multi_processor_count + 31) // 32
    some = (ctypes.c_uint32 * words)(*[0xffffffff if k < words // 2 else 0 for k in range(words)])
    every = (ctypes.c_uint32 * words)(*[0xffffffff] * words)
    grid_route, batch_route = sw.lib().sw_internal_ctx_resident, sw.lib().sw_internal_batch_resident
    grid_route.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    batch_route.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    torch.cuda.synchronize()
    for mask, resident in ((some, 0), (every, 1)):
        s = ctypes.c_void_p()
        assert h.hipExtStreamCreateWithCUMask(ctypes.byref(s), words, mask) == 0
        assert grid_route(a.ctx, s) == resident and batch_route(batch.handle, 9, s) == resident
        stream = torch.cuda.ExternalStream(s.value)
        a.step(5, stream=stream)
        batch.step(9, stream=stream)
        assert h.hipStreamSynchronize(s) == 0
        assert h.hipStreamDestroy(s) == 0
    for s in (None, torch.cuda.Stream().cuda_stream):
        assert grid_route(a.ctx, s) == 1
    b.step(10)
    same(a, b, "masked stream")
    ref.step(18)
    assert batch.sync_status() == ref.sync_status()
    for i in range(16):
        assert torch.equal(batch.interior(i, 0), ref.interior(i, 0))
