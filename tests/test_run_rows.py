"""Rows per run of the network's kernels that march down an image (host code,
CPU): the runs that take the fewest steps, without trying every length."""
import ctypes
import random

import pytest

from paper_1107_2157_amd import sw


def run_rows(B, H, slots, extra):
    nseg, trials = ctypes.c_int(), ctypes.c_int()
    f = sw.lib().sw_internal_run_rows
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int] + 2 * [ctypes.POINTER(ctypes.c_int)]
    rows = f(B, H, slots, extra, ctypes.byref(nseg), ctypes.byref(trials))
    return rows, nseg.value, trials.value


def every_length(B, H, slots, extra):
    best = None
    for k in range(1, H + 1):
        rows = -(-H // k)
        segs = -(-H // rows)
        cost = -(-B * segs // slots) * (rows + extra)
        if best is None or cost < best[0]:
            best = cost, rows, segs
        if rows <= 4:
            return best[1:]


RNG = random.Random(2)
CASES = [(64, 256, 256, 5), (48, 256, 512, 5), (1, 1, 256, 5), (1, 5, 256, 5), (257, 3, 256, 5), (32, 256, 256, 5)]
CASES += [(int(2 ** RNG.uniform(0, 10)), int(2 ** RNG.uniform(0, 11)), 256 * RNG.choice([1, 2, 3, 4]), 5) for _ in range(300)]


@pytest.mark.parametrize("B,H,slots,extra", CASES)
def test_same_runs_as_trying_every_length(B, H, slots, extra):
    assert run_rows(B, H, slots, extra)[:2] == every_length(B, H, slots, extra)


@pytest.mark.parametrize("B,H", [(1, 4_000_000), (300, 400_000), (7, 1_000_000), (1000, 100_000), (64, 256), (48, 256)])
def test_few_lengths_are_looked_at(B, H):
    """A launch looks at fewer than a thousand lengths, a tenth of a millisecond at most, however tall the images."""
    rows, nseg, trials = run_rows(B, H, 256, 5)
    assert rows * nseg >= H and trials < 1000, (rows, nseg, trials)
