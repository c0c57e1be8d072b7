"""The per-step batch path (a tile table over all grids, two chains of launches
replayed as graphs) at full size against whole-grid oracle runs: a launch shape
set by the caller is run as asked."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1107_2157_amd import ics, sw
from swtest import G, announce, rel_maxnorm

pytestmark = pytest.mark.gpu


def test_batch_of_512_grids_per_step_against_whole_grid_oracle():
    """512 grids, sides 64 to 1024, 40 steps with a CFL time step each: the
    smallest, the largest and a random grid, within the bounds the resident
    form is held to (1e-5 of each field's scale and of the time)."""
    k = 40
    sides = ics.batch_sides(512)
    announce(f"batch 512 grids, per-step launches, {k} steps, whole-grid oracle on 3 grids")
    b = sw.Batch(sides, dtype="f32")
    b.set_tuning(variant=2)
    route = sw.lib().sw_internal_batch_resident
    route.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    assert route(b.handle, k, None) == 0
    picks = {int(np.argmin(sides)), int(np.argmax(sides)), int(np.random.default_rng(12).integers(512))}
    states = {}
    for i, n in enumerate(sides):
        st = ics.bumps_state(n, n, seed=ics.SEED_BATCH_GRID0 + i, periodic=False, device="cuda")
        b.set_state(i, *st)
        if i in picks:
            states[i] = [x.to(torch.float32).to(torch.float64).cpu().numpy() for x in st]
    b.step(k)
    t, steps, _ = b.sync_status()
    for i in sorted(picks):
        H, U, V, t_ref = oracle.run(*states[i], k, g=G)
        err = rel_maxnorm(b.get_state(i), [H[1:-1, 1:-1], U[1:-1, 1:-1], V[1:-1, 1:-1]])
        print(f"grid {i} ({sides[i]}^2): rel max-norm {err:.2e}")
        assert steps[i] == k and abs(t[i] - t_ref) <= 1e-5 * t_ref and err <= 1e-5
