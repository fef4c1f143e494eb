"""The time-step minima where the reduction's remainders matter: grids of one cell, one short of,
equal to and one past the cells a workgroup takes at once, with the limiting cell last."""
import numpy as np
import pytest

import oracle
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 255, 1023, 1024, 1025, 4097])
def test_limiting_cell_last(arc, n):
    import torch

    rng = np.random.default_rng(n)
    shape = (1, 1, n) if n <= 2048 else (3, 1, 1366)
    bins = W.bins_blackbody()
    grid = {"n_h": rng.uniform(5e-4, 2e-3, shape), "x_hi": rng.uniform(0.3, 0.9, shape),
            "x_hei": rng.uniform(0.2, 0.6, shape), "x_heii": rng.uniform(0.0, 0.4, shape),
            "temp": rng.uniform(8e3, 2e4, shape)}
    grid = {k: v.astype(np.float32) for k, v in grid.items()}
    grid.update(cell_cm=W.COSMIC_CELL_CM, y_he=0.08)
    gamma = np.zeros((3,) + shape, np.float32)
    gamma[0] = rng.uniform(1e-16, 1e-15, shape)
    gamma[0].reshape(-1)[-1] = 3e-12
    ctx = arc.Context(0)
    try:
        got = ctx.rt_timestep(arc.device_grid(grid), torch.from_numpy(gamma).cuda(), bins, eps=0.1)
    finally:
        ctx.close()
    cp = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1, "max_sub": 100000,
          "t_floor": 1.0}
    state = {k: grid[k] for k in ("x_hi", "x_hei", "x_heii", "temp")}
    ref = oracle.timestep(grid, state, gamma.astype(np.float64), cp, float(bins["sigma"][0, 0]), 0.1)
    # FP32 rate fits, about 1e-5; the photoionisation rate dominates the limiting cell
    assert got == pytest.approx(ref, rel=1e-4)
