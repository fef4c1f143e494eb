"""The plain chemistry kernel per combination of its options (one instantiation each) and at
grid sizes around a wave's round and its chunk, against the FP64 oracle: fractions within the
parity tests' bar, temperatures to 1e-3 (FP32 rate fits, about 1e-5 per sub-step)."""
import numpy as np
import pytest

import oracle
from helpers import FRACTION_TOL
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(arc):
    c = arc.Context(0)
    yield c
    c.close()


def gas(n, y_he, seed):
    rng = np.random.default_rng(seed)
    shape = (1, 1, n) if n <= 2048 else (1, -(-n // 2000), 2000)
    grid = {"n_h": 10.0 ** rng.uniform(-4, -2, shape), "x_hi": 10.0 ** rng.uniform(-4, 0, shape),
            "x_hei": rng.uniform(0, 0.5, shape) if y_he else np.zeros(shape),
            "x_heii": rng.uniform(0, 0.5, shape) if y_he else np.zeros(shape), "temp": 10.0 ** rng.uniform(3.5, 4.5, shape)}
    grid = {k: v.astype(np.float32) for k, v in grid.items()}
    grid.update(cell_cm=W.COSMIC_CELL_CM, y_he=y_he)
    gamma = (10.0 ** rng.uniform(-17, -12, (3,) + shape)).astype(np.float32)
    heat = (gamma * rng.uniform(1e-12, 1e-11, gamma.shape)).astype(np.float32)
    return grid, gamma, heat


def check(arc, ctx, grid, gamma, heat, dt, chem, graph=False):
    import torch

    g = arc.device_grid(grid)
    st = ctx.chem_step(g, torch.from_numpy(gamma).cuda(), torch.from_numpy(heat).cuda(), dt, graph=graph, **chem)
    state = {k: grid[k] for k in ("x_hi", "x_hei", "x_heii", "temp")}
    o = oracle.chem(grid, state, gamma.astype(np.float64), heat.astype(np.float64), dt, chem)
    for k in ("x_hi", "x_hei", "x_heii"):
        assert float(np.abs(g[k].cpu().numpy() - o[k]).max()) <= FRACTION_TOL, k
    assert float(np.abs(g["temp"].cpu().numpy() / o["temp"] - 1.0).max()) <= 1e-3
    return st


@pytest.mark.parametrize("rates,isothermal,collisional", [(0, 1, 0), (0, 0, 0), (1, 1, 0), (1, 1, 1), (1, 0, 0), (1, 0, 1)])
@pytest.mark.parametrize("y_he", [0.0, 0.08])
def test_options(arc, ctx, rates, isothermal, collisional, y_he):
    grid, gamma, heat = gas(3000, y_he, 7)
    chem = {"isothermal": isothermal, "rates": rates, "collisional": collisional, "alpha_hii": 2.59e-13, "eps": 0.1,
            "max_sub": 100000, "t_floor": 1.0}
    st = check(arc, ctx, grid, gamma, heat, 0.05 * W.MYR_S, chem)
    assert st["capped"] == 0 and st["sub_total"] >= grid["n_h"].size


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 500000])
def test_sizes(arc, ctx, n):
    grid, gamma, heat = gas(n, 0.08, n)
    chem = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1, "max_sub": 100000,
            "t_floor": 1.0}
    st = check(arc, ctx, grid, gamma, heat, 0.01 * W.MYR_S, chem, graph=n % 2 == 0)
    assert st["cells"] == grid["n_h"].size


def test_cap_counts_cells(arc, ctx):
    """max_sub sub-steps, then one to the end: every cell that needed more is counted."""
    import torch

    grid, gamma, heat = gas(2000, 0.08, 3)
    base = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1, "t_floor": 1.0}
    args = (torch.from_numpy(gamma).cuda(), torch.from_numpy(heat).cuda(), 0.05 * W.MYR_S)
    free = ctx.chem_step(arc.device_grid(grid), *args, max_sub=100000, **base)
    assert free["sub_max"] > 3
    few = ctx.chem_step(arc.device_grid(grid), *args, max_sub=2, **base)
    assert few["sub_max"] == 3 and 0 < few["capped"] < grid["n_h"].size
    none = ctx.chem_step(arc.device_grid(grid), *args, max_sub=free["sub_max"], **base)
    assert none["capped"] == 0 and none["sub_max"] == free["sub_max"]
