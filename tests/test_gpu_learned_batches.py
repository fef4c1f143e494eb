"""Cells of the learned step wait until 64 that passed the gate's bins fill a wave: a cell's result
must not depend on where it waits. Cells known to be accepted are laid out densely, shuffled,
and one to a tile of 64 among cells the gate turns away (64 tiles wait for one batch), at sizes
around a tile; every layout gives each cell the same bits. The network's outputs are sums of
the cell's own products and exact zeros, so no rounding differs."""
import numpy as np
import pytest

from paper_1807_07094_amd import learned
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu

STATE = ("n_h", "x_hi", "x_hei", "x_heii", "temp")


@pytest.fixture(scope="module")
def accepted(arc):
    """Context, network, step options and cells [11][n] (state, rates, heating) that it accepts."""
    import torch

    ctx = arc.Context(0)
    X, Y = learned.training_set(ctx, arc, n=200_000, seed=5, sizes=(48, 64), n_src=(32, 48))
    net = arc.MLP(ctx)
    net.train(X, Y, epochs=5, batch=1024, lr=2e-3, seed=3)
    w = W.lognormal(48, 32, 78)
    g = arc.device_grid(w.grid)
    gamma = torch.empty((3,) + w.shape, dtype=torch.float32, device="cuda")
    heat = torch.empty_like(gamma)
    ctx.trace(g, w.sources, w.bins, w.dt, gamma, heat, level0=w.trace["level0"], eps_term=w.trace["eps_term"])
    cells = torch.cat([torch.stack([g[k].reshape(-1) for k in STATE]), gamma.reshape(3, -1), heat.reshape(3, -1)])
    o = dict(mlp=net, y_he=g["y_he"], cell_cm=g["cell_cm"], dt=w.dt, chem=w.chem)
    plain, _ = step(ctx, cells, dict(o, mlp=None))
    both, _ = step(ctx, cells, o)
    took = (plain != both).any(0)
    assert int(took.sum()) > 1000
    yield ctx, o, cells[:, took].contiguous()
    ctx.close()


def step(ctx, cells, o):
    """x_hi and temp [2][n] after the step, and the cells that fell back."""
    n = cells.shape[1]
    nx = next(d for d in range(min(n, 2048), 0, -1) if n % d == 0)
    ny = next(d for d in range(min(n // nx, 2048), 0, -1) if n // nx % d == 0)
    shape = (n // nx // ny, ny, nx)
    g = {k: cells[i].clone().reshape(shape) for i, k in enumerate(STATE)}
    g.update(y_he=o["y_he"], cell_cm=o["cell_cm"])
    kw = dict(o["chem"])
    if o["mlp"] is not None:
        kw.update(mode="mlp_gated", mlp=o["mlp"], gate_tol=1e-3)
    st = ctx.chem_step(g, cells[5:8].clone().reshape((3,) + shape), cells[8:11].clone().reshape((3,) + shape), o["dt"], **kw)
    import torch

    return torch.stack([g["x_hi"].reshape(-1), g["temp"].reshape(-1)]), st.get("fallback")


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 4096, 4097 * 64, 409600])
def test_sizes_and_order(accepted, n):
    import torch

    ctx, o, cells = accepted
    pick = torch.arange(n, device="cuda") % cells.shape[1]
    ref, back = step(ctx, cells, o)
    assert back == 0
    got, back = step(ctx, cells[:, pick], o)
    assert back == 0 and torch.equal(got, ref[:, pick])
    shuffled = pick[torch.randperm(n, device="cuda", generator=torch.Generator("cuda").manual_seed(n))]
    got, back = step(ctx, cells[:, shuffled], o)
    assert back == 0 and torch.equal(got, ref[:, shuffled])


@pytest.mark.parametrize("tiles,per_tile", [(1, 1), (65, 63), (2 ** 12, 33), (2 ** 19, 1), (2 ** 19, 3)])
def test_few_to_a_tile(accepted, tiles, per_tile):
    import torch

    ctx, o, cells = accepted
    ref, _ = step(ctx, cells, o)
    at = (torch.arange(tiles, device="cuda")[:, None] * 64
          + (7 * torch.arange(tiles, device="cuda")[:, None] + 11 * torch.arange(per_tile, device="cuda")) % 64).reshape(-1)
    pick = torch.arange(at.numel(), device="cuda") % cells.shape[1]
    away = cells[:, :1].clone()
    away[5:] = 0.0  # without light: outside the gate's range
    every = away.repeat(1, tiles * 64)
    every[:, at] = cells[:, pick]
    got, back = step(ctx, every, o)
    assert back == tiles * 64 - at.numel()
    assert torch.equal(got[:, at], ref[:, pick])
    dark = torch.ones(tiles * 64, dtype=torch.bool, device="cuda")
    dark[at] = False
    alone, _ = step(ctx, away, dict(o, mlp=None))
    assert bool((got[:, dark] == alone).all())
