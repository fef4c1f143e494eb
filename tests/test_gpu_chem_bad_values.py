"""What one species' bad rate, or an empty cell, does to the others in the plain step: with a
single sub-step a non-finite helium rate leaves x_HI as it is without it (hydrogen's update reads
the start of the sub-step), and a cell without gas keeps its helium fractions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE = (4, 4, 12)


def step(arc, ctx, poison, isothermal, rates, n_h=None):
    import torch

    rng = np.random.default_rng(5)
    g = {k: torch.from_numpy(rng.uniform(lo, hi, SHAPE).astype(np.float32)).cuda()
         for k, lo, hi in (("n_h", 1e-4, 1e-2), ("x_hi", 0.05, 0.95), ("x_hei", 0.1, 0.4), ("x_heii", 0.1, 0.4),
                           ("temp", 5e3, 4e4))}
    g.update(cell_cm=1e21, y_he=0.08)
    if n_h is not None:
        g["n_h"].view(-1)[n_h] = 0.0
    before = {k: g[k].clone() for k in ("x_hei", "x_heii")}
    gamma = torch.from_numpy(rng.uniform(1e-15, 1e-13, (3,) + SHAPE).astype(np.float32)).cuda()
    heat = gamma * 1e-12
    for species, cell, value in poison:
        gamma[species].view(-1)[cell] = value
    # a limit that never binds: one sub-step to the end
    st = ctx.chem_step(g, gamma, heat, 1e11, isothermal=isothermal, rates=rates, eps=1e30, max_sub=4)
    assert st["sub_total"] == g["n_h"].numel()
    return g, before


@pytest.mark.parametrize("isothermal,rates", [(0, 1), (1, 1), (1, 0)])
def test_a_bad_helium_rate_leaves_hydrogen_alone(arc, isothermal, rates):
    import torch

    poison = [(1, 3, np.inf), (1, 70, np.nan), (2, 11, np.nan), (1, 150, 3e38)]
    ctx = arc.Context(0)
    try:
        clean, _ = step(arc, ctx, [], isothermal, rates)
        bad, _ = step(arc, ctx, poison, isothermal, rates)
    finally:
        ctx.close()
    assert torch.isfinite(bad["x_hi"]).all()
    assert torch.allclose(bad["x_hi"], clean["x_hi"], rtol=2.0 ** -23, atol=0.0)
    others = torch.ones(clean["x_hi"].numel(), dtype=torch.bool)
    others[[cell for _, cell, _ in poison]] = False
    for k in ("x_hei", "x_heii", "temp"):
        assert torch.equal(bad[k].view(-1)[others.cuda()], clean[k].view(-1)[others.cuda()]), k


def test_an_empty_cell_keeps_its_helium(arc):
    import torch

    cells = torch.tensor([0, 77, 191])
    ctx = arc.Context(0)
    try:
        clean, _ = step(arc, ctx, [], 0, 1)
        got, before = step(arc, ctx, [], 0, 1, n_h=cells.cuda())
    finally:
        ctx.close()
    others = torch.ones(clean["x_hi"].numel(), dtype=torch.bool)
    others[cells] = False
    for k in ("x_hei", "x_heii"):
        assert torch.equal(got[k].view(-1)[cells.cuda()], before[k].view(-1)[cells.cuda()]), k
        assert torch.equal(got[k].view(-1)[others.cuda()], clean[k].view(-1)[others.cuda()]), k
