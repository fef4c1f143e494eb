"""What a call hands to the host at its end and leaves for the next call: counters, statistics
and minima of a context in use equal those of a fresh one, and the stage times nest."""
import numpy as np
import pytest

from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu

COUNTS = ("crossings", "rays", "splits", "terminated", "escaped_rays", "tree_count", "kernel_crossings")


@pytest.mark.parametrize("schedule,graph", [("batched", False), ("batched", True), ("plain", False)])
def test_calls_do_not_carry_over(arc, schedule, graph):
    import torch

    chem = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1, "max_sub": 50, "t_floor": 1.0}

    def calls(ctx, seed):
        w = W.lognormal(0, 2 + seed, 5 + seed, source_cells="uniform", shape=(12, 10 + seed, 14))
        g = arc.device_grid(w.grid)
        gamma = torch.zeros((3,) + w.grid["n_h"].shape, device="cuda")
        heat = torch.zeros_like(gamma)
        led = ctx.trace(g, w.sources, w.bins, 1e11, gamma, heat, level0=1, schedule=schedule, graph=graph)
        assert led["ms_total"] >= led["ms_trace"] >= led["ms_kernel"] >= 0.0 and led["ms_trace"] > 0.0
        assert led["ms_kernel"] > 0.0 or schedule == "plain"
        dt = ctx.rt_timestep(g, gamma, w.bins, eps=0.1)
        st = ctx.chem_step(g, gamma, heat, 1e11, graph=graph, **chem)
        assert st["ms"] > 0.0
        return ([led[k] for k in COUNTS], [st[k] for k in ("cells", "sub_total", "sub_max", "capped")], dt,
                [led["absorbed"], led["escaped"]])

    used = arc.Context(0)
    try:
        for seed in (2, 0, 1, 0):
            fresh = arc.Context(0)
            try:
                a, b = calls(used, seed), calls(fresh, seed)
            finally:
                fresh.close()
            assert a[:3] == b[:3]
            assert np.allclose(a[3], b[3], rtol=1e-12, atol=0.0)  # FP64 sums in any order
    finally:
        used.close()
