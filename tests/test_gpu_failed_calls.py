"""A context after a call that failed part way: a spill area that could not be had is not used, and
the field that arc_get_field hands out is the last trace's or none."""
import numpy as np
import pytest

from helpers import run_gpu_trace
from paper_1807_07094_amd import workload as W
from test_gpu_batching import deep_subtrees

pytestmark = pytest.mark.gpu


def test_the_spill_area_is_there_after_one_too_large(arc):
    w = deep_subtrees()
    shape = dict(tune_item_level=w.trace["level0"], tune_waves=1)
    ctx = arc.Context(0)
    try:
        a = run_gpu_trace(arc, ctx, w, **shape)
        assert a["ledger"]["spills"] > 0
        with pytest.raises(arc.ArcError) as e:  # 400 TB
            run_gpu_trace(arc, ctx, w, spill_cap=2 ** 31 - 1, **shape)
        assert e.value.status == -3
        b = run_gpu_trace(arc, ctx, w, **shape)
        assert b["ledger"]["spills"] > 0
        assert np.array_equal(a["J"], b["J"])
    finally:
        ctx.close()


def test_no_field_after_a_call_that_replaced_its_buffer(arc):
    import torch

    small = W.lognormal(0, 2, 5, source_cells="uniform", shape=(12, 12, 12))
    large = W.lognormal(0, 2, 5, source_cells="uniform", shape=(40, 40, 40))
    ctx = arc.Context(0)
    try:
        run_gpu_trace(arc, ctx, small)
        with pytest.raises(arc.ArcError) as e:  # planned for the larger grid, then refused
            run_gpu_trace(arc, ctx, large, tune_waves=3)
        assert e.value.status == -1
        J = torch.zeros((3,) + small.shape, dtype=torch.int64, device="cuda")
        with pytest.raises(arc.ArcError) as e:
            ctx.get_field(J)
        assert e.value.status == -1
        # arguments refused before any buffer is touched leave the field alone
        a = run_gpu_trace(arc, ctx, small)
        with pytest.raises(arc.ArcError) as e:
            run_gpu_trace(arc, ctx, large, eps_term=2.0)
        assert e.value.status == -2
        ctx.get_field(J)
        assert (J.cpu().numpy() == a["J"]).all()
    finally:
        ctx.close()
