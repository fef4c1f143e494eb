"""A context after a call that failed part way: a spill area that could not be had is not used."""
import numpy as np
import pytest

from helpers import run_gpu_trace
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
