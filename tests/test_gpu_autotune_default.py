"""The autotuner and the untuned schedule: the default refill threshold is one of those the tuner
tries, so that it can choose and time the default shape."""
import pytest

from helpers import run_gpu_trace
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu

TRIED = (16, 32, 48, 56, 64)


def test_the_default_refill_is_one_the_tuner_tries(arc):
    """One wave takes the root rays in their order, so the lines it adds to are a count that its
    refill threshold decides."""
    w = W.lognormal(0, 4, 11, source_cells="uniform", shape=(24, 24, 24))
    ctx = arc.Context(0)
    try:
        lines = {refill: run_gpu_trace(arc, ctx, w, tune_waves=1, tune_blocks=1, tune_refill=refill,
                                       tune_item_level=w.trace["level0"])["ledger"]["kernel_deposits"]
                 for refill in (0, 40) + TRIED}
    finally:
        ctx.close()
    assert len({lines[r] for r in TRIED}) == len(TRIED)  # the count tells them apart
    assert lines[0] in [lines[r] for r in TRIED], lines
