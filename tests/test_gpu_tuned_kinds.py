"""A launch shape tuned for one kind of trace (without the correction, without thin spheres) is not
taken for another, whose kernels differ."""
import time

import numpy as np
import pytest

from helpers import run_gpu_trace
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["conserving", "fc", "thin", "radii out", "thin beside the sample"])
def test_another_kind_of_kernel_is_tuned_afresh(arc, kind):
    """The first tuned call of a kind times the candidate shapes (over thirty traces), later ones
    take the shape found."""
    n_src = 300 if kind == "thin beside the sample" else 12  # (one in two of 300 is timed)
    w = W.lognormal(40, n_src, 22, source_cells="uniform")
    other = w.subset(np.arange(n_src))
    kw = {}
    if kind == "thin":
        other.sources["r_thin"] = np.full(n_src, 2.0)
    elif kind == "radii out":
        other.sources["r_thin_out"] = np.empty(n_src)
    elif kind == "thin beside the sample":
        other.sources["r_thin"] = np.where(np.arange(n_src) == 1, 2.0, 0.0)
    else:
        kw["correction"] = kind
    ctx = arc.Context(0)
    try:
        run_gpu_trace(arc, ctx, w, schedule="batched_tuned")
        ref = run_gpu_trace(arc, ctx, other, schedule="batched", **kw)  # buffers of this kind
        took = []
        for _ in range(3):
            t = time.perf_counter()
            got = run_gpu_trace(arc, ctx, other, schedule="batched_tuned", **kw)
            took.append(time.perf_counter() - t)
            assert np.array_equal(got["J"], ref["J"])
    finally:
        ctx.close()
    assert took[0] > 3.0 * min(took[1:]), took
