"""The measured R_tau<0.1 of a ray whose FP32 depth meets 0.1 twice. Along +x the depth at the end
of the third crossing lies within half an ulp of 0.1: start plus increment round to 0.1, the
compensated sum to the float below it, so a dense cell further on in the same pass meets 0.1 again.
The least of the two lengths is the ray's, and of the source's other rays, which leave the grid
thin, none is shorter."""
import numpy as np
import pytest

from helpers import run_gpu_trace
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu

# depths of the first crossings' cells (the first is crossed for half a cell)
DEPTHS = [tuple(float.fromhex(v) for v in row) for row in (
    ("0x1.34a714p-4", "0x1.4e72f2p-5", "0x1.603258p-6"),
    ("0x1.6a547ep-4", "0x1.5fc5e0p-5", "0x1.a46350p-7"),
    ("0x1.1c13eep-4", "0x1.4ea538p-5", "0x1.90f418p-6"),
)]


def meets_twice(k):
    """The compensated sum of the tracer in FP32."""
    f = np.float32
    tau, lo = f(f(k[0]) * f(0.5)), f(0)
    for inc in (f(k[1]), f(k[2])):
        start = f(tau + lo)
        s = f(max(tau, inc) + min(tau, inc))
        lo = f(lo + f(min(tau, inc) - f(s - max(tau, inc))))
        tau = s
    return start < f(0.1) and f(start + f(k[2])) >= f(0.1) and f(tau + lo) < f(0.1)


@pytest.mark.parametrize("schedule", ["plain", "batched"])
@pytest.mark.parametrize("dense_at", [4, 5])
@pytest.mark.parametrize("k", DEPTHS)
def test_the_least_of_a_rays_lengths(arc, k, dense_at, schedule):
    assert meets_twice(k)
    n, c = 17, 8
    n_h = np.full((n, n, n), 1e-3, np.float32)
    x_hi = np.zeros_like(n_h)
    for i, depth in enumerate(k):
        n_h[c, c, c + i], x_hi[c, c, c + i] = depth, 1.0
    n_h[c, c, c + dense_at], x_hi[c, c, c + dense_at] = 1.0, 1.0
    w = W.lognormal(0, 1, 3, source_cells="uniform", shape=(n, n, n))
    zero = np.zeros_like(n_h)
    # cell length times cross section is one: a cell's depth is its density
    w.grid = {"n_h": n_h, "x_hi": x_hi, "x_hei": zero, "x_heii": zero, "temp": np.full_like(n_h, 1e4),
              "cell_cm": 2.0 ** 60, "y_he": 0.0}
    w.bins = dict(W.bins_monochromatic(), sigma=np.array([[2.0 ** -60, 0.0, 0.0]]))
    w.sources = {"pos": np.full((1, 3), c + 0.5), "ndot": np.array([1e48]), "r_thin_out": np.empty(1)}
    w.trace = dict(w.trace, level0=0)
    ctx = arc.Context(0)
    try:
        run_gpu_trace(arc, ctx, w, schedule=schedule, max_level=0)
    finally:
        ctx.close()
    assert w.sources["r_thin_out"][0] == pytest.approx(2.5, rel=1e-6)
