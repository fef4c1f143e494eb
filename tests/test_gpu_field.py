"""The tracer's deposits and cell steps where they can go wrong: grids of one cell, grids whose
sides are just off the 2-cell tiles and 8-cell blocks of the field's layout, one to four bins,
optically thick gas (bins die out one after the other) and waves whose rays share no tiles.
Checked against the FP64 oracle with the bars of the parity tests, and bitwise across
schedules."""
import numpy as np
import pytest

from helpers import CONSERVATION_TOL, GAMMA_REL_TOL, conservation, rate_errors, run_gpu_trace, run_oracle
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu

EDGES = {2: (13.6, 24.6), 3: (13.6, 24.6, 54.4), 4: (13.6, 24.6, 39.0, 54.4)}


@pytest.fixture(scope="module")
def ctx(arc):
    c = arc.Context(0)
    yield c
    c.close()


def gas(shape, n_src, nb, dense=1.0, seed=31):
    w = W.lognormal(0, n_src, seed, source_cells="uniform", shape=shape)
    w.grid["n_h"] *= np.float32(dense)
    if nb > 1:
        w.bins = W.bins_blackbody(1e5, EDGES[nb])
    else:
        w.bins = W.bins_monochromatic(13.6)
    return w


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 9), (2, 1, 7), (7, 9, 8), (8, 8, 8), (16, 17, 31), (3, 65, 5)])
@pytest.mark.parametrize("nb", [1, 2, 3, 4])
def test_layout_edges(arc, ctx, shape, nb):
    w = gas(shape, 1 if shape == (1, 1, 1) else 2, nb)
    g = run_gpu_trace(arc, ctx, w)
    assert max(rate_errors(g, run_oracle(w))) <= GAMMA_REL_TOL
    assert conservation(g["ledger"]) <= CONSERVATION_TOL
    assert np.array_equal(g["J"], run_gpu_trace(arc, ctx, w, schedule="plain")["J"])


@pytest.mark.parametrize("dense", [0.01, 5.0, 300.0])
@pytest.mark.parametrize("eps_term", [1e-6, 1e-30, 0.0])
def test_bins_that_die_out(arc, ctx, dense, eps_term):
    w = gas((24, 20, 28), 3, 3, dense)
    g = run_gpu_trace(arc, ctx, w, eps_term=eps_term)
    o = run_oracle(w, eps_term=eps_term)
    assert max(rate_errors(g, o)) <= GAMMA_REL_TOL
    assert conservation(g["ledger"]) <= CONSERVATION_TOL
    for k in ("crossings", "rays", "splits", "escaped_rays"):
        assert g["ledger"][k] == o["ledger"][k] or eps_term > 0.0, k


@pytest.mark.parametrize("correction", ["none", "conserving"])
def test_scattered_rays_in_one_wave(arc, ctx, correction):
    """Many sources over a small grid, one wave taking roots of all of them: tiles of different
    blocks want the same table entries."""
    w = gas((40, 36, 44), 40, 3, 0.2)
    one = run_gpu_trace(arc, ctx, w, tune_waves=1, tune_blocks=1, tune_refill=1, tune_item_level=1,
                        correction=correction)
    many = run_gpu_trace(arc, ctx, w, correction=correction)
    assert np.array_equal(one["J"], many["J"])
    if correction == "none":
        assert max(rate_errors(one, run_oracle(w))) <= GAMMA_REL_TOL
    else:
        assert np.array_equal(one["moved_lo"], many["moved_lo"]) and np.array_equal(one["moved_hi"], many["moved_hi"])
        assert conservation(one["ledger"]) <= CONSERVATION_TOL
