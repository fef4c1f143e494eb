"""The geometric correction's modes that drop the removed share, with thin spheres and without: the
batched field is bitwise the plain schedule's, for one to four bins, and the rates with thin
spheres are the oracle's."""
import numpy as np
import pytest

from helpers import GAMMA_REL_TOL, rate_errors, run_gpu_trace, run_oracle
from paper_1807_07094_amd import workload as W
from test_gpu_thin import THIN_R_TOL, thin_workload

pytestmark = pytest.mark.gpu

MODES = {"fc": 1, "fc_squared": 3}
EDGES = {2: (13.6, 24.6), 3: (13.6, 24.6, 54.4), 4: (13.6, 24.6, 39.0, 54.4)}


@pytest.fixture(scope="module")
def ctx(arc):
    c = arc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("thin", [False, True])
@pytest.mark.parametrize("bins", [1, 2, 3, 4])
@pytest.mark.parametrize("mode", list(MODES))
def test_share_modes_plain_equals_batched_bitwise(arc, ctx, mode, bins, thin):
    w = thin_workload(seed=51, radii=(0.0, 1.5, 4.0, 9.25, 20.0))
    w.bins = W.bins_monochromatic() if bins == 1 else W.bins_blackbody(1e5, EDGES[bins])
    if not thin:
        w.sources.pop("r_thin")
    fields, radii = [], []
    for schedule in ("plain", "batched"):
        if thin:
            w.sources["r_thin_out"] = np.empty(5)
        r = run_gpu_trace(arc, ctx, w, schedule=schedule, correction=mode)
        fields.append(r["J"])
        radii.append(w.sources.get("r_thin_out", np.empty(0)))
    assert np.array_equal(*fields)
    assert np.array_equal(*radii)


@pytest.mark.parametrize("mode", list(MODES))
def test_share_modes_with_thin_spheres_against_the_oracle(arc, ctx, mode):
    w = thin_workload(seed=45, radii=(0.0, 3.5, 7.0, 0.0, 11.0))
    w.sources["r_thin_out"] = np.empty(len(w.sources["ndot"]))
    w.trace["correction"] = MODES[mode]
    try:
        o = run_oracle(w)
    finally:
        w.trace.pop("correction")
    g = run_gpu_trace(arc, ctx, w, correction=mode)
    assert max(rate_errors(g, o)) <= GAMMA_REL_TOL
    np.testing.assert_allclose(w.sources["r_thin_out"], o["r_thin_out"], rtol=THIN_R_TOL)
