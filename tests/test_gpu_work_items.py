"""How rays reach the persistent launch: fewer items than its waves, some to each wave, all that
fit and a queue beyond; single rays and families; levels whose last workgroup is nearly empty.
The field is bitwise the plain schedule's and every ray is traced once."""
import numpy as np
import pytest

from helpers import run_gpu_trace
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(arc):
    c = arc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_src,level0,item_level", [
    (1, 0, 0), (3, 0, 0), (4, 0, 0), (1, 0, 1), (5, 1, 1), (11, 1, 2), (2, 1, 0), (7, 1, 4), (40, 1, 0)])
@pytest.mark.parametrize("blocks", [0, 1, 7])
def test_every_item_once(arc, ctx, n_src, level0, item_level, blocks):
    w = W.lognormal(0, n_src, 3 + n_src, source_cells="uniform", shape=(20, 17, 23))
    w.trace["level0"] = level0
    a = run_gpu_trace(arc, ctx, w, tune_item_level=item_level, tune_blocks=blocks)
    b = run_gpu_trace(arc, ctx, w, schedule="plain")
    assert np.array_equal(a["J"], b["J"])
    for k in ("crossings", "rays", "splits", "terminated", "escaped_rays"):
        assert a["ledger"][k] == b["ledger"][k], k
