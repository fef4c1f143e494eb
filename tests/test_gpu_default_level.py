"""The default level of the work items from level 0: five levels below the first, and the sixth
for the source counts where it is the faster one. The crossings of the persistent launch alone
tell which it was."""
import pytest

from helpers import run_gpu_trace
from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu


# (40^3 reaches level 8, 24^3 does not)
@pytest.mark.parametrize("n,n_src,level", [(24, 3, 5), (24, 4, 6), (24, 64, 6), (24, 65, 5), (40, 3, 5), (40, 4, 6),
                                           (40, 512, 6), (40, 513, 5)])
def test_default_level(arc, n, n_src, level):
    w = W.lognormal(n, n_src, 4, source_cells="uniform")
    w.trace["level0"] = 0
    ctx = arc.Context(0)
    try:
        crossings = {k: run_gpu_trace(arc, ctx, w, tune_item_level=k)["ledger"]["kernel_crossings"] for k in (0, 5, 6)}
    finally:
        ctx.close()
    assert crossings[5] != crossings[6]
    assert crossings[0] == crossings[level], crossings
