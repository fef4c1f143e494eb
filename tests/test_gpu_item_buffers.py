"""Device memory that the work items take: the last of the levels before the persistent launch
leaves one record per split ray, not one per child."""
import pytest

from paper_1807_07094_amd import workload as W

pytestmark = pytest.mark.gpu

RECORD = 48  # bytes
N_SRC = 1024


@pytest.mark.parametrize("item_level", [0, 4, 5, 6])
def test_ray_buffers_hold_the_records_they_are_written(arc, item_level):
    import torch

    w = W.lognormal(0, N_SRC, 9, source_cells="uniform", shape=(16, 16, 16))
    g = arc.device_grid(w.grid)
    gamma = torch.empty((3,) + w.shape, device="cuda")
    heat = torch.empty_like(gamma)
    # from level 0 with many sources the default is level 5 or 6
    level = item_level or 6
    items = N_SRC * 12 * 4 ** (level - 1) * RECORD  # families of that level, the rays of the one before
    waves = torch.cuda.get_device_properties(0).multi_processor_count * 16
    ctx = arc.Context(0)
    try:
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ctx.trace(g, w.sources, w.bins, w.dt, gamma, heat, level0=0, tune_item_level=item_level)
        used = free - torch.cuda.mem_get_info()[0]
    finally:
        ctx.close()
    spill = waves * 4096 * RECORD
    assert used <= 2 * items + spill + (64 << 20), (used, items, spill)
