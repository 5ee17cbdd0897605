"""Work-list edges of the persistent scheduler against the naive grid.

Whatever way items reach the workgroups (a workgroup's first item by its
index, later ones from the queue counters), every row must be run exactly
once: with few enough kept blocks that no row is split, the persistent launch
equals the naive grid bit for bit, and rows left out would keep the NaN that
the output starts with.
"""

import numpy as np
import pytest

import synth

from _gpu_util import custom_config, geometry_of, lib, tiling_of, to_dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize(
    "heads,grid,tile",
    [
        (1, (1, 8, 8), (1, 8, 8)),  # one item, seven empty queues
        (1, (1, 8, 40), (1, 8, 8)),  # fewer items than queues
        (3, (1, 8, 24), (1, 8, 8)),  # 9 items: one queue holds two
        (7, (2, 16, 24), (2, 8, 8)),  # 42 items, uneven queues
        (40, (1, 16, 52), (1, 8, 8)),  # 560 items: more than two per CU
        (160, (2, 8, 40), (2, 8, 8)),  # 800 items of five blocks
    ],
)
def test_every_item_runs_once(heads, grid, tile):
    torch, fva = torch_mod(), lib()
    cfg = custom_config("sched", heads, grid, tile, np.linspace(0.3, 5.0, heads), seed=61)
    geo = geometry_of(cfg)
    rng = np.random.default_rng(62)
    q, k, v = (torch.randn((1, heads, cfg.N, 128), generator=torch.Generator().manual_seed(63 + i)).bfloat16().cuda()
               for i in range(3))
    # uneven rows, some empty (an empty row's output is zero)
    mask = (rng.random((1, heads, geo.nb, geo.nb)) < rng.random((1, heads, geo.nb, 1))).astype(np.uint8)
    m = torch.from_numpy(mask).cuda()
    assert mask.sum(-1).max() <= 32  # the smallest automatic chunk: nothing is split
    want = fva.fva_attn(q, k, v, tiling_of(cfg), m, flags=fva.FVA_SCHED_NAIVE)
    for flags in (0, fva.FVA_SCHED_UNPAIRED):
        out = torch.full_like(q, float("nan"))
        fva.fva_attn(q, k, v, tiling_of(cfg), m, flags=flags, out=out)
        assert torch.equal(out, want)
