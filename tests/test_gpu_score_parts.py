"""Routing with a query tile's keys dealt out to several workgroups.

Calls with few (head, query tile) pairs score each pair in several parts: the
masks must equal the oracle's on both sides of every change of the number of
parts, and where a part has a wave without a key tile.
"""

import numpy as np
import pytest

import synth
from oracle import route_ref
from oracle.compare import compare_mask_rows

from _gpu_util import custom_config, f64, geometry_of, lib, tiling_of, to_dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize(
    "heads,nb",
    [
        (1, 64),  # 4 key tiles: one part
        (1, 65),  # 5 key tiles, two parts: three waves of the second have none
        (2, 129),  # 9 key tiles in three parts, one key in the last tile
        (25, 330),  # 525 pairs: one part although there are 21 key tiles
    ],
)
def test_routing_in_key_parts(heads, nb):
    torch, fva = torch_mod(), lib()
    cfg = custom_config("parts", heads, (1, 1, 64 * nb), (1, 1, 64), np.linspace(0.5, 4.0, heads), seed=81)
    geo = geometry_of(cfg)
    Qb, Kb, _ = synth.gen_qkv(cfg)
    mask, counts, kv = fva.fva_route(to_dev(Qb), to_dev(Kb), cfg.p, cfg.k_min, tiling_of(cfg))
    torch.cuda.synchronize()
    for h in {0, heads // 2, heads - 1}:
        ref = route_ref(f64(Qb[0, h : h + 1]), f64(Kb[0, h : h + 1]), cfg.p, cfg.k_min, geo)
        cmp = compare_mask_rows(mask[0, h].cpu().numpy(), ref["mask"].reshape(-1, nb), ref["order"].reshape(-1, nb),
                                ref["cum"].reshape(-1, nb), ref["scores"].reshape(-1, nb), ref["counts"].reshape(-1),
                                cfg.p, cfg.k_min)
        assert not cmp["mismatch"], (h, cmp)
