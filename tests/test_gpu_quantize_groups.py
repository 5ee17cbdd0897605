"""fva_quantize_v where its heads go through in several groups.

The amax of one group of heads (100 MB of V) and the tiles of the group before
share a launch: the heads at a group's edges must come out as any other, bit
for bit, also where a head's tokens end inside an amax workgroup's 256 rows.
"""

import numpy as np
import pytest

import synth

from _gpu_util import custom_config, geometry_of, tiling_of
from test_gpu_fp8 import check_quantizer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,edges", [(12, (0, 11)), (14, (0, 11, 12, 13))])  # one whole group; 12 + 2 heads
def test_quantize_v_over_head_groups(heads, edges):
    cfg = custom_config("qgroups", heads, (21, 30, 52), (2, 8, 8), np.full(heads, 1.0), seed=51)
    _, _, Vb = synth.gen_qkv(cfg)
    V = synth.bf16_bits_to_f32(Vb)
    V *= np.exp2(np.arange(heads) - 6.0).astype(np.float32)[None, :, None, None]  # every head its own exponents
    check_quantizer(f"{heads} heads", synth.f32_to_bf16_bits(V), tiling_of(cfg), geometry_of(cfg), heads=edges)
