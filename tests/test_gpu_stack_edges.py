"""The fused BF16 step stack (wv_stack_bf16.hip) at the edges of its tiles: subband widths of whole 58
column strips and one column either side, subband heights from one row up, planes narrower than a strip
and one to four mixture components."""
import os

import pytest
import torch

from gpu_common import need_gpu, say
from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 4])
def test_stack_tile_edges_equal_layer_by_layer_bitwise(K):
    """Subband widths 464, 232, 116, 58 / 472, 236, 118, 59 / 456, 228, 114, 57 and 8 .. 1 at heights of
    32 .. 1 rows: the same parameters as the layer-by-layer launches, bit for bit, at every step."""
    need_gpu()
    from paper_2405_12631_amd import codec, batch as B, WV_BF16
    say("stack tile edges", K)
    cfg = dict(get_config("ycbcr512x768"), mix_k=K)
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision=WV_BF16)
    sizes = [(16, 928), (48, 944), (64, 912), (32, 16)]
    imgs = [sinusoid_1f_planes(h, w, planes=3, seed=7 + K + k) for k, (h, w) in enumerate(sizes)]
    os.environ["WV_FUSED_STACKS"] = "0"
    try:
        layered = B.Batch(model, sizes)
    finally:
        del os.environ["WV_FUSED_STACKS"]
    fused = B.Batch(model, sizes)
    layered.load_images(imgs)
    fused.load_images(imgs)
    for i in range(fused.nsub):
        for step in range(4):
            assert torch.equal(fused.context_params(i, step), layered.context_params(i, step)), (i, step)
