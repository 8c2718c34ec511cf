"""The low-precision conv's two ways to bring its weights to LDS (wv_conv_bf16.hip): launches of single
plane groups choose by their number of workgroups, a plan's segment launches always go tap by tap."""
import os

import pytest
import torch

from gpu_common import need_gpu, say
from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_weights_all_at_once_equal_tap_by_tap_bitwise(prec):
    """Level-1 launches of 240 and 264 (line at 256) and 576 and 624 workgroups (line at 600), coarser
    levels far below: the parameters of every (subband, step) equal the plan's, bit for bit."""
    need_gpu()
    from paper_2405_12631_amd import codec, batch as B, WV_BF16, WV_FP8
    say("conv weights all at once", prec)
    cfg = get_config("ycbcr512x768")
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision={"bf16": WV_BF16, "fp8": WV_FP8}[prec])
    sizes = [(112, 320), (112, 336), (240, 384), (240, 400)]
    os.environ["WV_FUSED_STACKS"] = "0"
    try:
        plan = B.Batch(model, sizes)
    finally:
        del os.environ["WV_FUSED_STACKS"]
    plan.load_images([sinusoid_1f_planes(h, w, planes=3, seed=91 + k) for k, (h, w) in enumerate(sizes)])
    refs = []
    for b, w in enumerate(plan.ws):
        refs.append((codec.Workspace(model, w.N, w.H, w.W), plan.q[b].clone()))
    K = cfg["mix_k"]
    for i in range(plan.nsub):
        for g in range(4):
            got = plan.context_params(i, g).clone()
            n, first = plan.rows(i, g)
            for b, (ws, q) in enumerate(refs):
                one = codec.context_params(model, q, ws, i, g).reshape(-1)
                assert torch.equal(got[first[b] * 3 * K:first[b] * 3 * K + one.numel()], one), (i, g, b)
