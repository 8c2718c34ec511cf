"""The low-precision convs at the lines where all weights come before the loop: two and three workgroups
per compute unit (of 256), on either side."""
import os

import pytest
import torch

from gpu_common import need_gpu, say
from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_both_sides_of_two_and_three_workgroups_per_cu(prec):
    """Three planes of 256x512 and 352x384: layers of two blocks in 768 and 792 workgroups; of 192x224 and
    128x352: ConvLSTMs in 504 and 528 (and coarser levels below).  The parameters equal a plan's, whose
    launches bring weights tap by tap, bit for bit."""
    need_gpu()
    from paper_2405_12631_amd import codec, batch as B, WV_BF16, WV_FP8
    say("conv weights, lines", prec)
    cfg = get_config("ycbcr512x768")
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision={"bf16": WV_BF16, "fp8": WV_FP8}[prec])
    sizes = [(256, 512), (352, 384), (192, 224), (128, 352)]
    os.environ["WV_FUSED_STACKS"] = "0"
    try:
        plan = B.Batch(model, sizes)
    finally:
        del os.environ["WV_FUSED_STACKS"]
    plan.load_images([sinusoid_1f_planes(h, w, planes=3, seed=31 + k) for k, (h, w) in enumerate(sizes)])
    refs = [(codec.Workspace(model, w.N, w.H, w.W), plan.q[b].clone()) for b, w in enumerate(plan.ws)]
    K = cfg["mix_k"]
    for i in range(plan.nsub):
        for g in range(4):
            got = plan.context_params(i, g).clone()
            _, first = plan.rows(i, g)
            for b, (ws, q) in enumerate(refs):
                one = codec.context_params(model, q, ws, i, g).reshape(-1)
                assert torch.equal(got[first[b] * 3 * K:first[b] * 3 * K + one.numel()], one), (i, g, b)
