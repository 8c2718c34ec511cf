"""A level's two column steps in one launch of the FP32 lifting kernels (wv_lift_fused.hip, wv_lift_rows.hip)."""
import os

import pytest
import torch

from gpu_common import need_gpu, say
from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,planes", [(336, 3), (352, 3), (16, 1), (1008, 1), (1024, 1)])
def test_both_column_steps_in_one_launch_equal_tiles_bitwise(h, planes):
    """512 columns: the two sets of column steps together pass the line of 2048 strip rows at 342 rows of
    3 planes and at 1024 of one, with a band of columns left to the tiles; 16 rows: arrays of one row.
    Analysis and byte synthesis equal those in tiles alone, and planes analysed one by one."""
    need_gpu()
    from paper_2405_12631_amd import codec, WV_FP32
    say("lifting sets", h, planes)
    cfg = get_config("ycbcr512x768")
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision=WV_FP32)
    x = torch.from_numpy(sinusoid_1f_planes(h, 512, planes=planes, seed=h)).to(model.device)

    def run(x):
        ws = codec.Workspace(model, x.shape[0], h, 512)
        q, y, _ = codec.analyze(model, x, ws, want_y=True)
        return q, y, codec.synthesize(model, ws, q=q, want_u8=True)[1]

    got = run(x)
    os.environ["WV_LIFT_FORM"] = "tile"
    try:
        tiles = run(x)
    finally:
        del os.environ["WV_LIFT_FORM"]
    one = [torch.cat(p) for p in zip(*(run(x[k:k + 1].contiguous()) for k in range(planes)))]
    for a, b, c in zip(got, tiles, one):
        assert torch.equal(a, b)
        assert torch.equal(a.reshape(-1), c.reshape(-1))
