"""Synthesis on split 16-bit operands: against the oracle at the edges of its strips and segments,
bitwise the same whatever the launch geometry, NaN where the FP32 kernels give NaN, and bytes
that stay those of the FP32 kernels."""
import os

import numpy as np
import pytest
import torch

import oracle as O
from gpu_common import XHAT_ATOL, model_for, need_gpu, q_to_device, say
from wvgen import get_config, sinusoid_1f_planes

pytestmark = pytest.mark.gpu


def _fp32(fn):
    os.environ["WV_LIFT_FORM"] = "tile"
    try:
        out = fn()
        torch.cuda.synchronize()
        return out
    finally:
        del os.environ["WV_LIFT_FORM"]


# Strips have 28 or 124 output columns, segments as few as one row: level-1 arrays of 28, 56 + 4,
# 124, 124 + 4 and 248 columns, level-4 arrays of one row or column.
@pytest.mark.parametrize("H,W,N", [(16, 16, 1), (16, 64, 2), (48, 128, 1), (64, 256, 3), (80, 496, 1), (112, 512, 2)])
def test_split_synthesis_matches_oracle_and_is_geometry_invariant(H, W, N):
    need_gpu()
    from paper_2405_12631_amd import codec
    say("split lifting", H, W, N)
    cfg = get_config("ycbcr512x768")
    model, w = model_for(cfg)
    qs, _ = O.quantize(O.analyze(sinusoid_1f_planes(H, W, planes=N, seed=H + W), cfg, w), cfg)
    q = q_to_device(qs)
    ws = codec.Workspace(model, N, H, W)
    x, _ = codec.synthesize(model, ws, q=q)
    ref = O.synthesize(O.dequantize(qs, cfg), cfg, w)
    old = _fp32(lambda: codec.synthesize(model, ws, q=q)[0])
    err, err_old = (float(np.max(np.abs(a.cpu().numpy() - ref))) for a in (x, old))
    say("max error: split", err, "fp32", err_old)
    assert err <= XHAT_ATOL
    # 48 planes take other strips and segments than one: the same bits
    big = codec.synthesize(model, codec.Workspace(model, 48, H, W), q=q[:1].repeat(48, 1).contiguous())[0]
    one = codec.synthesize(model, codec.Workspace(model, 1, H, W), q=q[:1].contiguous())[0]
    assert torch.equal(one[0], x[0])
    assert all(torch.equal(big[k], x[0]) for k in (0, 17, 47))


def test_split_synthesis_nan_and_bytes():
    need_gpu()
    from paper_2405_12631_amd import codec
    say("split lifting, NaN and bytes")
    cfg = get_config("ycbcr512x768")
    model, w = model_for(cfg)
    H, W = 96, 160
    ws = codec.Workspace(model, 2, H, W)
    y = torch.from_numpy(np.random.default_rng(3).normal(0, 20, (2, H * W)).astype(np.float32)).cuda()
    y[0, 5] = float("nan")
    y[1, H * W // 2] = float("nan")
    x = codec.synthesize(model, ws, y=y)[0]
    old = _fp32(lambda: codec.synthesize(model, ws, y=y)[0])
    assert torch.equal(torch.isnan(x), torch.isnan(old)) and bool(torch.isnan(x).any())
    assert float((x - old)[~torch.isnan(x)].abs().max()) <= XHAT_ATOL
    q = torch.randint(-20, 21, (2, H * W), dtype=torch.int16, device="cuda")
    f, u8 = codec.synthesize(model, ws, q=q, want_u8=True)
    fo, uo = _fp32(lambda: codec.synthesize(model, ws, q=q, want_u8=True))
    assert torch.equal(u8, uo) and torch.equal(f, fo)
