"""The split-operand lifting kernel, asked for by its option, at the edges of its strips and segments:
against the oracle, the same bits whatever the launch geometry, NaN where FP32 gives NaN, and bytes that
are those of its floats."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_common import XHAT_ATOL, need_gpu, q_to_device, say
from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

pytestmark = pytest.mark.gpu


def _models(cfg, w):
    from paper_2405_12631_amd import codec, WV_FP32, WV_LIFT_SPLIT
    return [codec.Model(cfg, pack_weights(cfg, w), precision=p) for p in (WV_FP32, WV_FP32 | WV_LIFT_SPLIT)]


# Strips have 28 or 124 output columns, segments as few as one row: level-1 arrays of 28, 56 + 4,
# 124, 124 + 4 and 248 columns, level-4 arrays of one row or column; a tall narrow plane.
@pytest.mark.parametrize("H,W,N", [(16, 16, 1), (16, 64, 2), (48, 128, 1), (64, 256, 3), (80, 496, 1), (112, 512, 2),
                                   (1040, 16, 1)])
def test_split_kernel_matches_oracle_and_is_geometry_invariant(H, W, N):
    need_gpu()
    from paper_2405_12631_amd import codec
    say("split kernel", H, W, N)
    cfg = get_config("ycbcr512x768")
    w = make_weights(cfg)
    fp32, model = _models(cfg, w)
    qs, _ = O.quantize(O.analyze(sinusoid_1f_planes(H, W, planes=N, seed=H + W), cfg, w), cfg)
    q = q_to_device(qs)
    ws = codec.Workspace(model, N, H, W)
    x, u8 = codec.synthesize(model, ws, q=q, want_u8=True)
    ref = O.synthesize(O.dequantize(qs, cfg), cfg, w)
    old = codec.synthesize(fp32, ws, q=q)[0]
    err, err_old = (float(np.max(np.abs(a.cpu().numpy() - ref))) for a in (x, old))
    say("max error: split", err, "fp32", err_old)
    assert err <= XHAT_ATOL
    # a lost low part of an operand (2^-12 or 2^-17 of it) shows here; the largest of few thousand
    # roundings varies by less than a factor of four, and half a float's step is never counted against it
    assert err <= 4 * max(err_old, 2.0 ** -17)
    assert torch.equal(u8, x.round().clamp(0, 255).to(torch.uint8))
    # 48 planes take other strips and segments than one: the same bits
    big = codec.synthesize(model, codec.Workspace(model, 48, H, W), q=q[:1].repeat(48, 1).contiguous())[0]
    one = codec.synthesize(model, codec.Workspace(model, 1, H, W), q=q[:1].contiguous())[0]
    assert torch.equal(one[0], x[0])
    assert all(torch.equal(big[k], x[0]) for k in (0, 17, 47))


def test_split_kernel_keeps_nan():
    need_gpu()
    from paper_2405_12631_amd import codec
    say("split kernel, NaN")
    cfg = get_config("ycbcr512x768")
    fp32, model = _models(cfg, make_weights(cfg))
    H, W = 96, 160
    ws = codec.Workspace(model, 2, H, W)
    y = torch.from_numpy(np.random.default_rng(3).normal(0, 20, (2, H * W)).astype(np.float32)).cuda()
    y[0, 5] = float("nan")
    y[1, H * W // 2] = float("nan")
    x, old = (codec.synthesize(m, ws, y=y)[0] for m in (model, fp32))
    assert torch.equal(torch.isnan(x), torch.isnan(old)) and bool(torch.isnan(x).any())
    assert float((x - old)[~torch.isnan(x)].abs().max()) <= XHAT_ATOL


def test_split_decode_in_a_graph_batch_and_impulse_responses():
    """The option through the other users of synthesis: a captured decode, and impulse responses."""
    need_gpu()
    from paper_2405_12631_amd import codec
    say("split kernel, graph and impulse responses")
    cfg = get_config("ycbcr512x768")
    w = make_weights(cfg)
    fp32, model = _models(cfg, w)
    H, W = 64, 96
    q = torch.randint(-20, 21, (3, H * W), dtype=torch.int16, device="cuda")
    ws = codec.Workspace(model, 3, H, W)
    syms = codec.prepare_elided(model, q, ws)
    qd, x = torch.zeros_like(q), torch.empty((3, H, W), device="cuda")
    ref = codec.synthesize(model, ws, q=q)[0]
    step = lambda: (codec.zero(qd), codec.decode_elided(model, syms, ws, qd, xhat=x))  # noqa: E731
    step()
    graph = codec.Graph(step)
    for _ in range(3):
        x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, ref) and torch.equal(qd, q)
    a, b = (codec.impulse_responses(m, q[0], H, W) for m in (model, fp32))
    assert float((a - b).abs().max()) <= XHAT_ATOL and not torch.equal(a, b)
