"""Accuracy of synthesis against 64 bits, for filters of several scales and for large subbands: the FP32
kernels, and split operands, which may not be further off.

Bounds.  An FP32 filter value carries the rounding of 288 products and sums (about sqrt(288) half-units of
2^-24) and tanh's 2^-23; split operands carry 2^-23 of each operand instead, so their root-mean-square error
is expected below that of FP32 and bounded by twice it.  Losing the low parts of an operand leaves 2^-12
(FP16) or 2^-17 (two of three BF16 parts) of it: 60 to 2000 times the bound."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_common import need_gpu, say
from wvgen import get_config, make_weights, pack_weights

pytestmark = pytest.mark.gpu


def _weights(cfg, kind):
    w, rng = make_weights(cfg), np.random.default_rng(17)
    for k in w:
        if not k.startswith("lift."):
            continue
        layer, is_w = int(k.split(".")[2]), k.endswith(".w")
        a = w[k].astype(np.float64)
        if kind == "steep":
            a = a * 4
        elif kind == "flat":
            a = a / 64
        elif kind == "spread" and is_w:      # weights of one layer over six decades
            a = a * np.exp2(4 - rng.uniform(0, 20, a.shape))
        elif kind == "one large" and is_w and layer > 0:
            a.flat[7] = 64.0
        elif kind == "tiny" and layer > 0:   # the scale of layers 2 and 3 at its cap
            a = a * 2.0 ** -70
        elif kind == "zero" and is_w and layer == 1:
            a = a * 0
        w[k] = a.astype(np.float32)
    return w


@pytest.mark.parametrize("kind,std", [("as drawn", 20), ("as drawn", 3000), ("as drawn", 0.01), ("steep", 20), ("flat", 20),
                                      ("flat", 3000), ("spread", 20), ("spread", 3000), ("one large", 20), ("tiny", 20),
                                      ("zero", 20)])
def test_synthesis_error_against_64_bits(kind, std):
    need_gpu()
    from paper_2405_12631_amd import codec, WV_FP32, WV_LIFT_SPLIT
    cfg = get_config("ycbcr512x768")
    w, (H, W) = _weights(cfg, kind), (80, 160)
    y = np.random.default_rng(5).normal(0, std, (1, H * W)).astype(np.float32)
    ref = O.synthesize(O.unpack(y, cfg, H, W), cfg, w, add_offset=False)
    err = []
    for prec in (WV_FP32, WV_FP32 | WV_LIFT_SPLIT):
        model = codec.Model(cfg, pack_weights(cfg, w), precision=prec)
        x = codec.synthesize(model, codec.Workspace(model, 1, H, W), y=torch.from_numpy(y).cuda(), offset=0.0)[0]
        err.append(float(np.linalg.norm(x.cpu().numpy() - ref) / np.linalg.norm(ref)))
    say("error", kind, std, "fp32 %.3g split %.3g" % tuple(err))
    assert err[1] <= 2 * err[0]
    if kind == "as drawn" and std >= 20:
        assert err[0] <= 1e-7


def test_filters_beyond_the_split_range_are_refused():
    """Weights above 2^24, or none, in any layer: no model with split operands; FP32 takes them."""
    need_gpu()
    from paper_2405_12631_amd import codec, WvError, WV_LIFT_SPLIT
    cfg = get_config("ycbcr512x768")
    for key, v in (("lift.P_row.0.w", 3e7), ("lift.U_col.1.b", -2.0 ** 25), ("lift.P_col.2.w", float("nan")),
                   ("lift.U_row.2.b", float("inf"))):
        w = make_weights(cfg)
        w[key].flat[0] = v
        codec.Model(cfg, pack_weights(cfg, w))
        with pytest.raises(WvError):
            codec.Model(cfg, pack_weights(cfg, w), precision=WV_LIFT_SPLIT)
    w["lift.U_row.2.b"].flat[0] = 2.0 ** 24
    codec.Model(cfg, pack_weights(cfg, w), precision=WV_LIFT_SPLIT)


def test_split_operands_saturate_on_infinite_subbands():
    """Infinite and huge values: split operands saturate the filters they reach, so that no value is lost
    that FP32 keeps finite, and NaN stays NaN.  Opposite infinities side by side, where an FP32 sum is NaN,
    keep a finite filter value."""
    need_gpu()
    from paper_2405_12631_amd import codec, WV_FP32, WV_LIFT_SPLIT
    say("split operands and infinities")
    cfg, (H, W) = get_config("ycbcr512x768"), (96, 160)
    blob = pack_weights(cfg, make_weights(cfg))
    y = torch.from_numpy(np.random.default_rng(8).normal(0, 20, (4, H * W)).astype(np.float32)).cuda()
    inf = float("inf")
    out = []
    for prec in (WV_FP32, WV_FP32 | WV_LIFT_SPLIT):
        model = codec.Model(cfg, blob, precision=prec)
        ws = codec.Workspace(model, 4, H, W)
        at = ws.lay[-2]["offset"] + 20 * ws.lay[-2]["w"] + 30          # LH of level 1
        y[0, at], y[1, at], y[1, at + 1], y[2, at], y[3, at] = inf, inf, -inf, 3e38, float("nan")
        out.append(codec.synthesize(model, ws, y=y)[0])
    fp32, split = out
    assert bool((torch.isfinite(split) | ~torch.isfinite(fp32)).all())
    assert int(torch.isnan(split[1]).sum()) < int(torch.isnan(fp32[1]).sum())
    assert torch.equal(torch.isnan(split[3]), torch.isnan(fp32[3])) and bool(torch.isnan(fp32[3]).any())
    near = torch.isfinite(fp32) & (fp32.abs() < 1e4)
    assert float((split - fp32)[near].abs().max()) <= 1e-3
