"""The arithmetic of a model's synthesis is the model's own: FP32, or split 16-bit operands where its
creator asked for them; never a matter of which outputs a call wants or through which entry point
it comes."""
import ctypes
import os

import numpy as np
import pytest
import torch

from gpu_common import need_gpu, say
from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes, video_gop_420

SPLIT = 256   # WV_LIFT_SPLIT


def _pack_bytes(cfg, precision):
    from paper_2405_12631_amd import _lib as L, codec
    n = ctypes.c_size_t()
    return L.lib().wv_pack_bytes(ctypes.byref(codec.make_config(cfg)), precision, ctypes.byref(n)), n.value


def test_split_lifting_is_asked_for_and_refused_where_it_does_not_exist():
    from paper_2405_12631_amd import _lib as L
    big, small = get_config("ycbcr512x768"), get_config("gray64")
    for prec in (0, 1, 2):
        (rc0, n0), (rc1, n1) = _pack_bytes(big, prec), _pack_bytes(big, prec | SPLIT)
        # four filters of 5 + 36 + 2 rows of 64 16-byte operands, with scales and biases
        assert rc0 == rc1 == L.WV_OK and 4 * 43 * 1024 <= n1 - n0 <= 4 * 44 * 1024
    for cfg in (small, dict(big, lift_int=1), dict(big, lift_layers=4), dict(big, lift_layers=2)):
        assert _pack_bytes(cfg, 0)[0] == L.WV_OK and _pack_bytes(cfg, SPLIT)[0] == L.WV_EUNSUPPORTED
    for prec in (3, 3 | SPLIT, 2 * SPLIT, -1):
        assert _pack_bytes(big, prec)[0] == L.WV_EUNSUPPORTED


def _tiles(fn):
    os.environ["WV_LIFT_FORM"] = "tile"
    try:
        out = fn()
        torch.cuda.synchronize()
        return out
    finally:
        del os.environ["WV_LIFT_FORM"]


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp32 split", "bf16 split"])
def test_one_arithmetic_per_model(prec):
    """Floats with and without bytes, decode with and without bytes, elided decode, batch and server: one
    reconstruction.  A GOP's bytes are those of its floats.  Without the option, that of the FP32 tiles."""
    need_gpu()
    from paper_2405_12631_amd import codec, batch as B, serve
    say("one synthesis arithmetic", prec)
    split = prec.endswith("split")
    cfg = get_config("ycbcr512x768")
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)),
                        precision={"fp32": 0, "bf16": 1}[prec.split()[0]] | (SPLIT if split else 0))
    H, W = 96, 160
    img = sinusoid_1f_planes(H, W, planes=3, seed=12)
    ws = codec.Workspace(model, 3, H, W)
    data, q = codec.encode(model, torch.from_numpy(img).cuda(), ws)
    ref, u8 = codec.synthesize(model, ws, q=q, want_u8=True)
    assert torch.equal(u8, ref.round().clamp(0, 255).to(torch.uint8))
    assert torch.equal(codec.synthesize(model, ws, q=q)[0], ref)
    for want in (True, False):
        x, b, qd = codec.decode(model, data, ws, want_u8=want)
        assert torch.equal(qd, q) and torch.equal(x, ref) and (b is None or torch.equal(b, u8))
    syms = codec.prepare_elided(model, q, ws)
    assert torch.equal(codec.decode_elided(model, syms, ws, torch.zeros_like(q)), ref)
    bt = B.Batch(model, [(H, W), (32, 48)])
    for k, (b, p0) in enumerate(bt.where):
        if k == 0:
            bt.q[b][p0:p0 + 3] = q
            at = b, p0
    assert torch.equal(bt.synthesize()[at[0]][at[1]:at[1] + 3], ref)
    # a served GOP, and its bytes against those of a synthesis that wants bytes itself
    luma, chroma = video_gop_420(T=8, H=64, W=64, seed=5)
    prep = serve.Prepared(model, "gop", (luma, chroma))
    _, done = serve.Server(model, 2 * serve.footprint(model, prep)).run(
        [(0.0, 0)], {0: prep}, max_seconds=1e9, keep_outputs=True, tick=1.0)
    for (h, w, n, q_known, _, _), got in zip(prep.groups, done[0].xhat):
        wg = codec.Workspace(model, n, h, w)
        f = [codec.synthesize(model, wg, q=q_known, want_u8=want, offset=0.0)[0] for want in (True, False)]
        bytes_of = []
        for x in f:
            v = codec.temporal_haar(x.view(8, -1), inverse=True)
            bytes_of.append(codec.add_offset(v, 128.0, want_u8=True)[1].clone())
        assert torch.equal(f[0], f[1]) and torch.equal(f[0].view(-1), got.view(-1))
        assert torch.equal(bytes_of[0], bytes_of[1])
    y = codec.analyze(model, torch.from_numpy(img).cuda(), ws, want_y=True)[1]
    tiles = _tiles(lambda: codec.synthesize(codec.Model(cfg, pack_weights(cfg, make_weights(cfg))), ws, y=y)[0])
    x = codec.synthesize(model, ws, y=y)[0]
    assert torch.equal(x, tiles) != split
    assert float((x - tiles).abs().max()) <= 1e-3


@pytest.mark.gpu
def test_fp32_synthesis_keeps_fp32_infinities():
    """Opposite infinities in one 3 x 3 neighbourhood: the filters of a model without the option give NaN
    there, as an FP32 sum does, and a lone infinity saturates."""
    need_gpu()
    from paper_2405_12631_amd import codec
    say("infinities")
    cfg = get_config("ycbcr512x768")
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)))
    H, W = 96, 160
    ws = codec.Workspace(model, 2, H, W)
    y = torch.from_numpy(np.random.default_rng(8).normal(0, 20, (2, H * W)).astype(np.float32)).cuda()
    at = ws.lay[-2]["offset"] + 20 * ws.lay[-2]["w"] + 30          # LH of level 1
    y[0, at], y[0, at + 1] = float("inf"), -float("inf")
    y[1, at] = float("inf")
    x = codec.synthesize(model, ws, y=y)[0]
    old = _tiles(lambda: codec.synthesize(model, ws, y=y)[0])
    assert torch.equal(torch.isnan(x), torch.isnan(old)) and bool(torch.isnan(old[0]).any())
    assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(old))
