"""Timed work of the decode framework: what its users have it do, by size, direction and data type.

A case is one call, or the sequence of calls, of a user's program:

* tables  - CDF tables of one coding step's parameters;
* synth   - dequantisation and inverse lifting of planes, or of a GOP's temporal subbands
            followed by the inverse temporal Haar transform and the offset;
* analyze - lifting and quantisation of 8-bit planes (encoder side);
* decode  - coder-elided decode of one image: every (subband, step)'s parameters, tables and
            symbol scatter, then synthesis; eager, or replayed as one library graph;
* batch   - the same for images of uneven size through one plan;
* serve   - the continuous-batching server over staggered requests;
* stream  - a whole encode or decode through the host entropy coder.

Inputs are three-plane images with a 1/f spectrum and noise, made on the GPU from the seed;
symbols come from a 64-bit evaluation of the analysis transform, which `exact` shares.
"""
import functools
import math

import numpy as np
import torch

from paper_2405_12631_amd import WV_BF16, WV_FP32, WV_FP8, batch, codec, serve

_DEV = "cuda"
_PRECISION = {"fp32": WV_FP32, "bf16": WV_BF16, "fp8": WV_FP8}

# The repository's two model sizes: the small 64 x 64 grayscale model, and the model of the
# 512 x 768 image, the mixed-size batch and the server.
_BASE = dict(lift_layers=3, mix_k=3, dist="gauss", ctx_arch="plain", ll_ar=0, ar_ch=32, sym_min=-64,
             sym_max=64, cdf_bits=16, sigma_min=0.11, lift_int=0)
_MODELS = {
    "small": dict(_BASE, levels=2, lift_ch=16, ctx_ch=32, ctx_layers=3, step=8.0),
    "large": dict(_BASE, levels=4, lift_ch=32, ctx_ch=64, ctx_layers=4, step=4.0),
}
# Image sizes of the mixed-size batch and of the server's stills.
_SIZES = ((256, 256), (512, 768), (1024, 1024), (1088, 1920))
_PLANES = 3
_GOP = 8


def listed():
    return [
        # One coding step of an image's coarsest subband: the smallest table launch of a decode.
        {"name": "tables_small", "kind": "tables", "rows": 1152, "k": 3, "dist": "gauss"},
        # A level-1 coding step of a batch of images.
        {"name": "tables_batch", "kind": "tables", "rows": 2_400_000, "k": 3, "dist": "gauss"},
        # Inverse transform of one three-plane image.
        {"name": "synth_image", "kind": "synth", "h": 512, "w": 768, "planes": 3, "gop": False},
        # Inverse transform of the luma planes of a video GOP, with the temporal transform.
        {"name": "synth_gop", "kind": "synth", "h": 1088, "w": 1920, "planes": _GOP, "gop": True},
        # Encoder side of one three-plane image.
        {"name": "analyze_image", "kind": "analyze", "h": 512, "w": 768, "planes": 3},
        # The smallest whole decode, call by call: launches and latency.
        {"name": "decode_small", "kind": "decode", "model": "small", "h": 64, "w": 64, "planes": 1,
         "precision": "fp32", "graph": False},
        # One image at each precision, the decode captured once and replayed.
        {"name": "decode_fp32", "kind": "decode", "model": "large", "h": 512, "w": 768, "planes": 3,
         "precision": "fp32", "graph": True},
        {"name": "decode_bf16", "kind": "decode", "model": "large", "h": 512, "w": 768, "planes": 3,
         "precision": "bf16", "graph": True},
        {"name": "decode_fp8", "kind": "decode", "model": "large", "h": 512, "w": 768, "planes": 3,
         "precision": "fp8", "graph": True},
        # A batch of images of uneven size in one plan.
        {"name": "batch_bf16", "kind": "batch", "images": 12, "pick": 8, "precision": "bf16"},
        # Requests of uneven size that join and leave a running server.
        {"name": "serve_bf16", "kind": "serve", "images": 5, "gops": 1, "pick": 4, "gap": 3, "precision": "bf16"},
        # A bitstream in, pixels out, through the host entropy coder.
        {"name": "stream_decode", "kind": "stream", "h": 512, "w": 768, "planes": 3, "precision": "bf16",
         "encode": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi, unit=16):
    """An image side: any multiple of `unit` (2^levels), so odd subbands are as likely as even ones."""
    return unit * max(1, _log_int(rng, lo / unit, hi / unit))


def draw(rng):
    kind = rng.choice(("tables", "synth", "analyze", "decode", "decode", "batch", "serve", "stream"))
    if kind == "tables":
        k, dist = rng.choice(((3, "gauss"), (3, "gauss"), (2, "gauss"), (1, "laplace")))
        return {"kind": kind, "rows": _log_int(rng, 300, 2_400_000), "k": k, "dist": dist}
    if kind == "synth":
        if rng.random() < 0.3:
            return {"kind": kind, "h": _side(rng, 272, 1088), "w": _side(rng, 480, 1920), "planes": _GOP, "gop": True}
        return {"kind": kind, "h": _side(rng, 64, 1088), "w": _side(rng, 64, 1920), "planes": rng.choice((1, 3, 6)),
                "gop": False}
    if kind == "analyze":
        return {"kind": kind, "h": _side(rng, 64, 1088), "w": _side(rng, 64, 1920), "planes": rng.choice((1, 3))}
    if kind == "decode":
        if rng.random() < 0.2:
            return {"kind": kind, "model": "small", "h": _side(rng, 16, 128, 4), "w": _side(rng, 16, 128, 4),
                    "planes": rng.choice((1, 2, 3)), "precision": "fp32", "graph": False}
        return {"kind": kind, "model": "large", "h": _side(rng, 96, 1024), "w": _side(rng, 96, 1024),
                "planes": rng.choice((1, 3, 3)), "precision": rng.choice(("fp32", "bf16", "bf16", "fp8")),
                "graph": rng.random() < 0.5}
    if kind in ("batch", "serve"):
        case = {"kind": kind, "images": rng.randint(2, 10 if kind == "batch" else 5), "pick": rng.randrange(1 << 20),
                "precision": rng.choice(("bf16", "bf16", "fp8")) if kind == "batch" else "bf16"}
        if kind == "serve":
            case.update(gops=rng.randint(0, 1), gap=rng.randint(0, 8))
        most = max(work(c)["flops"] for c in listed())
        while work(case)["flops"] > most:
            case["images"] -= 1
        return case
    return {"kind": "stream", "h": _side(rng, 96, 512), "w": _side(rng, 96, 768), "planes": rng.choice((1, 3)),
            "precision": rng.choice(("fp32", "bf16")), "encode": rng.random() < 0.5}


# ---------------------------------------------------------------------------
# weights and models
# ---------------------------------------------------------------------------
def _config(case):
    cfg = dict(_MODELS[case.get("model", "large")])
    if case["kind"] == "tables":
        cfg.update(mix_k=case["k"], dist=case["dist"])
    return cfg


@functools.lru_cache(maxsize=None)
def _weights_of(key):
    """Random-init tensors in blob order: each conv's weight [Cout][Cin][3][3] and bias [Cout]."""
    cfg = dict(key)
    rng = np.random.default_rng(0)
    out = {}

    def conv(name, cin, cout):
        bound = 1.0 / math.sqrt(9.0 * cin)
        out[name] = (rng.uniform(-bound, bound, (cout, cin, 3, 3)).astype(np.float32),
                     rng.uniform(-bound, bound, cout).astype(np.float32))

    c, n = cfg["lift_ch"], cfg["lift_layers"]
    for f in ("P_row", "U_row", "P_col", "U_col"):
        for i, (a, b) in enumerate(zip([1] + [c] * (n - 1), [c] * (n - 1) + [1])):
            conv((f, i), a, b)
    c, n = cfg["ctx_ch"], cfg["ctx_layers"]
    conv("lstm", 1 + c, 4 * c)
    for t in range(4):
        for g in range(4):
            first = c if g == 0 else c + 1
            for i, (a, b) in enumerate(zip([first] + [c] * (n - 1), [c] * (n - 1) + [3 * cfg["mix_k"]])):
                conv((t, g, i), a, b)
    return out


def _weights(cfg):
    return _weights_of(tuple(sorted(cfg.items())))


@functools.lru_cache(maxsize=None)
def _model_of(key, precision):
    cfg = dict(key)
    blob = np.concatenate([np.concatenate([w.ravel(), b]) for w, b in _weights_of(key).values()])
    return codec.Model(cfg, blob, precision=_PRECISION[precision])


def _model(cfg, precision="fp32"):
    """The model handle a program makes once and keeps."""
    return _model_of(tuple(sorted(cfg.items())), precision)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, salt=0):
    g = torch.Generator(device=_DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _texture(h, w, gen, shift=0.0, wave=None):
    """A sum of random sinusoids with a 1/f spectrum, 64-bit [h][w], and its waves."""
    if wave is None:
        u = torch.rand(3, 256, generator=gen, device=_DEV, dtype=torch.float64)
        f = torch.exp(math.log(1.0 / max(h, w)) + u[0] * math.log(0.5 * max(h, w)))
        ang = math.pi * u[1]
        wave = (2 * math.pi * f * torch.cos(ang), 2 * math.pi * f * torch.sin(ang), 2 * math.pi * u[2], 1.0 / f)
    ax, ay, phase, amp = wave
    x = torch.arange(w, device=_DEV, dtype=torch.float64)[:, None] + shift
    y = torch.arange(h, device=_DEV, dtype=torch.float64)[:, None]
    cx, sx = torch.cos(x * ax + phase) * amp, torch.sin(x * ax + phase) * amp
    return torch.cos(y * ay) @ cx.T - torch.sin(y * ay) @ sx.T, wave


def _to_u8(v, gen):
    v = 128.0 + v + 5.0 * torch.randn(v.shape, generator=gen, device=_DEV, dtype=torch.float64)
    return v.round().clamp(0, 255).to(torch.uint8)


def _image(h, w, planes, seed, salt=0):
    """uint8 planes [planes][h][w]: luma contrast first, weaker chroma after it."""
    gen = _gen(seed, salt)
    out = torch.empty((planes, h, w), dtype=torch.uint8, device=_DEV)
    for p in range(planes):
        t, _ = _texture(h, w, gen)
        out[p] = _to_u8((t - t.mean()) * ((40.0, 20.0, 20.0)[p % 3] / t.std()), gen)
    return out


def _frames(h, w, seed, salt=0, std=40.0, shift=2.0):
    """uint8 frames [T][h][w] of a texture that moves to the left."""
    gen = _gen(seed, salt)
    base, wave = _texture(h, w, gen)
    mean, scale = base.mean(), std / base.std()
    return torch.stack([_to_u8((_texture(h, w, gen, shift * t, wave)[0] - mean) * scale, gen) for t in range(_GOP)])


def _picked(case):
    rng = np.random.default_rng(case["pick"])
    return [_SIZES[i] for i in rng.integers(0, len(_SIZES), case["images"])]


# ---------------------------------------------------------------------------
# the method in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _conv(x, wb):
    """3 x 3 convolution with zero padding, [n][h][w][cin] -> [n][h][w][cout]."""
    w, b = (torch.from_numpy(t).to(x.device, torch.float64) for t in wb)
    n, h, wd, cin = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    out = b.expand(n, h, wd, -1).clone()
    for dy in range(3):
        for dx in range(3):
            s = p[:, dy:dy + h, dx:dx + wd]
            if cin == 1:
                out += s * w[:, 0, dy, dx]
            else:
                out += (s.reshape(-1, cin) @ w[:, :, dy, dx].T).view(n, h, wd, -1)
    return out


def _filter(z, weights, name):
    out = torch.empty_like(z)
    for k in range(z.shape[0]):                # plane by plane: the channel maps are large in 64 bits
        a = z[k:k + 1, :, :, None]
        a = torch.tanh_(_conv(a, weights[(name, 0)]))
        a = torch.tanh_(_conv(a, weights[(name, 1)]))
        out[k] = _conv(a, weights[(name, 2)])[0, :, :, 0]
    return out


def _split(x, axis, weights, suffix):
    e, o = (x[:, :, 0::2], x[:, :, 1::2]) if axis == 2 else (x[:, 0::2], x[:, 1::2])
    hp = o - (e + _filter(e, weights, "P_" + suffix))
    return e + 0.5 * hp + _filter(hp, weights, "U_" + suffix), hp


def _merge(lp, hp, axis, weights, suffix):
    e = lp - (0.5 * hp + _filter(hp, weights, "U_" + suffix))
    o = hp + (e + _filter(e, weights, "P_" + suffix))
    return torch.stack((e, o), 3 if axis == 2 else 2).reshape(
        (e.shape[0], e.shape[1], -1) if axis == 2 else (e.shape[0], -1, e.shape[2]))


def _analysis(x, cfg):
    """Centred 64-bit planes -> subbands in coding order."""
    weights, details = _weights(cfg), []
    for _ in range(cfg["levels"]):
        lo, hi = _split(x, 2, weights, "row")
        x, lh = _split(lo, 1, weights, "col")
        hl, hh = _split(hi, 1, weights, "col")
        details.append((hl, lh, hh))
    return [x] + [s for d in reversed(details) for s in d]


def _synthesis(ys, cfg):
    weights, x = _weights(cfg), ys[0]
    for j in range(cfg["levels"]):
        hl, lh, hh = ys[1 + 3 * j:4 + 3 * j]
        x = _merge(_merge(x, lh, 1, weights, "col"), _merge(hl, hh, 1, weights, "col"), 2, weights, "row")
    return x


def _symbols(x, cfg):
    """Quantised subbands of centred 64-bit planes, and their packed int16 form."""
    qs = [(y / cfg["step"]).round().clamp(cfg["sym_min"], cfg["sym_max"]) for y in _analysis(x, cfg)]
    return qs, torch.cat([q.reshape(q.shape[0], -1) for q in qs], 1).to(torch.int16).contiguous()


def _haar(f, inverse):
    """Temporal Haar lifting of [T][...], in the order L, H, H, H, H, ... of the framework."""
    if inverse:
        n = 1
        while n < f.shape[0]:
            lo, hi = f[:n], f[n:2 * n]
            e = lo - 0.5 * hi
            f = torch.cat((torch.stack((e, hi + e), 1).reshape(2 * n, *f.shape[1:]), f[2 * n:]))
            n *= 2
        return f
    n = f.shape[0]
    f = f.clone()
    while n > 1:
        e, o = f[0:n:2].clone(), f[1:n:2].clone()
        f[n // 2:n] = o - e
        f[:n // 2] = e + 0.5 * (o - e)
        n //= 2
    return f


def _parameters(qs, cfg):
    """Mixture parameters of every (subband, step) in coding order, [planes][n][3K] each."""
    weights, k, layers = _weights(cfg), cfg["mix_k"], cfg["ctx_layers"]
    n, h, w = qs[0].shape
    hid = torch.zeros((n, h, w, cfg["ctx_ch"]), device=_DEV, dtype=torch.float64)
    cell, before, out = hid, torch.zeros_like(qs[0]), []
    up = lambda a: a.repeat_interleave(2, 1).repeat_interleave(2, 2)  # noqa: E731
    for i, q in enumerate(qs):
        h, w = q.shape[1:]
        if hid.shape[1] != h:
            hid, cell, before = up(hid), up(cell), up(before)
        gi, gf, gc, go = _conv(torch.cat((before[..., None], hid), 3), weights["lstm"]).chunk(4, 3)
        cell = torch.sigmoid(gf) * cell + torch.sigmoid(gi) * torch.tanh(gc)
        hid = torch.sigmoid(go) * torch.tanh(cell)
        step_of = 2 * (torch.arange(h, device=_DEV) % 2)[:, None] + (torch.arange(w, device=_DEV) % 2)
        for g in range(4):
            a = hid if g == 0 else torch.cat((torch.where(step_of < g, q, 0.0)[..., None], hid), 3)
            for layer in range(layers):
                a = _conv(a, weights[(0 if i == 0 else 1 + (i - 1) % 3, g, layer)])
                a = a if layer + 1 == layers else torch.relu_(a)
            a = a[:, g // 2::2, g % 2::2].reshape(n, -1, 3 * k)
            sig = torch.nn.functional.softplus(a[..., 2 * k:], threshold=700).clamp_min(cfg["sigma_min"])
            out.append(torch.cat((torch.softmax(a[..., :k], 2), a[..., k:2 * k], sig), 2))
        before = q
    return out


# ---------------------------------------------------------------------------
# states
# ---------------------------------------------------------------------------
def _mixtures(case, seed):
    """Parameters [rows][3K] as decodes meet them: narrow and wide scales, means around zero."""
    gen, n, k = _gen(seed), case["rows"], case["k"]
    w = torch.softmax(torch.randn(n, k, generator=gen, device=_DEV), 1)
    mu = torch.randn(n, k, generator=gen, device=_DEV) * torch.exp(torch.randn(n, 1, generator=gen, device=_DEV))
    sig = torch.exp(0.9 * torch.randn(n, k, generator=gen, device=_DEV)).clamp_min(0.11)
    return torch.cat((w, mu, sig), 1).float().contiguous()


def _planes(case, seed):
    """Centred 64-bit planes of a synth case: an image, or a GOP's temporal subbands."""
    if case["gop"]:
        return _haar(_frames(case["h"], case["w"], seed).double() - 128.0, inverse=False)
    return _image(case["h"], case["w"], case["planes"], seed).double() - 128.0


class _Decode:
    """A coder-elided decode of one set of planes whose steps keep their parameters and tables."""

    def __init__(self, model, q_known, n, h, w):
        self.model = model
        self.ws = codec.Workspace(model, n, h, w)
        self.syms = codec.prepare_elided(model, q_known, self.ws)
        self.q = torch.zeros_like(q_known)
        self.xhat = torch.empty((n, h, w), dtype=torch.float32, device=_DEV)
        rows = [[s.numel() for s in row] for row in self.syms]
        k3, total = 3 * model.cfg["mix_k"], sum(map(sum, rows))
        self.params = torch.empty(total * k3, dtype=torch.float32, device=_DEV)
        self.tables = torch.empty(total * (model.nsym + 1), dtype=torch.int16, device=_DEV)
        self.at, a = [], 0
        for row in rows:
            self.at.append([])
            for n_rows in row:
                self.at[-1].append((self.params[a * k3:(a + n_rows) * k3],
                                    self.tables[a * (model.nsym + 1):(a + n_rows) * (model.nsym + 1)]))
                a += n_rows
        self.graph = None

    def step(self):
        m, ws = self.model, self.ws
        codec.zero(self.q)
        for i in range(len(ws.lay)):
            for g in range(4):
                prm, tab = self.at[i][g]
                codec.cdf_tables(m, codec.context_params(m, self.q, ws, i, g, out=prm), out=tab)
                codec.scatter_symbols(m, self.syms[i][g], self.q, ws, i, g)
        codec.synthesize(m, ws, q=self.q, xhat=self.xhat)

    def run(self):
        if self.graph is None:
            self.step()
        else:
            self.graph.replay()
        return {"params": self.params, "tables": self.tables, "q": self.q, "xhat": self.xhat}


def prepare(case, seed):
    kind, cfg = case["kind"], _config(case)
    if kind == "tables":
        model = _model(cfg)
        return dict(case, m=model, params=_mixtures(case, seed),
                    out=torch.empty(case["rows"] * (model.nsym + 1), dtype=torch.int16, device=_DEV))
    if kind == "synth":
        n, h, w = case["planes"], case["h"], case["w"]
        model = _model(cfg)
        return dict(case, m=model, q=_symbols(_planes(case, seed), cfg)[1],
                    ws=codec.Workspace(model, n, h, w, coder=False, step_buffers=False),
                    xhat=torch.empty((n, h, w), dtype=torch.float32, device=_DEV))
    if kind == "analyze":
        n, h, w = case["planes"], case["h"], case["w"]
        model = _model(cfg)
        return dict(case, m=model, x=_image(h, w, n, seed),
                    ws=codec.Workspace(model, n, h, w, coder=False, step_buffers=False))
    if kind == "decode":
        n, h, w = case["planes"], case["h"], case["w"]
        d = _Decode(_model(cfg, case["precision"]), _symbols(_image(h, w, n, seed).double() - 128.0, cfg)[1], n, h, w)
        if case["graph"]:
            d.step()
            torch.cuda.synchronize()
            d.graph = codec.Graph(d.step)
        return dict(case, d=d)
    if kind == "batch":
        sizes = _picked(case)
        bt = batch.Batch(_model(cfg, case["precision"]), sizes, planes=_PLANES)
        for k, (b, p0) in enumerate(bt.where):
            x = _image(*sizes[k], _PLANES, seed, salt=k).double() - 128.0
            bt.q[b][p0:p0 + _PLANES] = _symbols(x, cfg)[1]
        syms, row = bt.known_symbols(), bt.model.nsym + 1
        tables = torch.empty(sum(s.numel() for r in syms for s in r) * row, dtype=torch.int16, device=_DEV)
        at, a = [], 0
        for r in syms:
            at.append([])
            for s in r:
                at[-1].append(tables[a * row:(a + s.numel()) * row])
                a += s.numel()
        return dict(case, bt=bt, syms=syms, tables=tables, at=at)
    if kind == "serve":
        model = _model(cfg, case["precision"])
        preps, reqs = {}, []
        for k, (h, w) in enumerate(_picked(case)):
            preps[k] = serve.Prepared(model, "image", _image(h, w, _PLANES, seed, salt=k).cpu().numpy())
        for k in range(case["gops"]):
            luma = _frames(544, 960, seed, salt=100 + k)
            chroma = [_frames(272, 480, seed, salt=200 + 2 * k + c, std=20.0, shift=1.0) for c in range(2)]
            preps[len(preps)] = serve.Prepared(model, "gop",
                                               (luma.cpu().numpy(), torch.stack(chroma, 1).cpu().numpy()))
        reqs = [(float(case["gap"] * k), k) for k in range(len(preps))]
        budget = sum(serve.footprint(model, p) for p in preps.values())
        return dict(case, srv=serve.Server(model, budget), preps=preps, reqs=reqs)
    if kind == "stream":
        n, h, w = case["planes"], case["h"], case["w"]
        model = _model(cfg, case["precision"])
        ws, x = codec.Workspace(model, n, h, w), _image(h, w, n, seed)
        return dict(case, m=model, ws=ws, x=x, data=None if case["encode"] else codec.encode(model, x, ws)[0])
    raise ValueError(kind)


def run(s):
    kind = s["kind"]
    if kind == "tables":
        return codec.cdf_tables(s["m"], s["params"], out=s["out"])
    if kind == "synth":
        xhat, _ = codec.synthesize(s["m"], s["ws"], q=s["q"], xhat=s["xhat"], offset=0.0 if s["gop"] else 128.0)
        if s["gop"]:
            codec.add_offset(codec.temporal_haar(xhat.view(_GOP, -1), inverse=True), 128.0)
        return xhat
    if kind == "analyze":
        q, y, clip = codec.analyze(s["m"], s["x"], s["ws"], want_y=True)
        return {"q": q, "y": y, "clip": clip}
    if kind == "decode":
        return s["d"].run()
    if kind == "batch":
        bt = s["bt"]
        for q in bt.q:
            codec.zero(q)
        for i in range(bt.nsub):
            for g in range(4):
                codec.cdf_tables(bt.model, bt.context_params(i, g), out=s["at"][i][g])
                bt.scatter(s["syms"][i][g], i, g)
        return {"tables": s["tables"], "q": bt.q, "xhat": bt.synthesize()}
    if kind == "serve":
        _, done = s["srv"].run(s["reqs"], s["preps"], max_seconds=1e9, keep_outputs=True, tick=1.0)
        return [slot.xhat for slot in sorted(done, key=lambda d: d.req["prep"])]
    if kind == "stream":
        if s["encode"]:
            data, q = codec.encode(s["m"], s["x"], s["ws"])
            return {"stream": np.frombuffer(data, np.uint8), "q": q}
        xhat, u8, q = codec.decode(s["m"], s["data"], s["ws"])
        return {"xhat": xhat, "u8": u8, "q": q}
    raise ValueError(kind)


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its values in 64 bits
# ---------------------------------------------------------------------------
def _lift_flops(cfg):
    """Per pixel of a plane: two predict and two update filters per level, on half-size arrays."""
    c = cfg["lift_ch"]
    return 2.0 * sum(4.0 ** -j for j in range(cfg["levels"])) * 2 * 9 * (c * c + 2 * c)


def _context_flops(cfg):
    """Per coefficient: the ConvLSTM and four stacks, each head at its quarter of the positions."""
    c, n, k = cfg["ctx_ch"], cfg["ctx_layers"], cfg["mix_k"]
    return 2.0 * 9 * ((1 + c) * 4 * c + sum((c + (g > 0)) * c + (n - 2) * c * c + c * 3 * k / 4 for g in range(4)))


def work(case):
    cfg = _config(case)
    k3, row = 3 * cfg["mix_k"], 2 * (cfg["sym_max"] - cfg["sym_min"] + 2)
    if case["kind"] == "tables":
        return {"bytes": case["rows"] * (4 * k3 + row), "flops": case["rows"] * 128 * cfg["mix_k"] * 4}
    if case["kind"] in ("batch", "serve"):
        n = _PLANES * sum(h * w for h, w in _picked(case)) + case.get("gops", 0) * _GOP * 544 * 960 * 3 // 2
    else:
        n = case["planes"] * case["h"] * case["w"]
    lift, ctx = n * _lift_flops(cfg), n * _context_flops(cfg)
    if case["kind"] == "synth":
        return {"bytes": n * 6, "flops": lift}
    if case["kind"] == "analyze":
        return {"bytes": n * 7, "flops": lift}
    if case["kind"] == "decode":    # symbols in; parameters, tables, symbols and pixels out
        return {"bytes": n * (1 + 4 * k3 + row + 2 + 4), "flops": lift + ctx}
    if case["kind"] == "batch":
        return {"bytes": n * (1 + row + 2 + 4), "flops": lift + ctx}
    if case["kind"] == "serve":
        return {"bytes": n * (1 + 4), "flops": lift + ctx}
    # about a byte of stream per symbol, and symbols or pixels on the other side
    return {"bytes": n * (1 + (1 if case["encode"] else 7)), "flops": lift + ctx}


def exact(case, seed):
    kind, cfg = case["kind"], _config(case)
    if kind == "synth":
        qs, _ = _symbols(_planes(case, seed), cfg)
        x = _synthesis([q * cfg["step"] for q in qs], cfg)
        return _haar(x, inverse=True) + 128.0 if case["gop"] else x + 128.0
    if kind == "analyze":
        ys = _analysis(_image(case["h"], case["w"], case["planes"], seed).double() - 128.0, cfg)
        return {"q": None, "y": torch.cat([y.reshape(y.shape[0], -1) for y in ys], 1), "clip": None}
    if kind == "decode":
        qs, _ = _symbols(_image(case["h"], case["w"], case["planes"], seed).double() - 128.0, cfg)
        xhat = _synthesis([q * cfg["step"] for q in qs], cfg) + 128.0
        params = torch.cat([p.reshape(-1) for p in _parameters(qs, cfg)])
        return {"params": params, "tables": None, "q": None, "xhat": xhat}
    if kind == "batch":
        sizes = _picked(case)
        groups = sorted(set(sizes), key=lambda hw: (hw[0] * hw[1], hw))
        xhat = [[] for _ in groups]
        for k, hw in enumerate(sizes):
            qs, _ = _symbols(_image(*hw, _PLANES, seed, salt=k).double() - 128.0, cfg)
            xhat[groups.index(hw)].append(_synthesis([q * cfg["step"] for q in qs], cfg) + 128.0)
        return {"tables": None, "q": None, "xhat": [torch.cat(x) for x in xhat]}
    return None     # integer tables; and symbols that only the framework's own encoder has
