"""Decode-path benchmark: decoded Mpixel/s of the GPU decode path (context
model + CDF tables + inverse lifting), p50/p99 latency, against the plain FP32
batch-1 path, on one GPU.

Default line (the headline): one step = one coder-elided decode of a batch of
64 three-plane images of uneven size (256x256, 512x768, 1024x1024, 1088x1920;
seed 3) with BF16 context convs: for each of the 13 subbands x 4 coding steps
one persistent launch over all images (the fused ConvLSTM at step 0, then the
fused step stack), the CDF tables of the step in one launch, the scatter of
that step's symbols (the symbols the host entropy coder would return are taken
from a device buffer), then synthesis; the whole decode replayed as one library
graph.  In the same process the plain FP32 batch-1 decode of the 512x768x3
image is measured the same way; vs_baseline = headline Mpixel/s / FP32
batch-1 Mpixel/s, and the FP32 line is nested as "baseline".  Inputs are
resident in HBM before timing.

    python bench.py [--steps K] [--warmup W] [--gpus 1] [--no-cpu-baseline]
                    [--precision fp32|bf16|fp8] [--nb-table 4,4,4,4]
                    [--workload headline|ycbcr512x768|batch64_mixed|serve_mix|
                                precision_report|coder512x768|hbm_copy]

--workload ycbcr512x768 prints the single-image line alone (FP32 unless
--precision), batch64_mixed the batch line alone; the layer-by-layer batch
forms (FP32, FP8, or WV_FUSED_STACKS=0) autotune their per-level channel
blocking before timing, and --nb-table fixes it (e.g. for a profiled run);
serve_mix runs the continuous-batching server under Poisson arrivals.

Prints one JSON line.
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

MFMA_PEAK_TFLOPS = {"fp32": 157.3, "bf16": 2500.0, "fp8": 5000.0}   # MI355X dense matrix peaks


# HBM bytes per context-conv launch from rocprofv3 FETCH_SIZE (x2.0) + WRITE_SIZE (x1.0), the
# factors being what each counter reads for a plain 1 GiB device copy; averaged over the 1326
# launches of six 512x768x3 decodes.  Valid only for the conv sources with these sha256.
TRAFFIC_SOURCES = {
    "paper_2405_12631_amd/csrc/wv_conv.hip": "3fc89fb6b86d2d4efabb039bf86840ce15ce9481e614399f23447f9a4011711b",
    "paper_2405_12631_amd/csrc/wv_conv_bf16.hip": "7e90ca9845574eceaa8be27cb403b1f0156b7cdfcea5dd8d6f6e3db5bfd68c14",
    "paper_2405_12631_amd/csrc/wv_device.h": "c8c3694e4ccee0d22f312951ebc1e3ddd60dff1757976d01528bb82a2e91748a",
    "paper_2405_12631_amd/csrc/wv_internal.h": "d6f1ee1d02aa4339f944aea57359f82c664966a2c22e65a3cfbcf8a114500b6c",
}
TRAFFIC_BYTES_PER_LAUNCH = {"fp32": 49.33e6, "bf16": 25.69e6, "fp8": 15.02e6}


def measured_traffic(precision):
    """Counter-measured HBM bytes per context-conv launch, or None if the kernels changed since."""
    import hashlib
    root = os.path.dirname(os.path.abspath(__file__))
    for rel, digest in TRAFFIC_SOURCES.items():
        try:
            with open(os.path.join(root, rel), "rb") as f:
                if hashlib.sha256(f.read()).hexdigest() != digest:
                    return None
        except OSError:
            return None
    return TRAFFIC_BYTES_PER_LAUNCH.get(precision)


# HBM bytes per launch of the fused step-stack kernel (steps 1-3) in the 64-image batch, from
# rocprofv3 FETCH_SIZE (x2.0) + WRITE_SIZE (x1.0), the factors being what each counter reads for a
# plain 1 GiB device copy; averaged over the 117 launches of three batch decodes.  The halo re-reads
# depend on the row pieces the library cuts (wv_pieces.h) as well as on the kernel, so the figure is
# valid only for both sources with these sha256 (else the line reports null).
STACK_TRAFFIC_SOURCES = {
    "paper_2405_12631_amd/csrc/wv_stack_bf16.hip": "51bef7e1657c03f772704f51e3272123a574ba832fbce100566b8184f3ad9a52",
    "paper_2405_12631_amd/csrc/wv_pieces.h": "0d54396e383a18cad9ef2cd634574bb352615ce1377f2c913d204376e22ba1ae",
}
STACK_TRAFFIC_BYTES_PER_LAUNCH = 1898.5e6


def measured_stack_traffic(args):
    import hashlib
    if args.precision != "bf16":
        return None
    for rel, digest in STACK_TRAFFIC_SOURCES.items():
        try:
            with open(os.path.join(ROOT, rel), "rb") as f:
                if hashlib.sha256(f.read()).hexdigest() != digest:
                    return None
        except OSError:
            return None
    return STACK_TRAFFIC_BYTES_PER_LAUNCH


def _precision(name):
    from paper_2405_12631_amd import WV_BF16, WV_FP32, WV_FP8
    return {"fp32": WV_FP32, "bf16": WV_BF16, "fp8": WV_FP8}[name]
HBM_PEAK_GBS = 8000.0


def context_flops_per_coef(cfg):
    """Algorithmic FLOPs of the context model per coefficient (all 4 steps).

    ConvLSTM: 9 (1 + C) 4C MACs at every position.  Step stacks: every layer
    but the last at all positions, the 3K-output head at the quarter of
    positions its step codes: sum_g [9 Cin_g C + (L - 2) 9 C^2 + 9 C 3K / 4].
    """
    C, Lc, K = cfg["ctx_ch"], cfg["ctx_layers"], cfg["mix_k"]
    lstm = 9 * (1 + C) * 4 * C
    stacks = 0
    for g in range(4):
        cin = C if g == 0 else C + 1
        stacks += 9 * cin * C + (Lc - 2) * 9 * C * C + 9 * C * 3 * K / 4.0
    return 2.0 * (lstm + stacks)


def stack_flops_per_coef(cfg, step):
    """Algorithmic FLOPs of one coding step's conv stack per coefficient of the subband: every
    layer but the head at all positions (the first with the symbol channel for step >= 1),
    the 3K-output head at the quarter of positions the step codes."""
    C, Lc, K = cfg["ctx_ch"], cfg["ctx_layers"], cfg["mix_k"]
    cin = C if step == 0 else C + 1
    return 2.0 * (9 * cin * C + (Lc - 2) * 9 * C * C + 9 * C * 3 * K / 4.0)


def lifting_cost_per_px(cfg):
    """Algorithmic FLOPs and HBM bytes of synthesis per pixel of one plane.

    Each predict/update application costs 9 (C^2 + 2 C) MACs per position and
    reads its filter input and the array it updates and writes the result
    (12 bytes).  Level j runs 2 (H/2^(j-1)) (W/2^(j-1)) applications: four over
    the quarter-size column pairs, two over the half-size row arrays.  Add the
    dequantisation (2 B in, 4 B out) and the final 8-bit rounding (4 B in, 1 B out).
    """
    C, J = cfg["lift_ch"], cfg["levels"]
    apps = 2.0 * sum(4.0 ** -j for j in range(J))
    return apps * 2.0 * 9 * (C * C + 2 * C), apps * 12.0 + 6.0 + 5.0


def cdf_bytes_per_row(cfg):
    """Algorithmic HBM bytes per CDF row: 3K float parameters in, one uint16 table out."""
    return 12.0 * cfg["mix_k"] + 2.0 * (cfg["sym_max"] - cfg["sym_min"] + 2)


def stage_rates(cfg, rows, px, cdf_ms, syn_ms):
    """Achieved algorithmic rates of the CDF and synthesis stages of one decode
    (CDF: one row per coefficient; synthesis: every pixel of every plane)."""
    cb = cdf_bytes_per_row(cfg) * rows
    lf, lb = lifting_cost_per_px(cfg)
    out = dict(cdf=dict(bound="hbm", bytes=cb, gb_per_s=round(cb / cdf_ms / 1e6, 1),
                        frac_hbm=round(cb / cdf_ms / 1e6 / HBM_PEAK_GBS, 4)),
               synthesis=dict(bound="mfma", flops=lf * px, tflop_per_s=round(lf * px / syn_ms / 1e9, 3),
                              frac_fp32_mfma=round(lf * px / syn_ms / 1e9 / MFMA_PEAK_TFLOPS["fp32"], 4),
                              bytes=lb * px, gb_per_s=round(lb * px / syn_ms / 1e6, 1)))
    return out


def _blas_threads():
    try:
        from threadpoolctl import threadpool_info
        return max([t.get("num_threads", 1) for t in threadpool_info()] + [1])
    except Exception:
        return os.cpu_count()


def cpu_baseline(cfg, w, q_planes, H, W):
    """The FP64 oracle's decode path (context model of every step, CDF tables, synthesis;
    symbols teacher-forced like the GPU's coder-elided decode) on a bounded sample: the
    three planes of one H x W image with every BLAS thread, and plane 0 alone on one
    thread.  Mpixel/s counts the image's H x W pixels once per image decode."""
    import oracle as O
    from threadpoolctl import threadpool_limits
    qs = O.unpack(q_planes, cfg, H, W)
    threads = _blas_threads()
    t0 = time.perf_counter()
    O.decode_path(qs, cfg, w)
    dt = time.perf_counter() - t0
    q1 = [q[:1] for q in qs]
    with threadpool_limits(1):
        t0 = time.perf_counter()
        O.decode_path(q1, cfg, w)
        dt1 = time.perf_counter() - t0
    nplanes = q_planes.shape[0]
    return dict(value=round(H * W / dt / 1e6, 6), unit="Mpixel/s", cores=int(threads), kind="oracle",
                seconds=round(dt, 3), nproc=os.cpu_count(), blas_threads=int(threads),
                one_core=dict(value=round(H * W / (dt1 * nplanes) / 1e6, 6), seconds_plane0=round(dt1, 3),
                              cores=1),
                sample=f"one {H}x{W}x{nplanes} image of the workload: context model of all 52 steps, CDF "
                       "tables and synthesis in float64 (teacher-forced symbols), all BLAS threads; "
                       "one_core: plane 0 of it on one thread, scaled to the image's planes")


def bench_batch(args):
    """Mixed-size batch: 64 three-plane images from four sizes (seed 3), reduced-precision
    context convs, one plan (persistent launches), the whole decode captured as one library
    graph; the layer-by-layer forms' per-level blocking autotuned before timing (or fixed by
    --nb-table), the fused BF16 kernels have none.  One step =
    one graph replay = one coder-elided decode of all 64 images.  Returns the line's dict,
    and the batch and one 256x256 image's symbols for the CPU baseline."""
    import torch
    from paper_2405_12631_amd import batch as B, codec
    from wvgen import batch_sizes, get_config, make_weights, pack_weights, sinusoid_1f_planes

    cfg = get_config("batch64_mixed")
    prec = _precision(args.precision)
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision=prec)
    sizes, seeds = batch_sizes(cfg["batch"], cfg["sizes"], seed=cfg["seed_image"])
    images = [sinusoid_1f_planes(h, w, planes=3, seed=sd) for (h, w), sd in zip(sizes, seeds)]
    bt = B.Batch(model, sizes)
    bt.load_images(images)
    del images
    syms = bt.known_symbols()
    log = (lambda m: print(m, file=sys.stderr, flush=True))
    # BF16 plans run the fused ConvLSTM and step-stack kernels, which have no channel blocking.
    fused = args.precision == "bf16" and os.environ.get("WV_FUSED_STACKS", "1") != "0"
    if args.nb_table:
        tab = [int(v) for v in args.nb_table.split(",")]
        bt.replan(tab)
    elif fused:
        tab = None
    else:
        tab, _ = B.autotune(bt, syms, reps=1, log=log)
    # Stage times from one eager decode, each context-model call bracketed by events on
    # the launch stream.
    stream = torch.cuda.current_stream()
    ev, ev_cdf = {}, []
    for q in bt.q:
        codec.zero(q)
    for i in range(bt.nsub):
        for g in range(4):
            e0, e1, e2 = (torch.cuda.Event(enable_timing=True) for _ in range(3))
            e0.record(stream)
            prm = bt.context_params(i, g)
            e1.record(stream)
            bt.cdf_tables(prm)
            e2.record(stream)
            ev[(i, g)] = (e0, e1)
            ev_cdf.append((e1, e2))
            bt.scatter(syms[i][g], i, g)
    es0, es1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    es0.record(stream)
    bt.synthesize()
    es1.record(stream)
    torch.cuda.synchronize()
    ctx_s = sum(a.elapsed_time(b) for a, b in ev.values()) * 1e-3
    # Steps 1-3 of every subband launch only the fused step-stack kernel (step 0 also runs the
    # ConvLSTM), so their event times are that kernel's launch times.
    stk_s = sum(a.elapsed_time(b) for (i, g), (a, b) in ev.items() if g > 0) * 1e-3
    cdf_s = sum(a.elapsed_time(b) for a, b in ev_cdf) * 1e-3
    syn_s = es0.elapsed_time(es1) * 1e-3
    known = [q.clone() for q in bt.q]
    graph = bt.capture(syms)
    for _ in range(args.warmup):
        graph.replay()
    torch.cuda.synchronize()
    lat = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        graph.replay()
        e1.record(stream)
        lat.append((e0, e1))
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    for b in range(len(bt.q)):
        assert torch.equal(bt.q[b], known[b]), "graph replay did not reproduce the symbols"
    lat = np.array([a.elapsed_time(b) for a, b in lat])
    pixels = bt.pixels
    mpx = pixels * args.steps / elapsed / 1e6
    flops = context_flops_per_coef(cfg) * pixels * 3
    stk_flops = sum(stack_flops_per_coef(cfg, g) for g in (1, 2, 3)) * pixels * 3
    peak = MFMA_PEAK_TFLOPS[args.precision]
    nlaunch = 3 * bt.nsub if fused else bt.nsub * (cfg["ctx_layers"] * 4 + 1)
    out = dict(
        metric="decoded Mpixel/s (ctx model+CDF+inverse lifting), p50/p99 latency vs plain FP32",
        value=round(mpx, 4), unit="Mpixel/s", n_gpus=1, steps=args.steps, warmup=args.warmup,
        ms_per_step=round(elapsed * 1e3 / args.steps, 3), higher_is_better=True, scaling="weak",
        vs_baseline=None,
        dtype=f"{args.precision} context convs (fp32 accumulate), fp32 lifting/cdf", data="synthetic",
        config=dict(workload=f"batch64_mixed: 64 three-plane images of uneven size, drawn from "
                             f"{[list(s_) for s_ in cfg['sizes']]} (seed 3), 1/f sinusoids + noise, 4-level "
                             f"CNN lifting (32 ch), 64-ch 4-layer context stacks, K=3 mixture, step 4, "
                             f"{args.precision.upper()} context convs, one plan (persistent launches) "
                             "replayed as one library graph, " +
                             ("fused ConvLSTM and step-stack kernels" if fused else f"channel blocking {tab}") +
                             ", coder elided",
                    batch=cfg["batch"], pixels=pixels, planes=3),
        p50_ms=round(float(np.percentile(lat, 50)), 3), p99_ms=round(float(np.percentile(lat, 99)), 3),
        launch="one wv_graph replay per batch decode (captured once); context time and roofline from an "
               "event-bracketed eager pass of the same decode",
        stage_ms=dict(context=round(ctx_s * 1e3, 3), step_stacks_1_3=round(stk_s * 1e3, 3),
                      cdf=round(cdf_s * 1e3, 3), synthesis=round(syn_s * 1e3, 3)),
        context_model=dict(tflop_per_s=round(flops / ctx_s / 1e12, 3), frac_of_peak=round(flops / ctx_s / 1e12 / peak, 4),
                           flops_per_decode=flops,
                           note="ConvLSTM + all step stacks, algorithmic FLOPs over the event-timed context calls"),
        roofline=dict(bound="mfma", achieved=round(stk_flops / stk_s / 1e12, 3), peak=peak, unit="TFLOP/s",
                      frac=round(stk_flops / stk_s / 1e12 / peak, 4), traffic=measured_stack_traffic(args),
                      traffic_unit="HBM bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
                      kernel=("stack_bf16_k<true> (fused step stacks of steps 1-3: three ReLU conv layers and "
                              "the mixture head per launch)") if fused else
                             "conv3x3_mfma_bf16_seg (step stacks of steps 1-3, layer by layer)",
                      flops_per_decode=stk_flops, launches_per_decode=nlaunch,
                      avg_launch_us=round(stk_s / nlaunch * 1e6, 2)),
        stage_rates=stage_rates(cfg, pixels * 3, pixels * 3, cdf_s * 1e3, syn_s * 1e3),
    )
    # The first 256x256 image of the batch, for the CPU baseline.
    k = next(k for k, s_ in enumerate(sizes) if tuple(s_) == (256, 256))
    gb, p0 = bt.where[k]
    sample = bt.q[gb][p0:p0 + 3].cpu().numpy().astype(np.int64)
    return out, sample


def bench_serve(args):
    """Serving mix: Poisson arrivals (seed 4), 70% stills of the four batch sizes, 30% GOPs
    of 8 frames 1088x1920 4:2:0 (temporal Haar, then the spatial codec per temporal
    subband), BF16 context convs, admission by HBM footprint, continuous batching.
    Each request refers to one of a few prepared inputs (symbols on the device, the
    coder elided).  Runs the offered rate over the arrival window, a bisection for the
    highest rate whose p99 stays stable, that rate confirmed over the full window (10 % lower
    until it holds, at most three times), and the same
    arrivals through the host coder (tables trimmed and copied to the host, rANS on host
    threads); value = sustained Mpixel/s (luma pixels x frames for GOPs) under the offered
    rate."""
    import torch
    from paper_2405_12631_amd import codec, serve
    from wvgen import get_config, make_weights, pack_weights, poisson_arrivals, sinusoid_1f_planes, \
        video_gop_420

    cfg = get_config("serve_mix")
    prec = _precision(args.precision)
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision=prec)
    log = (lambda m: print(m, file=sys.stderr, flush=True))
    preps, by_size = {}, {}
    for k, hw in enumerate(cfg["sizes"]):
        ids = []
        for r in range(2):
            pid = len(preps)
            preps[pid] = serve.Prepared(model, "image", sinusoid_1f_planes(hw[0], hw[1], 3, seed=100 + 2 * k + r),
                                        coder=args.serve_coder_seconds > 0)
            ids.append(pid)
        by_size[tuple(hw)] = ids
    gops = []
    for r in range(2):
        luma, chroma = video_gop_420(T=cfg["gop"], H=cfg["video_hw"][0], W=cfg["video_hw"][1],
                                     seed=5 + r, shift_px=cfg["shift_px"])
        pid = len(preps)
        preps[pid] = serve.Prepared(model, "gop", (luma, chroma), coder=args.serve_coder_seconds > 0)
        gops.append(pid)
    torch.cuda.synchronize()
    budget = int(args.serve_budget_gb * (1 << 30))

    def run(rate, seconds, coder=False):
        arr = poisson_arrivals(rate, seconds, cfg["frac_video"], cfg["sizes"], seed=cfg["seed_arrivals"])
        reqs = []
        for n, a in enumerate(arr):
            pid = gops[n % 2] if a["kind"] == "gop" else by_size[a["size"]][n % 2]
            reqs.append((a["t"], pid))
        offered = sum(preps[p].pixels for _, p in reqs) / seconds / 1e6
        srv = serve.Server(model, budget, coder=coder)
        stats, done = srv.run(reqs, preps, admit_until=seconds, max_seconds=seconds + args.serve_drain, log=log)
        # p99 stability: requests arriving in the second half of the window against those of
        # the first half; stable if every arrival finished and the later p99 is at most 1.5x the
        # earlier one (+ 50 ms), i.e. no queue builds up over the window.
        lat = {h: [1e3 * (d.req["finished"] - d.req["arrival"]) for d in done
                   if (d.req["arrival"] < seconds / 2) == (h == 0)] for h in (0, 1)}
        p99h = [round(float(np.percentile(v, 99)), 2) if v else None for v in (lat[0], lat[1])]
        all_done = stats["completed"] == len(reqs)
        stable = bool(all_done and p99h[0] is not None and p99h[1] is not None and
                      p99h[1] <= 1.5 * p99h[0] + 50.0)
        stats.update(rate_hz=rate, window_s=seconds, arrivals=len(reqs), offered_mpx_per_s=round(offered, 2),
                     p99_ms_first_half=p99h[0], p99_ms_second_half=p99h[1], stable=stable)
        torch.cuda.empty_cache()
        return stats

    runs = {}
    rates = [float(r) for r in args.serve_rates.split(",")] if args.serve_rates else None
    if rates:
        for r in rates:
            runs[f"{r:g}_req_s"] = run(r, args.serve_seconds)
        hi = runs[f"{rates[0]:g}_req_s"]
        best = None
        coder_rate = rates[0]
    else:
        hi = runs[f"{cfg['rate_hz']:g}_req_s"] = run(cfg["rate_hz"], args.serve_seconds)
        # Highest stable rate: bisection on shorter windows between a stable lower bound and
        # the offered rate, then the best rate found confirmed over the full window.
        lo_r, hi_r = 5.0, cfg["rate_hz"]
        search = []
        for _ in range(5):
            mid = round((lo_r + hi_r) / 2, 1)
            st = run(mid, args.serve_search_seconds)
            search.append(st)
            log(f"search {mid} req/s: stable={st['stable']} p99 halves {st['p99_ms_first_half']} / "
                f"{st['p99_ms_second_half']}")
            if st["stable"]:
                lo_r = mid
            else:
                hi_r = mid
        # Confirm over the full window; a rate whose p99 still grows there is stepped down by
        # 10 % (at most three times), and only a full-window stable run is reported as such.
        best = None
        for _ in range(4):
            st = run(lo_r, args.serve_seconds)
            runs[f"full_{lo_r:g}_req_s"] = st
            log(f"confirm {lo_r} req/s over {args.serve_seconds:g} s: stable={st['stable']}")
            if st["stable"]:
                best = st
                break
            lo_r = round(lo_r * 0.9, 1)
        coder_rate = best["rate_hz"] if best else st["rate_hz"]
        runs["search"] = search
    if args.serve_coder_seconds > 0:
        # The same arrivals through the host coder: tables trimmed on the device and copied to
        # the host every iteration, rANS decoding on host threads, symbols copied back.
        runs[f"coder_{coder_rate:g}_req_s"] = run(coder_rate, args.serve_coder_seconds, coder=True)
    out = dict(
        metric="decoded Mpixel/s (ctx model+CDF+inverse lifting), p50/p99 latency vs plain FP32",
        value=hi["mpx_per_s"], unit="Mpixel/s", n_gpus=1, steps=hi["iterations"], warmup=0,
        ms_per_step=round(hi["wall_s"] * 1e3 / max(hi["iterations"], 1), 3), higher_is_better=True,
        scaling="weak", vs_baseline=None,
        dtype=f"{args.precision} context convs (fp32 accumulate), fp32 lifting/cdf", data="synthetic",
        config=dict(workload=f"serve_mix: Poisson arrivals at {hi['rate_hz']:g} req/s for "
                             f"{args.serve_seconds:g} s (then at most {args.serve_drain:g} s to drain), "
                             "70% stills of the four batch sizes, 30% 8-frame 1088x1920 4:2:0 GOPs, "
                             f"HBM budget {args.serve_budget_gb:g} GiB, continuous batching, coder elided",
                    budget_gib=args.serve_budget_gb),
        p50_ms=hi["p50_ms"], p99_ms=hi["p99_ms"],
        highest_stable_rate_hz=(best or {}).get("rate_hz"),
        coder_run={k: v for k, v in runs.items() if k.startswith("coder_")},
        highest_stable=best, runs=runs,
    )
    print(json.dumps(out))


def precision_report(args):
    """The 512x768x3 image with BF16 and FP8 context convs against the FP32 path and the FP64
    oracle: parameter error on plane 0 (every subband and step, the oracle run on the
    decoded symbols), bits per pixel of real GPU-encoded bitstreams, and the GPU encode ->
    GPU decode round trip."""
    import torch
    import oracle as O
    from paper_2405_12631_amd import codec, WV_BF16, WV_FP32, WV_FP8
    from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

    cfg = get_config("ycbcr512x768")
    H, W, N = cfg["H"], cfg["W"], cfg["planes"]
    w = make_weights(cfg)
    blob = pack_weights(cfg, w)
    x = sinusoid_1f_planes(H, W, planes=N, seed=cfg["seed_image"])
    out = dict(workload="ycbcr512x768 precision report", H=H, W=W, planes=N)
    qs_ref = None
    for name, prec in (("fp32", WV_FP32), ("bf16", WV_BF16), ("fp8", WV_FP8)):
        model = codec.Model(cfg, blob, precision=prec)
        data, q_enc = codec.encode(model, x)
        _, _, q_dec = codec.decode(model, data)
        torch.cuda.synchronize()
        r = dict(bytes=len(data), bpp=round(len(data) * 8 / (H * W), 5),
                 roundtrip_bit_exact=bool(torch.equal(q_enc, q_dec)))
        if qs_ref is None:
            qs_ref = O.unpack(q_enc.cpu().numpy().astype(np.int64)[:1], cfg, H, W)
            t0 = time.perf_counter()
            ref = O.context_params_all(qs_ref, cfg, w)
            out["oracle_seconds_plane0"] = round(time.perf_counter() - t0, 2)
        ws = codec.Workspace(model, 1, H, W)
        got = codec.params_all(model, torch.from_numpy(O.pack(qs_ref).astype(np.int16)).cuda(), ws)
        rel = []
        for i in range(len(ref)):
            for g in range(4):
                a = got[i][g].cpu().numpy().astype(np.float64).reshape(-1, 9)
                b = ref[i][g].reshape(-1, 9)
                den = np.abs(b)
                den[:, :6] = np.maximum(den[:, :6], 1e-2)
                rel.append((np.abs(a - b) / den).ravel())
        rel = np.concatenate(rel)
        r.update(param_rel_err_max=float(rel.max()), param_rel_err_mean=float(rel.mean()))
        out[name] = r
    out["bpp_delta_bf16_vs_fp32"] = round(out["bf16"]["bpp"] - out["fp32"]["bpp"], 5)
    out["bpp_delta_fp8_vs_fp32"] = round(out["fp8"]["bpp"] - out["fp32"]["bpp"], 5)
    print(json.dumps(out))


def bench_coder(args):
    """End-to-end decode of the 512x768x3 image through the host entropy coder: for every
    step the CDF rows are trimmed on the device, copied to the host (PCIe), the host rANS
    decoder runs per plane, the symbols go back and are scattered; then synthesis.  Reports
    the PCIe-inclusive rate and the bytes copied per decode with and without the trim."""
    import torch
    from paper_2405_12631_amd import codec
    from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

    cfg = get_config("ycbcr512x768")
    H, W, N = cfg["H"], cfg["W"], cfg["planes"]
    model = codec.Model(cfg, pack_weights(cfg, make_weights(cfg)), precision=_precision(args.precision))
    x = sinusoid_1f_planes(H, W, planes=N, seed=cfg["seed_image"])
    data, q_enc = codec.encode(model, x)
    ws = codec.Workspace(model, N, H, W)
    for _ in range(args.warmup):
        codec.decode(model, data, ws=ws)
    torch.cuda.synchronize()
    t = []
    for _ in range(args.steps):
        t0 = time.perf_counter()
        _, _, q_dec = codec.decode(model, data, ws=ws)
        torch.cuda.synchronize()
        t.append(time.perf_counter() - t0)
    assert torch.equal(q_dec, q_enc), "host-coder decode did not reproduce the symbols"
    # bytes a decode copies device -> host for the tables: trimmed vs full rows
    full = trimmed = 0
    for i in range(len(ws.lay)):
        for g in range(4):
            prm = codec.context_params(model, q_enc, ws, i, g)
            cdf = codec.cdf_tables(model, prm, out=ws.cdf)
            tr = codec.cdf_trim_to_host(model, cdf, ws)
            full += cdf.numel() * 2
            trimmed += tr.lolen.nbytes + tr.packed.nbytes
    t = np.array(t)
    out = dict(
        metric="decoded Mpixel/s end to end with the host entropy coder (PCIe-inclusive)",
        value=round(H * W / t.mean() / 1e6, 4), unit="Mpixel/s", n_gpus=1, steps=args.steps, warmup=args.warmup,
        ms_per_step=round(t.mean() * 1e3, 3), higher_is_better=True, scaling="weak", vs_baseline=None,
        dtype=args.precision, data="synthetic",
        config=dict(workload="ycbcr512x768 through the host rANS decoder: 52 table copies (trimmed) and "
                             "symbol copies per plane group, coder on host threads", bytes=len(data)),
        p50_ms=round(float(np.percentile(t, 50)) * 1e3, 3), p99_ms=round(float(np.percentile(t, 99)) * 1e3, 3),
        table_bytes_to_host=dict(full=full, trimmed=trimmed, ratio=round(full / max(trimmed, 1), 2)),
    )
    print(json.dumps(out))


def hbm_copy():
    """Three plain device copies of 1 GiB: the reference a profiler's FETCH_SIZE and
    WRITE_SIZE readings are scaled by (run under rocprofv3 --pmc, one counter a run)."""
    import torch
    n = 1 << 28   # floats: 1 GiB
    x = torch.ones(n, dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    for _ in range(3):
        y.copy_(x)
    torch.cuda.synchronize()
    print(json.dumps({"workload": "hbm_copy", "copies": 3, "bytes_each": 4 * n}))


def bench_single(args):
    """The plain batch-1 decode of the 512x768x3 image (FP32 unless --precision): one step =
    one coder-elided decode (52 steps of context model, CDF tables and symbol scatter, then
    synthesis), replayed as one library graph.  Returns the line's dict and the CPU-baseline
    inputs."""
    import torch
    from paper_2405_12631_amd import codec
    from wvgen import get_config, make_weights, pack_weights, sinusoid_1f_planes

    cfg = get_config("ycbcr512x768")
    H, W, N = cfg["H"], cfg["W"], cfg["planes"]
    w = make_weights(cfg)
    prec = _precision(args.precision)
    model = codec.Model(cfg, pack_weights(cfg, w), precision=prec)
    x = sinusoid_1f_planes(H, W, planes=N, seed=cfg["seed_image"])
    ws = codec.Workspace(model, N, H, W)
    q_known, _, _ = codec.analyze(model, torch.from_numpy(x).cuda(), ws)
    syms = codec.prepare_elided(model, q_known, ws)
    q = torch.zeros_like(q_known)
    xhat = torch.empty((N, H, W), dtype=torch.float32, device="cuda")
    nsub = len(ws.lay)
    stream = torch.cuda.current_stream()

    def step(ev=None):
        codec.zero(q)
        for i in range(nsub):
            for g in range(4):
                if ev is not None:
                    ev[0].append(torch.cuda.Event(enable_timing=True))
                    ev[0][-1].record(stream)
                prm = codec.context_params(model, q, ws, i, g)
                if ev is not None:
                    ev[1].append(torch.cuda.Event(enable_timing=True))
                    ev[1][-1].record(stream)
                codec.cdf_tables(model, prm, out=ws.cdf)
                if ev is not None:
                    ev[4].append(torch.cuda.Event(enable_timing=True))
                    ev[4][-1].record(stream)
                codec.scatter_symbols(model, syms[i][g], q, ws, i, g)
        if ev is not None:
            ev[2].append(torch.cuda.Event(enable_timing=True))
            ev[2][-1].record(stream)
        codec.synthesize(model, ws, q=q, xhat=xhat)
        if ev is not None:
            ev[3].append(torch.cuda.Event(enable_timing=True))
            ev[3][-1].record(stream)

    # Eager pass, every call event-bracketed on the launch stream: stage times and the roofline.
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    assert torch.equal(q, q_known), "decode did not reproduce the symbols"
    n_eager = max(1, min(args.steps, 5))
    ev = ([], [], [], [], [])
    e_starts = [torch.cuda.Event(enable_timing=True) for _ in range(n_eager)]
    e_ends = [torch.cuda.Event(enable_timing=True) for _ in range(n_eager)]
    torch.cuda.synchronize()
    for k in range(n_eager):
        e_starts[k].record(stream)
        step(ev)
        e_ends[k].record(stream)
    torch.cuda.synchronize()
    lat_eager = np.array([s_.elapsed_time(e_) for s_, e_ in zip(e_starts, e_ends)])
    ctx_ms = np.array([a.elapsed_time(b) for a, b in zip(ev[0], ev[1])]).reshape(n_eager, -1)
    syn_ms = np.array([a.elapsed_time(b) for a, b in zip(ev[2], ev[3])])
    cdf_ms = np.array([a.elapsed_time(b) for a, b in zip(ev[1], ev[4])]).reshape(n_eager, -1)

    # Timed steps: the same decode captured once as a library graph and replayed (no host
    # launch gaps between the ~350 kernels of a decode).
    torch.cuda.synchronize()
    graph = codec.Graph(step)
    torch.cuda.synchronize()
    for _ in range(args.warmup):
        graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(q, q_known), "graph replay did not reproduce the symbols"
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        starts[k].record(stream)
        graph.replay()
        ends[k].record(stream)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    assert torch.equal(q, q_known), "graph replay did not reproduce the symbols"

    lat = np.array([s_.elapsed_time(e_) for s_, e_ in zip(starts, ends)])
    ms_step = elapsed * 1e3 / args.steps
    mpx = H * W * args.steps / elapsed / 1e6

    ctx_flops = context_flops_per_coef(cfg) * H * W * N
    ctx_time = ctx_ms.sum(axis=1).mean() * 1e-3
    n_ctx_launch = nsub * (cfg["ctx_layers"] * 4) + nsub      # step layers + one LSTM per subband
    peak = MFMA_PEAK_TFLOPS[args.precision]
    kname = {"fp32": "conv3x3_f32p", "bf16": "conv3x3_mfma_bf16",
             "fp8": "conv3x3_mfma_bf16 (e4m3 form)"}[args.precision]
    roof = dict(bound="mfma", achieved=round(ctx_flops / ctx_time / 1e12, 3),
                peak=peak, unit="TFLOP/s",
                frac=round(ctx_flops / ctx_time / 1e12 / peak, 4), traffic=measured_traffic(args.precision),
                traffic_unit="HBM bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
                kernel=f"{kname} (context model: ConvLSTM + step stacks)",
                flops_per_decode=ctx_flops, launches_per_decode=n_ctx_launch,
                avg_launch_us=round(ctx_time / n_ctx_launch * 1e6, 2))

    out = dict(
        metric="decoded Mpixel/s (ctx model+CDF+inverse lifting), p50/p99 latency vs plain FP32",
        value=round(mpx, 4), unit="Mpixel/s", n_gpus=1, steps=args.steps, warmup=args.warmup,
        ms_per_step=round(ms_step, 3), higher_is_better=True, scaling="weak", vs_baseline=None,
        dtype="f32" if args.precision == "fp32" else
        f"{args.precision} context convs (fp32 accumulate), fp32 lifting/cdf",
        data="synthetic",
        config=dict(workload="ycbcr512x768: one 512x768 3-plane YCbCr image, 1/f sinusoids + noise "
                             "(seed 2), 4-level CNN lifting (32 ch), 64-ch 4-layer context stacks, "
                             f"K=3 mixture, step 4, {args.precision.upper()} context, batch 1, "
                             "coder elided",
                    batch=1, planes=N, H=H, W=W),
        p50_ms=round(float(np.percentile(lat, 50)), 3), p99_ms=round(float(np.percentile(lat, 99)), 3),
        launch="one wv_graph replay per decode (captured once); stage_ms and roofline from an "
               "event-bracketed eager pass of the same decode",
        eager_ms_per_step=round(float(lat_eager.mean()), 3),
        stage_ms=dict(context=round(float(ctx_ms.sum(1).mean()), 3),
                      cdf=round(float(cdf_ms.sum(1).mean()), 3),
                      synthesis=round(float(syn_ms.mean()), 3),
                      scatter_rest=round(float(lat_eager.mean() - ctx_ms.sum(1).mean() - cdf_ms.sum(1).mean()
                                               - syn_ms.mean()), 3)),
        roofline=roof,
        stage_rates=stage_rates(cfg, N * H * W, N * H * W, float(cdf_ms.sum(1).mean()), float(syn_ms.mean())),
    )
    return out, (cfg, w, q_known.cpu().numpy().astype(np.int64), H, W)


def bench_headline(args):
    """The headline: the BF16 batched decode of 64 mixed-size images, with the plain FP32
    batch-1 decode measured in the same process as its baseline."""
    base_args = argparse.Namespace(**vars(args))
    base_args.precision = "fp32"
    base, _ = bench_single(base_args)
    batch_args = argparse.Namespace(**vars(args))
    batch_args.precision = args.precision or "bf16"
    out, sample = bench_batch(batch_args)
    out["vs_baseline"] = round(out["value"] / base["value"], 4)
    out["vs_baseline_meaning"] = ("value / the plain FP32 batch-1 decode's Mpixel/s (512x768x3, same "
                                  "process, same protocol), nested as baseline")
    out["baseline"] = {k: base[k] for k in ("value", "unit", "ms_per_step", "p50_ms", "p99_ms", "dtype",
                                            "config", "stage_ms", "roofline", "stage_rates")}
    out["paper_context"] = ("Table 1: pWave++ (4-step LL) decodes a 512x768 luma image in 0.35 s on an "
                            "RTX A6000 incl. entropy coding and post-processing (about 1.1 Mpixel/s); "
                            "other hardware and scope, not the target")
    if not args.no_cpu_baseline:
        from wvgen import get_config, make_weights
        cfg = get_config("batch64_mixed")
        out["cpu_baseline"] = cpu_baseline(cfg, make_weights(cfg), sample, 256, 256)
    print(json.dumps(out))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--precision", choices=["fp32", "bf16", "fp8"], default=None,
                    help="context-conv precision (lifting and CDFs stay FP32); default bf16 for the "
                         "headline, batched and serving workloads, fp32 for the single-image ones")
    ap.add_argument("--nb-table", default=None,
                    help="batch: per-level output-channel blocks, e.g. 4,4,4,4 (no autotuning)")
    ap.add_argument("--workload", choices=["headline", "ycbcr512x768", "batch64_mixed", "serve_mix",
                                           "precision_report", "coder512x768", "hbm_copy"],
                    default="headline")
    ap.add_argument("--serve-seconds", type=float, default=60.0, help="arrival window of the serving run")
    ap.add_argument("--serve-drain", type=float, default=20.0, help="time allowed to drain after it")
    ap.add_argument("--serve-rates", default=None,
                    help="comma-separated arrival rates (req/s) for the serving run; default: the "
                         "offered rate, then a search for the highest rate with a stable p99")
    ap.add_argument("--serve-search-seconds", type=float, default=15.0,
                    help="arrival window of each step of the stable-rate search")
    ap.add_argument("--serve-coder-seconds", type=float, default=20.0,
                    help="arrival window of the host-coder run at the highest stable rate (0: skip)")
    ap.add_argument("--serve-budget-gb", type=float, default=150.0, help="HBM admission budget")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU; this build has no multi-GPU path (run with --gpus 1)",
              file=sys.stderr)
        sys.exit(2)
    if args.workload == "hbm_copy":
        return hbm_copy()
    if args.workload == "headline":
        return bench_headline(args)
    if args.workload == "batch64_mixed":
        args.precision = args.precision or "bf16"
        out, sample = bench_batch(args)
        if not args.no_cpu_baseline:
            from wvgen import get_config, make_weights
            cfg = get_config("batch64_mixed")
            out["cpu_baseline"] = cpu_baseline(cfg, make_weights(cfg), sample, 256, 256)
        print(json.dumps(out))
        return
    if args.workload == "precision_report":
        return precision_report(args)
    if args.workload == "coder512x768":
        args.precision = args.precision or "fp32"
        return bench_coder(args)
    if args.workload == "serve_mix":
        args.precision = args.precision or "bf16"
        return bench_serve(args)
    args.precision = args.precision or "fp32"
    out, (cfg, w, q_planes, H, W) = bench_single(args)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg, w, q_planes, H, W)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
