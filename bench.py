"""Benchmark of the projector hot path on one MI355X.

Workload: 512^3 FP32 volume of 200 seeded random ellipsoids plus a uniform
cylinder; circular cone beam, 720 projections of a 768 x 768 detector
(pitch 1.5, SOD 1600, SDD 3200), ray-march step 0.5 voxel.  One step is one
SIRT iteration of Eq. (1) over all 720 projections: forward projection with
the fused correction R (b - A x), exact-transpose backprojection, update.
The SIRT weights R and C are built once per geometry (during warm-up).

Metric: FP+BP Gsamples/s = 2 N_s / (time per step) with N_s the exact
number of trilinear samples of one forward projection.  Kernel times come
from HIP events the library records on its launch stream inside the timed
steps.  The CPU baseline is the FP64 oracle on a bounded view subset.

The JSON line also carries, when the trained correction networks are
present, the time-to-PSNR comparison of the learned pipeline (4 stages of an
ordered-subset SIRT epoch + U-Net) against 50 plain SIRT iterations on one
held-out phantom of the learned-correction configuration (256^3, 180 x 384^2,
Poisson noise).

Roofline: the dominant kernel (the exact-transpose backprojector) is
reported against the plain-ALU issue roof: algorithmic FP32 VALU lane
operations per sample (44 for the backprojector, 32 for the forward
projector: position, corner indices and fractions, trilinear weights or
blend, accumulation) x samples per launch / launch time, against 256 CUs x 4
SIMDs x 32 lanes per clock x 2.4 GHz = 78.6e12 lane operations per second
(the fp32 vector peak of 157.3 TFLOP/s counts an FMA as two).  The
backprojector's 8 algorithmic LDS 64-bit atomics per sample (before the
register merge of same-cell samples) are also set against the LDS roof (128
bytes per clock per CU: 16 such lane operations); the issue counters of the
committed summary give its measured LDS and VALU rates, the fraction of
cycles lost to LDS bank conflicts and an LDS-pipe estimate (4 clocks per LDS
wave-instruction plus the conflict clocks), the kernel's actual limit; for the
forward projector they give the texture addresser's busy and L1-stalled
fractions, its limit.  HBM traffic and
the L2 hit rate per kernel are read from the committed counter summary
(rocprofv3 --pmc passes: FETCH_SIZE, WRITE_SIZE scaled by the same counters
of a plain copy kernel of known size, ``--copy-calibrate``; TCC_HIT_sum and
TCC_MISS_sum); they are null when the kernel's sources changed since.  The
gather-equivalent bandwidth (32 B per FP32 sample, the on-chip bytes of 8
voxel reads or accumulations) is reported beside it as the fraction of the
achievable HBM bandwidth (a stream copy timed in the same run), the figure
the 60% target is stated in.

The ``unet`` object times the correction network alone (forward pass and one
Adam training step on a 256^3 volume) with its FLOP rate against the BF16
dense MFMA peak of 2.5 PFLOP/s.

The ``voxel_bp`` object repeats the SIRT run with the paper's voxel-driven
backprojector in place of the exact transpose (speed, and residual and PSNR
after the same number of iterations); the ``cylinder`` object runs SIRT on the
aligned cylindrical domain (a polar grid inscribed in the same box) with the
same scan.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--dtype f32|bf16]
                       [--copy-calibrate] [--no-learned] [--no-voxel-bp] [--no-cylinder]
                       [--no-bf16] [--no-helical] [--no-autograd] [--no-unet]
"""

from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "FP+BP Gsamples/s @512³×720 proj; time-to-PSNR learned vs plain SIRT"
HBM_PEAK_GBS = 8000.0
GATHER_BYTES = {"f32": 32, "bf16": 16}   # 8 voxel reads per sample
# plain-ALU issue roof: 256 CUs x 4 SIMDs x 32 lanes per clock x 2.4 GHz
CLOCK_HZ = 2.4e9
ALU_PEAK_TOPS = 256 * 4 * 32 * CLOCK_HZ / 1e12
# LDS roof for 64-bit atomics: 128 bytes per clock per CU = 16 lane operations
LDS_ATOMIC_PEAK_TOPS = 256 * 16 * 2.4e9 / 1e12
# algorithmic VALU lane operations per sample (position 3 FMA; floor, convert
# and fraction per axis 9; clamps and address 5; blend 14 or 8 weights and
# their fixed-point conversion; accumulate 1)
# (the row "bp_brick_kernel" is the exact backprojection, whose default form is
# bp_own_kernel, and "vbp_kernel" the voxel-driven one, vbp_tile_kernel)
ALU_OPS = {"fp_kernel": 32, "bp_brick_kernel": 44}
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic_sirt_512cube_720x768sq.md")
WEIGHTS_FILE = os.path.join(ROOT, "paper_2609_30166_amd", "weights", "unet_learned_256.npz")
KERNEL_SOURCES = {
    "bp_brick_kernel": ["backproject.hip", "ray_common.h", "ctrex_internal.h", "launch_order.h",
                        "warp_bounds.h"],
    "fp_kernel": ["projector.hip", "ray_common.h", "ctrex_internal.h", "launch_order.h"],
    "vbp_kernel": ["voxel_bp.hip", "ray_common.h", "ctrex_internal.h"],
}


def _log(msg):
    print("[bench] " + msg, file=sys.stderr, flush=True)


def _oracle_fp_bp(cfg, x, views):
    import numpy as np

    import oracle

    xd = x.astype(np.float64)
    t0 = time.perf_counter()
    y, cnt = oracle.forward(cfg.P, cfg.shape, cfg.n_u, cfg.n_v, xd, cfg.step, views=views,
                            return_count=True)
    t1 = time.perf_counter()
    oracle.back(cfg.P, cfg.shape, cfg.n_u, cfg.n_v, y, cfg.step, views=views)
    t2 = time.perf_counter()
    return y, cnt, t1 - t0, t2 - t1


def cpu_baseline(cfg, x, n_views):
    """FP64 oracle, FP + BP samples/s: ``n_views`` evenly spaced projections
    of the benchmark workload (the reported value), plus the whole tiny
    configuration and 36 of the 360 projections of the differentiation one.
    Returns (record, the oracle's projections of the sampled views, views)."""
    import numpy as np

    import oracle
    from synth.configs import make_config, make_phantom

    views = list(range(0, cfg.n_proj, cfg.n_proj // n_views))[:n_views]
    y, cnt, t_fp, t_bp = _oracle_fp_bp(cfg, x, views)
    rate = 2.0 * cnt / (t_fp + t_bp) / 1e9
    extra = {}
    for name, sub in (("tiny", None), ("diff", 36)):
        c = make_config(name)
        xc, _ = make_phantom(c, seed=0)
        vv = None if sub is None else list(range(0, c.n_proj, c.n_proj // sub))[:sub]
        _, n2, a, b = _oracle_fp_bp(c, xc, vv)
        extra[name] = {"gsamples_per_s": 2.0 * n2 / (a + b) / 1e9, "samples_each_way": n2,
                       "views": c.n_proj if vv is None else len(vv), "fp_s": a, "bp_s": b}
    rec = {"value": rate, "unit": "Gsamples/s", "cores": oracle.num_threads(), "kind": "oracle",
           "sample": "FP64 oracle FP+BP over %d of the 720 views of the same 512^3 phantom "
                     "(%d samples each way; FP %.1f s, BP %.1f s)" % (len(views), cnt, t_fp, t_bp),
           "other_configs": extra}
    return rec, y, views


def source_hash(kernel):
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel]:
        with open(os.path.join(ROOT, "paper_2609_30166_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def counter_record(kernel, dtype):
    """Counter record of ``kernel`` (HBM bytes per launch, L2 hits and
    misses) from the committed summary, or None if absent or taken on other
    sources."""
    try:
        text = open(TRAFFIC_FILE).read()
    except OSError:
        return None
    m = re.search(r"```json\n(.*?)\n```", text, re.S)
    if not m:
        return None
    rec = json.loads(m.group(1)).get("%s/%s" % (kernel, dtype))
    if not rec or rec.get("source_hash") != source_hash(kernel):
        return None
    return rec


def measured_traffic(kernel, dtype):
    rec = counter_record(kernel, dtype)
    return None if rec is None else rec["hbm_bytes_per_launch"]


def l2_hit_rate(kernel, dtype):
    rec = counter_record(kernel, dtype)
    if rec is None or "tcc_hit" not in rec:
        return None
    return rec["tcc_hit"] / max(rec["tcc_hit"] + rec["tcc_miss"], 1.0)


def achievable_bandwidth(dev, n=1 << 28, reps=5):
    """Stream copy of n floats (read + write, 8n bytes), timed with HIP events
    on the launch stream: the achievable HBM bandwidth, the better of the
    library's conversion kernel and the runtime's device-to-device copy
    (median GB/s of each)."""
    import ctypes

    import torch
    from paper_2609_30166_amd import _lib

    src = torch.ones(n, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    ctx = ctypes.c_void_p()
    L = _lib.lib()
    _lib.check(None, L.ctrex_create(ctypes.byref(ctx), dev.index))
    s = torch.cuda.current_stream(dev)
    rates = []
    for i in range(reps + 1):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(s)
        _lib.check(ctx, L.ctrex_convert(ctx, ctypes.c_void_p(src.data_ptr()), _lib.F32,
                                        ctypes.c_void_p(dst.data_ptr()), _lib.F32, n,
                                        ctypes.c_void_p(s.cuda_stream)))
        e1.record(s)
        e1.synchronize()
        if i:
            rates.append(8.0 * n / (e0.elapsed_time(e1) * 1e-3) / 1e9)
    L.ctrex_destroy(ctx)
    rt = []
    for i in range(reps + 1):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(s)
        dst.copy_(src)
        e1.record(s)
        e1.synchronize()
        if i:
            rt.append(8.0 * n / (e0.elapsed_time(e1) * 1e-3) / 1e9)
    del src, dst
    rates.sort()
    rt.sort()
    return max(rates[len(rates) // 2], rt[len(rt) // 2])


def copy_calibration(dev):
    """A plain copy of 2^27 floats (512 MiB read + 512 MiB written) through the
    library's conversion kernel, for scaling the FETCH/WRITE counters."""
    import torch
    from paper_2609_30166_amd import _lib

    n = 1 << 27
    src = torch.ones(n, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    import ctypes
    ctx = ctypes.c_void_p()
    L = _lib.lib()
    _lib.check(None, L.ctrex_create(ctypes.byref(ctx), dev.index))
    for _ in range(3):
        _lib.check(ctx, L.ctrex_convert(ctx, ctypes.c_void_p(src.data_ptr()), _lib.F32,
                                        ctypes.c_void_p(dst.data_ptr()), _lib.F32, n, None))
    torch.cuda.synchronize()
    L.ctrex_destroy(ctx)
    _log("copy calibration: 3 copies of %d bytes" % (4 * n))


def time_to_psnr(dev):
    """Learned 4-stage pipeline vs 50 plain SIRT iterations on one held-out
    phantom; None when the trained weights are not present."""
    if not os.path.exists(WEIGHTS_FILE):
        return None
    import numpy as np

    import torch

    from paper_2609_30166_amd import learned
    from paper_2609_30166_amd.train_unet import load
    from synth import configs

    cfg, geom = learned.learned_geometry(device=dev)
    net = load(WEIGHTS_FILE, dev)
    seed = list(configs.TEST_SEEDS)[0]
    meta = json.loads(str(np.load(WEIGHTS_FILE, allow_pickle=False)["meta"]))
    stages, per = int(meta.get("stages", 4)), int(meta.get("iters_per_stage", 1))
    subsets = int(meta.get("subsets", 0)) or None
    res = learned.compare(geom, net, cfg, [seed], sirt_iters=50, n_stages=stages,
                          iters_per_stage=per, log=lambda s: _log("learned: " + s),
                          fov=bool(meta.get("fov_mask", False)), subsets=subsets)
    r = res["rows"][0]
    # the network's gain, as the time the pipeline's physics steps alone need
    # to reach the learned PSNR (OS-SIRT epochs, one at a time, up to 16)
    x_true, b = learned.make_sample(cfg, geom, seed)
    mask = learned.fov_mask(geom.shape, geom.device)
    subs = learned._subsets(geom, subsets)
    xp = torch.zeros(geom.shape, dtype=torch.float32, device=geom.device)
    t_alone, epochs, p_alone, best, best_ep = 0.0, 0, float("nan"), -1e9, 0
    while epochs < 16:
        _, dt = learned._timed(lambda: learned.physics(geom, xp, b, per, subs))
        t_alone += dt
        epochs += 1
        p_alone = learned.psnr(xp, x_true, mask)
        if p_alone > best:
            best, best_ep = p_alone, epochs
        if p_alone >= r["psnr_learned"]:
            break
    # the learned configuration as first specified: 4 x (one plain SIRT
    # iteration + U-Net), with these networks (trained on OS-SIRT iterates)
    pipe = learned.LearnedSirt(geom, net, 4, 1,
                               mask="fov" if meta.get("fov_mask", False) else None)
    pipe(b)   # warm the plain-SIRT workspace and weights outside the timing
    (x_lit, st_lit), t_lit = learned._timed(lambda: pipe(b))
    x4 = torch.zeros(geom.shape, dtype=torch.float32, device=geom.device)
    geom.sirt(x4, b, 4, norms=False)
    lit = {"psnr_learned": learned.psnr(x_lit, x_true, mask),
           "psnr_sirt_same_budget": learned.psnr(x4, x_true, mask), "t_learned": t_lit,
           "accepted": sum(1 for q in st_lit if q.get("corrected")),
           "psnr_sirt": r["psnr_sirt"]}
    return {"sirt_iters": 50, "stages": stages, "iters_per_stage": per, "phantom_seed": seed,
            "physics_steps": res["physics"],
            "psnr_sirt_db": r["psnr_sirt"], "psnr_learned_db": r["psnr_learned"],
            "psnr_physics_alone_same_steps_db": r["psnr_sirt_same_budget"],
            "t_physics_alone_s": r["t_same_budget"],
            "resid_sirt": r["resid_sirt"], "resid_learned": r["resid_learned"],
            "t_sirt_s": r["t_sirt"], "t_learned_s": r["t_learned"],
            "time_ratio": r["t_learned"] / r["t_sirt"],
            "reaches_sirt_psnr": bool(r["psnr_learned"] >= r["psnr_sirt"]),
            "physics_alone_reaches_sirt_psnr": bool(r["psnr_sirt_same_budget"] >= r["psnr_sirt"]),
            "physics_alone_time_ratio": r["t_same_budget"] / r["t_sirt"],
            "target_met_by": "the ordered-subset physics steps already meet the <= 1/3 "
                             "time-to-PSNR target on their own; the networks add "
                             "%.2f dB at %.3f s more" % (
                                 r["psnr_learned"] - r["psnr_sirt_same_budget"],
                                 r["t_learned"] - r["t_same_budget"]),
            "network_gain": {"physics_alone_epochs_run": epochs,
                             "reached_learned_psnr": bool(p_alone >= r["psnr_learned"]),
                             "psnr_db_last": p_alone, "t_s": t_alone,
                             "best_psnr_db_physics_alone": best, "best_at_epoch": best_ep},
            "as_first_specified": {
                "form": "4 x (1 plain SIRT iteration + U-Net), networks trained on OS-SIRT "
                        "iterates, residual acceptance rule",
                "psnr_learned_db": lit["psnr_learned"], "psnr_sirt4_db": lit["psnr_sirt_same_budget"],
                "t_learned_s": lit["t_learned"], "corrections_kept": lit["accepted"],
                "reaches_sirt_psnr": bool(lit["psnr_learned"] >= lit["psnr_sirt"])},
            "workload": "256^3, 180 projections of 384x384, Poisson I0=1e4, seeded held-out "
                        "phantom; inference only"}


def unet_flops(n):
    """Multiply-add FLOPs (2 per MAC) of one U-Net forward pass on an n^3
    volume: 3x3x3 convolutions 54 cin cout per output voxel, 2x2x2 stride-2
    up-sampling 2 cin cout per output voxel, the 16-channel head 32 per voxel."""
    from paper_2609_30166_amd.unet import LAYERS

    level = dict(e1a=1, e1b=1, e2a=2, e2b=2, bna=3, bnb=3, up2=2, d2a=2, d2b=2, up1=1,
                 d1a=1, d1b=1)   # level of each layer's output
    total = 32.0 * n ** 3
    for name, kind, cin, cout in LAYERS:
        vox = n ** 3 / 8 ** (level[name] - 1)
        total += (54.0 if kind == "conv" else 2.0) * cin * cout * vox
    return total


def unet_run(dev, args, n=256, reps=5):
    """The correction U-Net alone on a 256^3 volume (He-normal weights from a
    seed, uniform synthetic input): forward pass (launched kernel by kernel,
    and as replays of its captured HIP graph) and one training step (forward,
    MSE, backward, Adam), mean of ``reps`` after one warm-up, timed with HIP
    events on the library's launch stream."""
    import torch

    from paper_2609_30166_amd.unet import UNet

    net = UNet(device=dev, seed=1)
    gen = torch.Generator(device="cpu").manual_seed(3)
    x = torch.rand((n, n, n), generator=gen).to(dev)
    t = x + 0.01 * torch.rand((n, n, n), generator=gen).to(dev)
    s = torch.cuda.current_stream(dev)

    def timed(fn):
        fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(s)
        for _ in range(reps):
            fn()
        e1.record(s)
        e1.synchronize()
        return e0.elapsed_time(e1) / reps

    out = torch.empty_like(x)
    fwd_ms = timed(lambda: net.forward(x, out=out))
    graph = net.capture_forward(x, out)
    graph_ms = timed(graph.replay)
    del graph
    step_ms = timed(lambda: net.train_step(x, t))
    f = unet_flops(n)
    peak = 2.5e15
    del net, x, t, out
    return {"workload": "U-Net 16/32/64 channels, 3 levels, BF16 activations, FP32 "
                        "accumulation, %d^3 volume, batch 1" % n,
            "forward_ms": fwd_ms, "forward_graph_ms": graph_ms, "train_step_ms": step_ms,
            "forward_gflop": f / 1e9,
            "forward_tflops": f / (fwd_ms * 1e-3) / 1e12,
            "forward_frac_of_bf16_peak": f / (fwd_ms * 1e-3) / peak,
            "train_step_tflops_est": 3.0 * f / (step_ms * 1e-3) / 1e12,
            "note": "training step counted as 3x the forward FLOPs (data and weight "
                    "gradients); per-kernel rates are in the committed kernel trace"}


def bf16_run(g, xt, b32, vol32, y_or, views, args):
    """The benchmark's SIRT run repeated with BF16 storage of the volume the
    rays gather and of the sinogram (FP32 accumulation and FP32 master
    volume): per-step and per-kernel times; the BF16 forward projection of
    the phantom against the FP64 oracle on the sampled views; the volume
    after the same iterations against the FP32 run's."""
    import numpy as np
    import torch

    bt = torch.bfloat16
    y16 = g.forward(xt.to(bt), views=views, out_dtype=bt).float().cpu().numpy()
    fp_err = float(np.linalg.norm(y16 - y_or) / np.linalg.norm(y_or))
    b16 = b32.to(bt)
    vol = torch.zeros_like(vol32)
    ws = g.workspace(gather_dtype=bt)
    for _ in range(args.warmup):
        g.sirt(vol, b16, 1, gather_dtype=bt, workspace=ws, norms=False)
    g.profile(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        g.sirt(vol, b16, 1, gather_dtype=bt, workspace=ws, norms=False)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = g.profile_read()
    g.profile(False)
    norms = g.sirt(vol, b16, 1, gather_dtype=bt, workspace=ws)
    n_s = g.sample_count()
    ms = 1e3 * (t1 - t0) / args.steps
    d = (vol - vol32).double()
    res = {"ms_per_step": ms, "gsamples_per_s": 2.0 * n_s / (ms * 1e-3) / 1e9,
           "fp_ms": prof["forward"][0] / max(prof["forward"][1], 1),
           "bp_ms": prof["back"][0] / max(prof["back"][1], 1),
           "update_ms": prof["update"][0] / max(prof["update"][1], 1),
           "forward_rel_l2_vs_fp64_oracle": fp_err,
           "forward_views_compared": list(views),
           "sirt_volume_rel_l2_vs_f32_run": float(d.norm() / vol32.double().norm()),
           "residual_norm_after": float(norms[0]),
           "iterations": args.warmup + args.steps + 1}
    del vol, ws, b16
    return res


def helical_run(dev, args):
    """Per-projection geometry configuration: 256^3, helical scan (pitch 1.0)
    with seeded rigid jitter, 1200 projections of 512x256, 4 angular
    sub-views each, a 32^3 displacement field applied during traversal: SIRT
    iterations over all projections, per-kernel times and rates."""
    import torch

    from paper_2609_30166_amd import Geometry
    from synth.configs import make_config, make_phantom

    cfg = make_config("helical")
    x, _ = make_phantom(cfg, seed=0)
    g = Geometry(cfg.P, cfg.n_u, cfg.n_v, cfg.shape, cfg.step, device=dev, U=cfg.U, tau=cfg.tau)
    n_s = g.sample_count()
    b = g.forward(torch.from_numpy(x).to(dev))
    vol = torch.zeros(cfg.shape, dtype=torch.float32, device=dev)
    ws = g.workspace()
    for _ in range(args.warmup):
        g.sirt(vol, b, 1, workspace=ws, norms=False)
    g.profile(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        g.sirt(vol, b, 1, workspace=ws, norms=False)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = g.profile_read()
    g.profile(False)
    norms = g.sirt(vol, b, 1, workspace=ws)
    fp_ms = prof["forward"][0] / max(prof["forward"][1], 1)
    bp_ms = prof["back"][0] / max(prof["back"][1], 1)
    ms = 1e3 * (t1 - t0) / args.steps
    res = {"workload": "SIRT iteration, 256^3, helical cone beam (pitch 1.0, rigid jitter), "
                       "1200 projections x 4 sub-views of 512x256, 32^3 displacement warp",
           "samples_per_fp": n_s, "ms_per_step": ms,
           "gsamples_per_s": 2.0 * n_s / (ms * 1e-3) / 1e9,
           "sirt_iterations_per_s": 1e3 / ms,
           "fp_ms": fp_ms, "bp_ms": bp_ms,
           "update_ms": prof["update"][0] / max(prof["update"][1], 1),
           "fp_gsamples_per_s": n_s / (fp_ms * 1e-3) / 1e9,
           "bp_gsamples_per_s": n_s / (bp_ms * 1e-3) / 1e9,
           "residual_norm_data": float(torch.linalg.vector_norm(b.double())),
           "residual_norm_after": float(norms[0])}
    del b, vol, ws
    g.close()
    return res


def autograd_run(dev, args):
    """Differentiation configuration: 256^3, 360 projections of 384x384,
    Poisson-noised data (I0 = 1e4); one step = the loss ||A x - b||^2 +
    1e-3 TV(x) and its gradient through the autograd functions (forward
    projection with the residual epilogue, scaled exact-transpose
    backprojection, TV kernels)."""
    import numpy as np
    import torch

    from paper_2609_30166_amd import Geometry, reconstruction_loss
    from synth.configs import make_config, make_phantom
    from synth.noise import poisson_log_transform

    cfg = make_config("diff")
    x_true, _ = make_phantom(cfg, seed=0)
    g = Geometry(cfg.P, cfg.n_u, cfg.n_v, cfg.shape, cfg.step, device=dev)
    y = g.forward(torch.from_numpy(x_true).to(dev)).cpu().numpy()
    b = torch.from_numpy(poisson_log_transform(y, cfg.extra["I0"],
                                               np.random.default_rng([0, 4, 1]))
                         .astype(np.float32)).to(dev)
    x = torch.zeros(cfg.shape, dtype=torch.float32, device=dev, requires_grad=True)

    def step():
        x.grad = None
        loss = reconstruction_loss(x, b, g, lam=1e-3)
        loss.backward()
        return loss

    for _ in range(max(args.warmup, 1)):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    n = max(args.steps, 3)
    for _ in range(n):
        loss = step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    n_s = g.sample_count()
    ms = 1e3 * (t1 - t0) / n
    res = {"workload": "loss ||A x - b||^2 + 1e-3 TV(x) and its gradient, 256^3, 360 "
                       "projections of 384x384, Poisson I0 = 1e4",
           "ms_per_step": ms, "steps": n, "samples_per_fp": n_s,
           "gsamples_per_s": 2.0 * n_s / (ms * 1e-3) / 1e9, "loss": float(loss.detach())}
    del x, b
    g.close()
    return res


def voxel_bp_comparison(g, b, sdt, xt, vol_exact, norms_exact, args, bp_ms_exact, ms_exact):
    """The same SIRT run (warm-up + timed steps + one more) with the paper's
    voxel-driven backprojector B and C = 1 / (B 1) in place of the exact
    transpose: per-step and per-kernel times, and the residual norm and PSNR
    reached after the same number of iterations as the exact-transpose run."""
    import numpy as np
    import torch

    from paper_2609_30166_amd.learned import fov_mask, psnr

    vol = torch.zeros_like(vol_exact)
    ws = g.workspace(gather_dtype=sdt)
    for _ in range(args.warmup):
        g.sirt(vol, b, 1, gather_dtype=sdt, workspace=ws, norms=False, voxel_bp=True)
    g.profile(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        g.sirt(vol, b, 1, gather_dtype=sdt, workspace=ws, norms=False, voxel_bp=True)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = g.profile_read()
    g.profile(False)
    norms = g.sirt(vol, b, 1, gather_dtype=sdt, workspace=ws, voxel_bp=True)
    mask = fov_mask(g.shape, g.device)
    bp_ms = prof["back"][0] / max(prof["back"][1], 1)
    n_vv = float(np.prod(g.shape)) * g.n_proj
    res = {
        "iterations": args.warmup + args.steps + 1,
        "ms_per_step": 1e3 * (t1 - t0) / args.steps,
        "fp_ms": prof["forward"][0] / max(prof["forward"][1], 1),
        "bp_ms": bp_ms,
        "update_ms": prof["update"][0] / max(prof["update"][1], 1),
        "bp_voxel_views_per_s": n_vv / (bp_ms * 1e-3),
        "bp_speedup_vs_exact": bp_ms_exact / bp_ms,
        "step_speedup_vs_exact": ms_exact / (1e3 * (t1 - t0) / args.steps),
        "residual_norm_after": float(norms[0]),
        "residual_norm_after_exact": float(norms_exact[0]),
        "psnr_db": psnr(vol, xt, mask),
        "psnr_db_exact": psnr(vol_exact, xt, mask),
    }
    del ws, vol
    return res


def cylinder_sirt(dev, cfg, args):
    """SIRT on the aligned cylindrical domain with the same scan (720 x 768^2):
    a polar grid of 256 rings x 1608 angles x 512 slices (dr = dz = 1; the
    cylinder inscribed in the 512^3 box, ~1 voxel arc spacing at the rim)
    holding a seeded vial phantom; forward projection clipped to the
    cylinder, voxel-driven backprojection over the polar voxels.  Reports
    per-step and per-kernel times, samples of one forward projection and the
    residual norms of the iterates."""
    import numpy as np
    import torch

    from paper_2609_30166_amd import CylinderGeometry
    from synth.phantoms import vial_polar

    n_r, n_phi, n_z = 256, 1608, 512
    g = CylinderGeometry(cfg.P, cfg.n_u, cfg.n_v, n_r, n_phi, n_z, 1.0, 1.0, cfg.step,
                         device=dev)
    x = torch.from_numpy(vial_polar(n_r, n_phi, n_z, 1.0, 1.0, np.random.default_rng(17))).to(dev)
    b = g.forward(x)
    n_s = g.sample_count()
    vol = torch.zeros_like(x)
    ws = g.workspace()
    for _ in range(args.warmup):
        g.sirt(vol, b, 1, workspace=ws, norms=False)
    g.profile(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        g.sirt(vol, b, 1, workspace=ws, norms=False)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = g.profile_read()
    g.profile(False)
    norms = g.sirt(vol, b, 1, workspace=ws)
    fp_ms = prof["forward"][0] / max(prof["forward"][1], 1)
    bp_ms = prof["back"][0] / max(prof["back"][1], 1)
    res = {
        "workload": "SIRT iteration on a 256 x 1608 x 512 polar grid (dr = dz = 1), 720 "
                    "circular cone-beam projections of 768x768, step 0.5",
        "iterations": args.warmup + args.steps + 1,
        "ms_per_step": 1e3 * (t1 - t0) / args.steps,
        "fp_ms": fp_ms,
        "bp_ms": bp_ms,
        "update_ms": prof["update"][0] / max(prof["update"][1], 1),
        "samples_per_fp": n_s,
        "fp_gsamples_per_s": n_s / (fp_ms * 1e-3) / 1e9,
        "bp_voxel_views_per_s": float(n_r * n_phi * n_z) * g.n_proj / (bp_ms * 1e-3),
        "residual_norm_data": float(torch.linalg.vector_norm(b.double())),
        "residual_norm_after": float(norms[0]),
    }
    del x, b, vol, ws
    g.close()
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--dtype", choices=["f32", "bf16"], default="f32")
    ap.add_argument("--cpu-views", type=int, default=8,
                    help="views of the CPU-oracle baseline sample (0 = skip)")
    ap.add_argument("--n-proj", type=int, default=720, help=argparse.SUPPRESS)
    ap.add_argument("--copy-calibrate", action="store_true",
                    help="also run a plain copy kernel of known size (counter calibration)")
    ap.add_argument("--no-learned", action="store_true",
                    help="skip the learned-vs-SIRT time-to-PSNR comparison")
    ap.add_argument("--no-voxel-bp", action="store_true",
                    help="skip the SIRT run with the voxel-driven backprojector")
    ap.add_argument("--no-cylinder", action="store_true",
                    help="skip the SIRT run on the aligned cylindrical domain")
    ap.add_argument("--no-bf16", action="store_true",
                    help="skip the repeat of the SIRT run with BF16 storage")
    ap.add_argument("--no-helical", action="store_true",
                    help="skip the helical / sub-view / warp configuration")
    ap.add_argument("--no-autograd", action="store_true",
                    help="skip the differentiable-loss configuration")
    ap.add_argument("--no-unet", action="store_true",
                    help="skip the U-Net forward / training-step timing")
    args = ap.parse_args()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path "
              "(--gpus %d requested)" % args.gpus, file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_2609_30166_amd import Geometry
    from synth.configs import make_config, make_phantom

    dev = torch.device("cuda", 0)
    _log("achievable bandwidth (stream copy) ...")
    bw = achievable_bandwidth(dev)
    _log("copy: %.0f GB/s" % bw)
    cfg = make_config("full", n_proj=args.n_proj)
    _log("phantom 512^3 ...")
    x, _ = make_phantom(cfg, seed=0)
    g = Geometry(cfg.P, cfg.n_u, cfg.n_v, cfg.shape, cfg.step, device=dev)
    n_s = g.sample_count()
    _log("samples per forward projection: %d" % n_s)
    xt = torch.from_numpy(x).to(dev)
    sdt = torch.float32 if args.dtype == "f32" else torch.bfloat16
    b = g.forward(xt if sdt == torch.float32 else xt.to(sdt), out_dtype=sdt)
    vol = torch.zeros(cfg.shape, dtype=torch.float32, device=dev)
    ws = g.workspace(gather_dtype=sdt)
    torch.cuda.synchronize()

    for i in range(args.warmup):
        g.sirt(vol, b, 1, gather_dtype=sdt, workspace=ws, norms=False)
        torch.cuda.synchronize()
        _log("warmup %d done" % i)

    g.profile(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        g.sirt(vol, b, 1, gather_dtype=sdt, workspace=ws, norms=False)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = g.profile_read()
    g.profile(False)
    _log("timed %d steps in %.3f s" % (args.steps, t1 - t0))
    norms = g.sirt(vol, b, 1, gather_dtype=sdt, workspace=ws)

    ms_step = 1e3 * (t1 - t0) / args.steps
    value = 2.0 * n_s * args.steps / (t1 - t0) / 1e9
    fp_ms = prof["forward"][0] / max(prof["forward"][1], 1)
    bp_ms = prof["back"][0] / max(prof["back"][1], 1)
    up_ms = prof["update"][0] / max(prof["update"][1], 1)
    dom, dom_ms = ("bp_brick_kernel", bp_ms) if bp_ms >= fp_ms else ("fp_kernel", fp_ms)

    def kernel_row(name, ms):
        gb = GATHER_BYTES[args.dtype] * n_s / (ms * 1e-3) / 1e9
        tops = ALU_OPS[name] * n_s / (ms * 1e-3) / 1e12
        hbm = measured_traffic(name, args.dtype)
        row = {"ms": ms, "gsamples_per_s": n_s / (ms * 1e-3) / 1e9,
               "alu_tops": tops, "alu_frac": tops / ALU_PEAK_TOPS,
               "hbm_bytes_per_launch": hbm,
               "hbm_GBps": None if hbm is None else hbm / (ms * 1e-3) / 1e9,
               "l2_hit_rate": l2_hit_rate(name, args.dtype),
               "gather_equiv_GBps": gb, "gather_equiv_frac_of_achievable": gb / bw}
        if name == "bp_brick_kernel":
            lds = 8 * n_s / (ms * 1e-3) / 1e12
            row["lds_atomic_tops"] = lds
            row["lds_atomic_frac"] = lds / LDS_ATOMIC_PEAK_TOPS
        rec = counter_record(name, args.dtype)
        if rec is not None and "sq_insts_valu" in rec:
            # issue counters per launch (summed over the chip) against this
            # run's launch time: VALU wave-instructions per CU per clock, LDS
            # wave-instructions per CU per clock, bank-conflict cycles as a
            # fraction of every CU's cycles
            cu_clk = 256 * ms * 1e-3 * CLOCK_HZ
            row["counters"] = {"valu_per_cu_clock": rec["sq_insts_valu"] / cu_clk,
                               "lds_per_cu_clock": rec["sq_insts_lds"] / cu_clk,
                               "lds_bank_conflict_frac": rec["sq_lds_bank_conflict"] / cu_clk,
                               # LDS pipe: 4 clocks per wave instruction (64 lanes x 8 B
                               # at 128 B per clock) plus the bank-conflict clocks
                               "lds_busy_est": (4 * rec["sq_insts_lds"] +
                                                rec["sq_lds_bank_conflict"]) / cu_clk}
            if "ta_busy_sum" in rec:
                # texture addresser (one per CU): busy, and stalled waiting on the L1
                row["counters"]["ta_busy"] = rec["ta_busy_sum"] / cu_clk
                row["counters"]["ta_stalled_by_l1"] = rec["ta_addr_stalled_by_tc_sum"] / cu_clk
        return row

    kernels = {"fp_kernel": kernel_row("fp_kernel", fp_ms),
               "bp_brick_kernel": kernel_row("bp_brick_kernel", bp_ms)}
    d = kernels[dom]
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "Gsamples/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.dtype,
        "data": "synthetic (seeded 512^3 ellipsoid+cylinder phantom, noise-free)",
        "config": {
            "workload": "SIRT iteration, 512^3 volume, 720 circular cone-beam projections of "
                        "768x768, step 0.5 voxel (FP with fused correction + exact-transpose BP "
                        "+ update)",
            "samples_per_fp": n_s,
            "fp_ms": fp_ms, "bp_ms": bp_ms, "update_ms": up_ms,
            "sirt_iterations_per_s": 1e3 / ms_step,
            "residual_norm_after": float(norms[0]),
        },
        "roofline": {
            "bound": "alu",
            "kernel": dom,
            "achieved": d["alu_tops"],
            "peak": ALU_PEAK_TOPS,
            "unit": "Tops/s",
            "frac": d["alu_tops"] / ALU_PEAK_TOPS,
            "traffic": d["hbm_bytes_per_launch"],
            "basis": "%d algorithmic FP32 VALU lane operations per sample x %d samples per "
                     "launch / mean launch time; peak = 256 CUs x 4 SIMDs x 32 lanes x 2.4 GHz "
                     "(fp32 vector 157.3 TFLOP/s counting an FMA as 2)" % (ALU_OPS[dom], n_s),
            "l2_hit_rate": d["l2_hit_rate"],
            "hbm_GBps": d["hbm_GBps"],
            "counters": d.get("counters"),
        },
        "kernels": kernels,
        "gather_equivalent": {
            "definition": "%d B per sample (8 voxel reads or accumulations) x samples / launch "
                          "time, against the achievable HBM bandwidth of a stream copy in the "
                          "same run; the target is 0.6" % GATHER_BYTES[args.dtype],
            "bw_achievable_GBps": bw,
            "bw_achievable_frac_of_8TBps": bw / HBM_PEAK_GBS,
            "bp_frac": kernels["bp_brick_kernel"]["gather_equiv_frac_of_achievable"],
            "fp_frac": kernels["fp_kernel"]["gather_equiv_frac_of_achievable"],
            "step_frac": GATHER_BYTES[args.dtype] * 2 * n_s / (ms_step * 1e-3) / 1e9 / bw,
        },
    }
    y_or = views_or = None
    if args.cpu_views > 0:
        _log("cpu baseline (oracle) ...")
        out["cpu_baseline"], y_or, views_or = cpu_baseline(cfg, x, args.cpu_views)
    if not args.no_bf16:
        _log("SIRT with BF16 storage ...")
        if y_or is None:
            import oracle
            views_or = [0, 180]
            y_or = oracle.forward(cfg.P, cfg.shape, cfg.n_u, cfg.n_v, x.astype(np.float64),
                                  cfg.step, views=views_or)
        out["bf16"] = bf16_run(g, xt, b, vol, y_or, views_or, args)
    if not args.no_voxel_bp:
        _log("SIRT with the voxel-driven backprojector ...")
        out["voxel_bp"] = voxel_bp_comparison(g, b, sdt, xt, vol, norms, args, bp_ms, ms_step)
    if args.copy_calibrate:
        copy_calibration(dev)
    del b, vol, ws, xt
    g.close()
    torch.cuda.empty_cache()
    if not args.no_cylinder:
        _log("SIRT on the aligned cylindrical domain ...")
        out["cylinder"] = cylinder_sirt(dev, cfg, args)
        torch.cuda.empty_cache()
    if not args.no_helical:
        _log("helical scan with sub-views and warp ...")
        out["helical"] = helical_run(dev, args)
        torch.cuda.empty_cache()
    if not args.no_autograd:
        _log("differentiable loss ...")
        out["autograd"] = autograd_run(dev, args)
        torch.cuda.empty_cache()
    if not args.no_unet:
        _log("U-Net forward and training step ...")
        out["unet"] = unet_run(dev, args)
        torch.cuda.empty_cache()
    if not args.no_learned:
        _log("learned pipeline vs SIRT-50 ...")
        out["time_to_psnr"] = time_to_psnr(dev)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
