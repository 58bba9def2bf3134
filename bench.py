#!/usr/bin/env python3
"""Benchmark of the rendering hot path on one MI355X.

One step = forward + backward of the whole path (preprocess, depth sort,
count scan, key emission, pair sort, tile ranges, forward walk with Top-K
list, Top-K feature blend, feature backward, backward walk, preprocess
backward) over one 1920x1080 frame of a 1M-surfel plane-structured scene with
128-d FP32 features, K = 16, exact-ellipse tile lists.  Inputs are synthetic
(seeded) and already resident in HBM; workspaces and outputs are allocated
before the timed region.

Prints ONE JSON line.  `value` is fwd+bwd it/s of the Top-K + precise-tile
form; the same line carries the forward FPS, the dense-blend + AABB form on
the same GPU (the factor the paper's Sec. 5 is about), the Table-3-style
ablation, per-stage times from HIP events on the render stream, the roofline
of the dominant kernel and the CPU oracle timed on a bounded sample.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "fwd FPS & fwd+bwd it/s, 1080p, 1M surfels, 128-d feat, Top-K vs full blend"
WORKLOAD = "planes1m_1080p"

# MI355X published peaks (dense; no sparsity)
HBM_PEAK_GBS = 8000.0
FP32_VALU_PEAK_TFLOPS = 78.6   # 256 CU x 4 SIMD x 16 lanes x 2 flop x 2.4 GHz, unpacked FP32 FMA

# Algorithmic work per unit of the walks (what the method must compute, not
# what the kernels happen to issue)
FLOP_PER_EVAL = 17.0       # one pixel x list entry: FP64 centred offset 2, u' 3, v' 3, w' 4, rho w'^2 3, 9 w'^2 test 2
FLOP_PER_CONTRIB = 26.0    # contributor: 1/w', u, v, rho, exp, alpha, clamp, T', weight, 7 blend FMAs, depth, list test
BWD_FLOP_PER_EVAL = 17.0   # backward: the same test for each entry up to the pixel's last contributor
BWD_FLOP_PER_CONTRIB = 70.0  # backward contributor: T recovery, e_i, d alpha, d rho, du, dv, dz, 17 terms, suffix


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default=WORKLOAD)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-ablation", action="store_true")
    ap.add_argument("--cpu-tiles", type=int, default=1200)
    ap.add_argument("--no-batch", action="store_true", help="skip the 8-camera batched workload")
    ap.add_argument("--launch", default=None,
                    help="schedule,bwd_schedule,blend_pass,bwd_pass[,tile_w] for the headline form "
                         "(default: the library's autotuner)")
    ap.add_argument("--table", action="store_true",
                    help="the configuration table: every configuration on the tile-mode x blend grid, quality "
                         "proxy, oracle timings (one JSON line)")
    ap.add_argument("--headline-only", action="store_true",
                    help="time only the headline fwd+bwd step (for profiler runs: every kernel of the run is "
                         "one of its dispatches)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run a plain 1 GiB device copy (reference for HBM byte counters)")
    return ap.parse_args()


def calibrate_copy():
    """A plain device-to-device copy of known size: rocprofv3 --pmc FETCH_SIZE /
    WRITE_SIZE on this run gives the counters' scale for 1 GiB read + 1 GiB written."""
    import torch
    n = 1 << 28  # 2^28 float32 = 1 GiB
    a = torch.ones(n, dtype=torch.float32, device="cuda:0")
    b = torch.empty_like(a)
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes": 4 * n, "launches": 3}), flush=True)


class Form:
    """One (tile mode, blend) configuration with preallocated buffers."""

    def __init__(self, psm, t, cam, K, tile_mode, blend, gout, device, launch=None, tune=False, flags=0,
                 tune_bwd=True):
        import torch
        self.psm, self.t, self.K = psm, t, K
        self.tile_mode, self.blend = tile_mode, blend
        self.cam = psm.camera_struct(cam)
        self.cfg = psm.config_struct(K, tile_mode, blend, psm.FLAG_NO_SYNC | psm.FLAG_PROFILE | flags)
        self.s = psm._surfels(t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"])
        # the pairs each tile shape needs (only the launch's shape, or every
        # shape when the autotuner picks it), and a workspace that fits them
        shapes = TILE_WIDTHS if (tune and launch is None) else ((launch[4] if launch and len(launch) > 4 else 0),)
        need = 0
        for tw in shapes:
            _, ws = psm.forward(t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"], self.cam, K,
                                tile_mode, blend, flags=flags, launch=(0, 0, 0, 0, tw))
            st = psm.read_stats(ws, self.s.n, self.cam, psm.config_struct(K, tile_mode, blend, flags, tile_w=tw),
                                self.s.c, ws.capacity)
            need = max(need, int(st.pairs_required))
            del ws
        cap = int(need * 1.05 + 4096)
        self.ws = psm.alloc_workspace_shapes(self.s.n, [self.cam], self.cfg, self.s.c, cap, device, shapes)
        feature_only = bool(flags & psm.FLAG_FEATURE_ONLY)
        self.out = psm.alloc_images(self.cam, self.s.c, device, feature_only=feature_only)
        if feature_only:  # only the feature map is rendered, so only its upstream gradient
            gout = {k: (v if k == "feat" else None) for k, v in gout.items()}
        n, c = self.s.n, self.s.c
        z = lambda *sh: torch.empty(*sh, dtype=torch.float32, device=device)
        self.grads = {"means": z(n, 3), "scales": z(n, 2), "quats": z(n, 4), "opacity": z(n), "rgb": z(n, 3),
                      "feat": z(n, c)}
        self.gout = gout
        self.ctx = psm.context(device.index or 0)
        self.tuned_ms = None
        if launch is not None:
            self.cfg.schedule, self.cfg.bwd_schedule, self.cfg.blend_pass, self.cfg.bwd_pass = launch[:4]
            self.cfg.tile_w = launch[4] if len(launch) > 4 else 0
        elif tune:
            tcfg = psm.config_struct(K, tile_mode, blend)
            out = dict(self.out)
            # the median of 9 timed runs per candidate (3 leave the ~1 ms
            # forwards to noise); tuned for what is timed: fwd+bwd, or the
            # forward alone
            self.tuned_ms = psm.autotune(self.ctx, self.s, psm.camera_array([self.cam]), tcfg, self.ws, out,
                                         self.gout if tune_bwd else None, self.grads if tune_bwd else None,
                                         reps=9, cache=False)
            self.cfg.schedule, self.cfg.bwd_schedule = tcfg.schedule, tcfg.bwd_schedule
            self.cfg.blend_pass, self.cfg.bwd_pass, self.cfg.tile_w = tcfg.blend_pass, tcfg.bwd_pass, tcfg.tile_w

    def launch(self):
        """(schedule, bwd_schedule, blend_pass, bwd_pass, tile_w) in use."""
        return (int(self.cfg.schedule), int(self.cfg.bwd_schedule), int(self.cfg.blend_pass or 32),
                int(self.cfg.bwd_pass or 16), int(self.cfg.tile_w or 16))

    def step(self, bwd: bool):
        self.psm.forward_into(self.ctx, self.s, self.cam, self.cfg, self.ws, self.out)
        if bwd:
            self.psm.backward_into(self.ctx, self.s, self.cam, self.cfg, self.ws, self.gout, self.grads)

    def stats(self):
        return self.psm.read_stats(self.ws, self.s.n, self.cam, self.cfg, self.s.c, self.ws.capacity)


def timed(form, bwd, steps, warmup):
    import torch
    psm = form.psm
    for _ in range(warmup):
        form.step(bwd)
    torch.cuda.synchronize()
    psm.profile_reset(form.ctx)
    t0 = time.perf_counter()
    for _ in range(steps):
        form.step(bwd)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    prof = psm.profile_read(form.ctx)
    st = form.stats()
    if st.pairs_required > st.pair_capacity:
        raise RuntimeError("pair capacity exceeded inside the timed region")
    per_stage = {k: v[0] / max(v[1], 1) for k, v in prof.items() if v[1] > 0}
    return el * 1000.0 / steps, per_stage, st


def kernel_source_hash() -> str:
    """SHA-256 over the kernel sources (csrc/*.hip, csrc/*.h), in name order."""
    import glob
    import hashlib
    h = hashlib.sha256()
    for f in sorted(glob.glob(os.path.join(ROOT, "paper_2604_10982_amd", "csrc", "*.h")) +
                    glob.glob(os.path.join(ROOT, "paper_2604_10982_amd", "csrc", "*.hip"))):
        h.update(os.path.basename(f).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(stage: str, workload: str, launch=None):
    """HBM bytes per launch (read + written) of a stage's kernel from the
    committed rocprofv3 counter summary, or None when there is none, the
    kernel sources changed since the counters were taken, or the counters
    were taken with other launch choices."""
    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{stage}_{workload}.md")
    if not os.path.exists(path):
        return None
    fields = {}
    with open(path) as f:
        for line in f:
            if line.startswith("- ") and ":" in line:
                k, v = line[2:].split(":", 1)
                fields[k.strip()] = v.strip().strip("`")
    if fields.get("kernel sources sha256") != kernel_source_hash():
        return None
    if launch is not None:
        # only the launch choices that change this stage's kernel must agree
        # (schedule, bwd schedule, blend pass, bwd pass, tile width)
        rel = {"walk": (0, 4), "feature_blend": (2, 4), "bwd_feature": (1, 3, 4), "bwd_walk": (1, 4)}.get(stage, (4,))
        try:
            rec = [int(v) for v in fields.get("launch choice", "").split(",")]
            if len(rec) < 5 or any(rec[i] != int(launch[i]) for i in rel):
                return None
        except ValueError:
            return None
    try:
        return float(fields["bytes per launch (read + write)"])
    except (KeyError, ValueError):
        return None


def stage_work(name, st, K, C, b, S):
    """Algorithmic work of one launch of a stage: ("flop", F) for the walks
    (ALU-bound), ("byte", B) for the streaming stages.  U = distinct selected
    surfels, SP = (tile, surfel) pairs with a selection (the feature rows the
    Top-K adjoint writes and the reduction reads back; 0 for the dense blend,
    whose partial rows are left out), b = bytes per stored feature element."""
    P, N, U = st.pairs, st.n, max(st.selected_unique, 0)
    SP = max(getattr(st, "selected_pairs", -1), 0)
    if name == "walk":
        return "flop", FLOP_PER_EVAL * st.pairs_walked + FLOP_PER_CONTRIB * st.contributors
    if name == "bwd_walk":
        # the backward evaluates each pixel's list up to its last contributor
        return "flop", BWD_FLOP_PER_EVAL * st.bwd_entries + BWD_FLOP_PER_CONTRIB * st.contributors
    bytes_by = {
        "feature_blend": S * (8 * K + 4 * C) + U * C * b,
        "bwd_feature": S * (8 * K + 4 * C + 4 * K) + U * C * b + SP * 4 * C,
        "preprocess": N * (40 + 12) + st.visible * (64 + 48) + N * 12,
        "depth_sort": N * 8 * 2,
        "pair_sort": P * 8 * 2,
        "emit": P * 8 + st.visible * 56,
        "count_scan": N * 8,
        "bwd_reduce": N * (64 + 40 + 52) + P * 80 + P + SP * 4 * C + N * 4 * C,
        "ranges": P * 4,
        "fill": 0,
    }
    return "byte", bytes_by.get(name, 0)


def stage_table(stages, st, K, C, b, S):
    """Every stage of the step against its roofline: HBM GB/s for the
    streaming stages, TFLOP/s of the unpacked vector ALU for the walks."""
    out = {}
    for name, ms in stages.items():
        kind, w = stage_work(name, st, K, C, b, S)
        if kind == "flop":
            a = w / (ms * 1e-3) / 1e12
            out[name] = {"ms": ms, "bound": "alu", "tflops": a, "frac": a / FP32_VALU_PEAK_TFLOPS}
        elif w:
            a = w / (ms * 1e-3) / 1e9
            out[name] = {"ms": ms, "bound": "hbm", "gbs": a, "frac": a / HBM_PEAK_GBS}
        else:
            out[name] = {"ms": ms}
    return out


def step_bytes(st, K, C, b, S, bwd=True):
    """Algorithmic HBM bytes of one forward (+ backward): the parameters, the
    pair list written and read once, the selected features, the FP32 maps,
    and for the backward the upstream maps, the saved per-pixel state and the
    FP32 gradients."""
    N, P, U = st.n, st.pairs, max(st.selected_unique, 0)
    fwd = N * 40 + st.visible * 12 + P * 24 + U * C * b + S * (32 + 4 * C)
    if not bwd:
        return fwd
    return fwd + S * (32 + 4 * C) + S * (8 + 8 * K) + P * 24 + U * C * b + N * 4 * (13 + C)


def roofline(stages, st, K, C, S, b, workload=WORKLOAD, launch=None):
    """Roofline object for the dominant stage of the step."""
    name = max(stages, key=stages.get)
    ms = stages[name]
    traffic = measured_traffic(name, workload, launch)
    kind, w = stage_work(name, st, K, C, b, S)
    if kind == "flop":
        a = w / (ms * 1e-3) / 1e12
        return {"kernel": name, "bound": "alu", "achieved": a, "peak": FP32_VALU_PEAK_TFLOPS, "unit": "TFLOP/s",
                "frac": a / FP32_VALU_PEAK_TFLOPS, "traffic": traffic, "ms": ms,
                "work": {"pairs_walked": st.pairs_walked, "bwd_entries": st.bwd_entries,
                         "contributors": st.contributors, "flops": w}}
    a = w / (ms * 1e-3) / 1e9
    return {"kernel": name, "bound": "hbm", "achieved": a, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": a / HBM_PEAK_GBS, "traffic": traffic, "ms": ms, "work": {"bytes": w}}


def batch_workload(psm, scenes, steps, warmup, k=16):
    """The batched workload: a shared 2M-surfel street scene with 128-d FP16
    features seen by 8 cameras of uneven resolution, fwd+bwd in one call per
    stage, K = k.  Launch choices come from the library's autotuner; the step
    is also captured in a HIP graph and replayed."""
    import numpy as np
    import torch
    device = torch.device("cuda:0")
    sc, cams, K, dtype = scenes.batch_config(k=k)
    t = {k: torch.tensor(getattr(sc, k), device=device) for k in ("means", "scales", "quats", "opacity", "rgb")}
    t["feat"] = torch.tensor(sc.feat, device=device).to(torch.float16).contiguous()
    args = (t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"])
    carr = psm.camera_array(cams)
    need = 0
    for tw in TILE_WIDTHS:  # pairs of every tile shape the autotuner times
        c0 = psm.config_struct(K, tile_w=tw)
        _, ws0, _ = psm.forward_batch(*args, carr, K, cfg=c0)
        need = max(need, int(psm.read_stats_batch(ws0, carr, c0).pairs_required))
        del ws0
    cfg = psm.config_struct(K, "ellipse", "topk", psm.FLAG_NO_SYNC | psm.FLAG_PROFILE)
    ws = psm.alloc_workspace_shapes(sc.n, list(cams), cfg, sc.c, int(need * 1.05) + 4096, device, TILE_WIDTHS)
    out = psm.alloc_images_batch(carr, sc.c, device)
    P = psm.total_pixels(carr)
    g = torch.Generator(device=device).manual_seed(1)
    gout = {"rgb": torch.randn(P, 3, device=device, generator=g), "depth": torch.randn(P, device=device, generator=g),
            "normal": torch.randn(P, 3, device=device, generator=g), "alpha": torch.randn(P, device=device, generator=g),
            "feat": torch.randn(P, sc.c, device=device, generator=g)}
    n = sc.n
    z = lambda *sh: torch.empty(*sh, dtype=torch.float32, device=device)
    grads = {"means": z(n, 3), "scales": z(n, 2), "quats": z(n, 4), "opacity": z(n), "rgb": z(n, 3),
             "feat": z(n, sc.c)}
    s = psm._surfels(*args)
    ctx = psm.context(0)
    tune_cfg = psm.config_struct(K, "ellipse", "topk")
    tuned_ms = psm.autotune(ctx, s, carr, tune_cfg, ws, out, gout, grads, reps=9, cache=False)
    cfg.schedule, cfg.bwd_schedule = tune_cfg.schedule, tune_cfg.bwd_schedule
    cfg.blend_pass, cfg.bwd_pass, cfg.tile_w = tune_cfg.blend_pass, tune_cfg.bwd_pass, tune_cfg.tile_w

    def step(c):
        psm.forward_batch_into(ctx, s, carr, c, ws, out)
        psm.backward_batch_into(ctx, s, carr, c, ws, gout, grads)

    for _ in range(warmup):
        step(cfg)
    torch.cuda.synchronize()
    psm.profile_reset(ctx)
    t0 = time.perf_counter()
    for _ in range(steps):
        step(cfg)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1000.0 / steps
    prof = psm.profile_read(ctx)
    stages = {k: v[0] / max(v[1], 1) for k, v in prof.items() if v[1] > 0}
    st = psm.read_stats_batch(ws, carr, cfg)
    if st.pairs_required > st.pair_capacity:
        raise RuntimeError("pair capacity exceeded in the batched workload")
    # the same step captured once and replayed
    gcfg = psm.config_struct(K, "ellipse", "topk", psm.FLAG_NO_SYNC, tune_cfg.schedule, tune_cfg.blend_pass,
                             tune_cfg.bwd_pass, tune_cfg.bwd_schedule, tune_cfg.tile_w)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(gcfg)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(gcfg)
    for _ in range(warmup):
        graph.replay()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        graph.replay()
    torch.cuda.synchronize()
    gms = (time.perf_counter() - t0) * 1000.0 / steps
    # forward alone (eager)
    for _ in range(warmup):
        psm.forward_batch_into(ctx, s, carr, cfg, ws, out)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        psm.forward_batch_into(ctx, s, carr, cfg, ws, out)
    torch.cuda.synchronize()
    fms = (time.perf_counter() - t0) * 1000.0 / steps
    return {"workload": f"street40 scene, {n} surfels, 128-d f16 features, K={K}, 8 cameras "
                        + ", ".join(f"{c.width}x{c.height}" for c in cams),
            "k": K, "pixels": P, "fwd_ms": fms, "fwd_fps": 1000.0 / fms,
            "fwd_bwd_ms": ms, "fwd_bwd_its": 1000.0 / ms, "graph_replay_ms": gms,
            "graph_replay_its": 1000.0 / gms, "autotuned": {"schedule": ["grid", "persistent"][tune_cfg.schedule],
                                                           "bwd_schedule": ["grid", "persistent"][tune_cfg.bwd_schedule],
                                                           "blend_pass": tune_cfg.blend_pass,
                                                           "bwd_pass": tune_cfg.bwd_pass,
                                                           "tile": f"{tune_cfg.tile_w}x{256 // tune_cfg.tile_w}",
                                                           "tuned_ms": tuned_ms},
            "pairs": int(st.pairs), "stages_ms": stages,
            "stage_roofline": stage_table(stages, st, K, sc.c, 2, P)}


def labels_workload(psm, means, steps, warmup, nq=64, c=32):
    """Instance labels of the headline scene's surfels from nq localized
    queries (c-d FP32 instance features): forward (MFMA logits + softmax) and
    backward, timed with HIP events on the stream."""
    import numpy as np
    import torch
    device = means.device
    n = means.shape[0]
    rng = np.random.default_rng(3)
    f_ins = torch.tensor((rng.standard_normal((n, c)) * 3.0 / np.sqrt(c)).astype(np.float32), device=device)
    q_feat = torch.tensor((rng.standard_normal((nq, c)) * 3.0 / np.sqrt(c)).astype(np.float32), device=device)
    q_mean = torch.tensor(np.c_[rng.uniform(-12, 12, nq), rng.uniform(-6, 1.6, nq), rng.uniform(2, 60, nq)]
                          .astype(np.float32), device=device)
    prec = np.tile(np.array([0.25, 0, 0, 0.25, 0, 0.25], np.float32), (nq, 1))
    q_prec = torch.tensor(prec, device=device)
    ld = psm.label_width(nq)
    out = torch.empty(n, ld, device=device)
    dl = torch.randn(n, ld, device=device)
    fwd = lambda: psm.instance_labels_into(means, f_ins, q_feat, q_mean, q_prec, out, ld)
    bwd = lambda: psm.instance_labels_backward(means, f_ins, q_feat, q_mean, q_prec, dl, ld)
    res = {}
    for name, fn in (("fwd", fwd), ("bwd", bwd)):
        for _ in range(warmup):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        for _ in range(steps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        res[name + "_ms"] = e0.elapsed_time(e1) / steps
    bytes_fwd = n * (12 + 4 * c + 4 * ld)
    flops_fwd = 2.0 * n * nq * c
    res.update({"surfels": n, "queries": nq, "feat_dim": c,
                "fwd_hbm_gbs": bytes_fwd / (res["fwd_ms"] * 1e-3) / 1e9, "fwd_hbm_frac": bytes_fwd / (res["fwd_ms"] * 1e-3) / 1e9 / HBM_PEAK_GBS,
                "fwd_mfma_tflops": flops_fwd / (res["fwd_ms"] * 1e-3) / 1e12,
                "note": "labels (eqs. (4)-(7)) of every surfel; bytes = means + features in + labels out"})
    return res


FP32_MFMA_PEAK_TFLOPS = 157.3  # MI355X dense FP32 matrix


def attention_workload(psm, steps, warmup, nq=64, c=32, d=32):
    """Frustum-local cross-attention (eqs. (9)-(11)) of nq queries over the
    surfels of a 2M-surfel street scene that meet a 1920x1080 camera's
    frustum; c-d FP32 instance features, d-d projections.  Timed with HIP
    events on the stream (cull + compaction + projections + attention)."""
    import numpy as np
    import torch
    from paper_2604_10982_amd import scenes
    device = torch.device("cuda:0")
    sc = scenes.street40(2_000_000, 8, seed=1)
    cam = scenes.street_cameras()[-1]
    rng = np.random.default_rng(4)
    T = lambda a: torch.tensor(np.ascontiguousarray(a, np.float32), device=device)
    means, scales = T(sc.means), T(sc.scales)
    feat = T(rng.standard_normal((sc.n, c)) * 0.8)
    q = T(rng.standard_normal((nq, c)))
    wq, wk, wv = (T(rng.standard_normal((c, d)) / np.sqrt(c)) for _ in range(3))
    run = lambda: psm.frustum_attention(means, scales, feat, q, wq, wk, wv, cam, 16.0)
    _, act = psm.frustum_attention(means, scales, feat, q, wq, wk, wv, cam, 16.0, return_active=True)
    m = int(act.sum().item())
    for _ in range(warmup):
        run()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(steps):
        run()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    # per active key: K and V projections (2 c d MACs), scores and P V (2 nq d MACs)
    flops = 2.0 * m * (2 * c * d + 2 * nq * d)
    return {"ms": ms, "surfels": sc.n, "active": m, "queries": nq, "feat_dim": c, "proj_dim": d,
            "mfma_tflops": flops / (ms * 1e-3) / 1e12, "mfma_frac": flops / (ms * 1e-3) / 1e12 / FP32_MFMA_PEAK_TFLOPS,
            "note": "psm_frustum_attention: 99% frustum cull, compaction, FP32 MFMA projections, scores, online "
                    "softmax and P V; flops = 2 M (2 c d + 2 n_q d) over the M active surfels"}


def geometry_workload(psm, means, scales, quats, sc, steps, warmup, k=512):
    """SOGMM geometric loss (eq. (3), eq. (13), L_iso) of the headline scene's
    surfels against a k-component synthetic plane prior: MAP assignment, both
    losses and their gradients, timed with HIP events on the stream."""
    import numpy as np
    import torch
    from paper_2604_10982_amd import scenes
    gm = [torch.tensor(a, device=means.device) for a in scenes.plane_gmm(sc, k, seed=3)]
    run = lambda: psm.geometry_loss(means, scales, quats, gm[0], gm[1], gm[2], 0.4)
    for _ in range(warmup):
        run()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(steps):
        run()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    n = int(means.shape[0])
    flops = 23.0 * n * k   # per (surfel, component) score: 3 sub, 9 mul, 8 add (FP32), 3 for the minimum
    return {"ms": ms, "surfels": n, "components": k, "surfels_per_s": n / (ms * 1e-3),
            "alu_tflops": flops / (ms * 1e-3) / 1e12, "alu_frac": flops / (ms * 1e-3) / 1e12 / FP32_VALU_PEAK_TFLOPS,
            "note": "psm_geometry_loss: MAP component by a matrix-core bound and exact FP32 scores of the contenders "
                    "(alu_tflops: the operations of a full scan over the time), FP64 loss terms and "
                    "gradients, ordered FP64 sums"}


def cpu_baseline(sc, cam, K, feat64, tiles):
    """The FP64 oracle (test infrastructure) on a bounded sample of the same
    frame: forward + backward of the pixels of `tiles` random 16x16 tiles.
    The whole-scene key stage and binning are timed separately and counted
    once per frame; the per-pixel cost is scaled to the full frame."""
    import numpy as np
    from oracle import oracle as O
    from paper_2604_10982_amd import scenes
    rng = np.random.default_rng(0)
    ntx, nty = (cam.width + 15) // 16, (cam.height + 15) // 16
    pick = rng.choice(ntx * nty, tiles, replace=False)
    pix = []
    for t in pick:
        ty, tx = divmod(int(t), ntx)
        ys, xs = np.mgrid[ty * 16:min(ty * 16 + 16, cam.height), tx * 16:min(tx * 16 + 16, cam.width)]
        pix.append((ys * cam.width + xs).ravel())
    pix = np.concatenate(pix).astype(np.int64)
    one = pix[:1]
    t0 = time.perf_counter()
    O.render(sc, cam, K, O.TOPK, feat=feat64, pix=one)
    t_prep = time.perf_counter() - t0
    t0 = time.perf_counter()
    O.render(sc, cam, K, O.TOPK, feat=feat64, pix=pix)
    t_fwd = time.perf_counter() - t0
    g = scenes.upstream(cam.height, cam.width, sc.c, seed=1)
    gs = {k: v.reshape(cam.width * cam.height, -1)[pix] for k, v in g.items()}
    t0 = time.perf_counter()
    O.backward(sc, cam, gs, K=K, blend=O.TOPK, feat=feat64, pix=pix)
    t_bwd = time.perf_counter() - t0
    S = cam.width * cam.height
    scale = S / len(pix)
    frame = 2 * t_prep + (t_fwd - t_prep) * scale + (t_bwd - t_prep) * scale
    return {"value": 1.0 / frame, "unit": "it/s", "cores": O.num_threads(), "kind": "oracle",
            "sample": (f"FP64 oracle fwd+bwd (Top-K, exact ellipse) on {tiles} random 16x16 tiles ({len(pix)} px) "
                       f"of the same frame; whole-scene key stage + binning {t_prep:.2f}s counted once per pass, "
                       f"per-pixel cost scaled to {S} px"),
            "sample_seconds": {"prepare": t_prep, "fwd": t_fwd, "bwd": t_bwd}, "est_frame_s": frame}


TILE_WIDTHS = (8, 16, 32, 64)
TABLE_CONFIGS = (("c1_box2k", False), ("c2_planes200k", False), ("c3_planes500k", True),
                 ("c4_street1m", True), ("room_1296x968", True))
TABLE_GRID = (("sphere", "full"), ("aabb", "full"), ("ellipse", "full"),
              ("sphere", "topk"), ("aabb", "topk"), ("ellipse", "topk"))


def host_cpu():
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"model": model, "logical_cpus": os.cpu_count()}


def table_cpu_leg(sc, cam, K, feat64, name, bwd):
    """The FP64 oracle (as it stands) on the configuration: the whole frame
    for the two small configurations (all threads, then one), forward and,
    where the configuration has one, backward; a sample of 200 random tiles
    for the large ones, scaled to the frame as in cpu_baseline."""
    from oracle import oracle as O
    from paper_2604_10982_amd import scenes
    threads = O.num_threads()
    out = {"threads": threads}
    if name in ("c1_box2k", "c2_planes200k"):
        for label, nt in (("all_threads", threads), ("one_thread", 1)):
            O.set_threads(nt)
            t0 = time.perf_counter()
            O.render(sc, cam, K, O.TOPK, feat=feat64)
            out[label] = {"threads": nt, "fwd_s": time.perf_counter() - t0}
            if bwd or name == "c1_box2k":
                g = scenes.upstream(cam.height, cam.width, sc.c, seed=1)
                t0 = time.perf_counter()
                O.backward(sc, cam, g, K=K, blend=O.TOPK, feat=feat64)
                out[label]["bwd_s"] = time.perf_counter() - t0
        O.set_threads(threads)
        out["kind"] = "whole frame"
        return out
    r = cpu_baseline(sc, cam, K, feat64, 200)
    out.update({"kind": "sample", "est_frame_s": r["est_frame_s"], "sample": r["sample"]})
    return out


def run_table(psm, scenes, steps, warmup, with_cpu):
    """Every configuration on the {dense, Top-K} x {square, AABB, ellipse}
    grid: forward FPS, fwd+bwd it/s where the configuration has a backward,
    pairs and work counters, every stage against its roofline, the quality
    proxy of the Top-K blend against the dense blend, and the oracle timed on
    the host cores."""
    import numpy as np
    import torch
    device = torch.device("cuda:0")
    res = {"host_cpu": host_cpu(), "configs": {}}
    for name, bwd in TABLE_CONFIGS:
        sc, cam, K, dtype = scenes.config(name)
        tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
        fbytes = {"f32": 4, "f16": 2, "bf16": 2}[dtype]
        t = {k: torch.tensor(getattr(sc, k), device=device) for k in ("means", "scales", "quats", "opacity", "rgb")}
        t["feat"] = torch.tensor(sc.feat, device=device).to(tdt).contiguous()
        g = scenes.upstream(cam.height, cam.width, sc.c, seed=1)
        gout = {k: torch.tensor(v, device=device) for k, v in g.items()}
        del g
        S = cam.width * cam.height
        entry = {"surfels": sc.n, "width": cam.width, "height": cam.height, "feat_dim": sc.c, "dtype": dtype, "k": K,
                 "rows": {}}
        feats = {}
        for tm, bl in TABLE_GRID:
            f = Form(psm, t, cam, K, tm, bl, gout, device, tune=True, tune_bwd=bwd)
            ms_fwd, st_fwd, st = timed(f, False, steps, warmup)
            row = {"launch": f.launch(), "fwd_ms": ms_fwd, "fwd_fps": 1000.0 / ms_fwd, "pairs": int(st.pairs),
                   "pairs_per_tile": st.pairs / st.tiles, "pairs_walked": int(st.pairs_walked),
                   "contributors": int(st.contributors), "selected_unique": int(st.selected_unique),
                   "selections": int(st.selections), "selected_pairs": int(st.selected_pairs),
                   "bwd_entries": int(st.bwd_entries)}
            stages = st_fwd
            if bwd:
                ms_step, stages, _ = timed(f, True, steps, warmup)
                row.update({"fwd_bwd_ms": ms_step, "fwd_bwd_its": 1000.0 / ms_step,
                            "step_hbm_frac": step_bytes(st, K, sc.c, fbytes, S) / (ms_step * 1e-3) / 1e9
                            / HBM_PEAK_GBS})
            row["stage_roofline"] = stage_table(stages, st, K, sc.c, fbytes, S)
            if tm == "ellipse":
                f.step(False)
                feats[bl] = f.out["feat"].clone()
            entry["rows"][f"{bl}/{tm}"] = row
            print(f"[table] {name} {bl}/{tm}: fwd {ms_fwd:.3f} ms" + (f", fwd+bwd {row['fwd_bwd_ms']:.3f} ms"
                  if bwd else "") + f", pairs {st.pairs}", file=sys.stderr, flush=True)
            del f
            torch.cuda.empty_cache()
        fk, ff = feats["topk"].reshape(-1, sc.c), feats["full"].reshape(-1, sc.c)
        covered = ff.abs().sum(1) > 0
        entry["quality_proxy"] = {
            "rel_l2_topk_vs_full": float((fk - ff).norm() / ff.norm()),
            "argmax_agreement": float((fk[covered].argmax(1) == ff[covered].argmax(1)).float().mean()),
            "pixels": int(covered.sum())}
        entry["headline_factor"] = {
            "fwd": entry["rows"]["full/aabb"]["fwd_ms"] / entry["rows"]["topk/ellipse"]["fwd_ms"]}
        if bwd:
            entry["headline_factor"]["fwd_bwd"] = (entry["rows"]["full/aabb"]["fwd_bwd_ms"]
                                                   / entry["rows"]["topk/ellipse"]["fwd_bwd_ms"])
        del feats, fk, ff
        if with_cpu:
            feat64 = t["feat"].float().cpu().numpy().astype(np.float64)
            entry["oracle"] = table_cpu_leg(sc, cam, K, feat64, name, bwd)
            del feat64
        res["configs"][name] = entry
        del t, gout
        torch.cuda.empty_cache()
    # the batched workload (8 cameras, one launch per stage) at each K
    res["batch_8cam"] = {}
    for k in (8, 16, 32):
        res["batch_8cam"][f"k{k}"] = batch_workload(psm, scenes, steps, warmup, k=k)
        print(f"[table] batch 8 cameras K={k}: fwd+bwd {res['batch_8cam'][f'k{k}']['fwd_bwd_ms']:.3f} ms",
              file=sys.stderr, flush=True)
        torch.cuda.empty_cache()
    return res


def main():
    args = parse()
    if args.calibrate_copy:
        calibrate_copy()
        return
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) > 1:
        print("bench.py measures one GPU: the library has no multi-GPU path (a camera-sharded path would "
              "need one all-reduce of the surfel gradients per step). Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch

    from paper_2604_10982_amd import psm, scenes

    if not torch.cuda.is_available():
        raise SystemExit("bench.py needs a HIP device")
    device = torch.device("cuda:0")
    psm.lib()
    if args.table:
        print(json.dumps(run_table(psm, scenes, max(3, args.steps // 2), 2, not args.no_cpu_baseline)), flush=True)
        return
    sc, cam, K, dtype = scenes.config(args.workload)
    tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    t = {k: torch.tensor(getattr(sc, k), device=device) for k in ("means", "scales", "quats", "opacity", "rgb")}
    t["feat"] = torch.tensor(sc.feat, device=device).to(tdt).contiguous()
    g = scenes.upstream(cam.height, cam.width, sc.c, seed=1)
    gout = {k: torch.tensor(v, device=device) for k, v in g.items()}
    S = cam.width * cam.height
    fbytes = {"f32": 4, "f16": 2, "bf16": 2}[dtype]
    print(f"[bench] {args.workload}: n={sc.n} {cam.width}x{cam.height} C={sc.c} K={K} {dtype}", file=sys.stderr,
          flush=True)

    launch = tuple(int(v) for v in args.launch.split(",")) if args.launch else None
    head = Form(psm, t, cam, K, "ellipse", "topk", gout, device, launch=launch, tune=launch is None)
    print(f"[bench] launch choice (schedule, bwd_schedule, blend_pass, bwd_pass, tile_w): {head.launch()}",
          file=sys.stderr, flush=True)
    ms_step, stages, st = timed(head, True, args.steps, args.warmup)
    print(f"[bench] topk+ellipse fwd+bwd {ms_step:.3f} ms", file=sys.stderr, flush=True)
    if args.headline_only:
        print(json.dumps({"workload": args.workload, "ms_per_step": ms_step, "steps": args.steps,
                          "warmup": args.warmup, "launch": head.launch(), "stages_ms": stages,
                          "stage_roofline": stage_table(stages, st, K, sc.c, fbytes, S)}), flush=True)
        return
    ms_fwd, stages_fwd, _ = timed(head, False, args.steps, args.warmup)
    print(f"[bench] topk+ellipse fwd {ms_fwd:.3f} ms", file=sys.stderr, flush=True)
    head_launch = head.launch()
    head_tuned_ms = head.tuned_ms
    del head
    # exact work reduction: the opacity-aware footprint (same outputs, fewer pairs)
    opa = Form(psm, t, cam, K, "ellipse", "topk", gout, device, launch=head_launch, flags=psm.FLAG_OPACITY_FOOTPRINT)
    ms_opa, _, st_opa = timed(opa, True, args.steps, args.warmup)
    print(f"[bench] opacity-aware footprint fwd+bwd {ms_opa:.3f} ms, pairs {st_opa.pairs} (standard {st.pairs})",
          file=sys.stderr, flush=True)
    opacity_footprint = {"fwd_bwd_ms": ms_opa, "fwd_bwd_its": 1000.0 / ms_opa, "pairs": int(st_opa.pairs),
                         "pairs_standard": int(st.pairs),
                         "note": "PSM_FLAG_OPACITY_FOOTPRINT: tile footprint of rho <= min(9, 2 ln(255 o)); "
                                 "outputs and gradients bit-identical to the standard footprint"}
    del opa
    # exact work reduction: feature-only rendering stops a pixel once its Top-K set is final
    fo = Form(psm, t, cam, K, "ellipse", "topk", gout, device, launch=head_launch, flags=psm.FLAG_FEATURE_ONLY)
    ms_fo_step, stages_fo, st_fo = timed(fo, True, args.steps, args.warmup)
    ms_fo_fwd, _, _ = timed(fo, False, args.steps, args.warmup)
    print(f"[bench] feature-only fwd {ms_fo_fwd:.3f} ms, fwd+bwd {ms_fo_step:.3f} ms, contributors "
          f"{st_fo.contributors} (full walk {st.contributors})", file=sys.stderr, flush=True)
    feature_only = {"fwd_ms": ms_fo_fwd, "fwd_fps": 1000.0 / ms_fo_fwd, "fwd_bwd_ms": ms_fo_step,
                    "fwd_bwd_its": 1000.0 / ms_fo_step, "contributors": int(st_fo.contributors),
                    "contributors_full_walk": int(st.contributors), "walk_ms": stages_fo.get("walk"),
                    "note": "PSM_FLAG_FEATURE_ONLY: feature map and Top-K selection bit-identical to the full walk; "
                            "no RGB/depth/normal/alpha maps; backward of the feature loss"}
    del fo
    # renormalised Top-K (the selected weights rescaled to sum 1)
    rn = Form(psm, t, cam, K, "ellipse", "topk", gout, device, launch=head_launch, flags=psm.FLAG_TOPK_RENORM)
    ms_rn_step, _, _ = timed(rn, True, args.steps, args.warmup)
    ms_rn_fwd, _, _ = timed(rn, False, args.steps, args.warmup)
    print(f"[bench] renormalised Top-K fwd {ms_rn_fwd:.3f} ms, fwd+bwd {ms_rn_step:.3f} ms", file=sys.stderr,
          flush=True)
    topk_renorm = {"fwd_ms": ms_rn_fwd, "fwd_fps": 1000.0 / ms_rn_fwd, "fwd_bwd_ms": ms_rn_step,
                   "fwd_bwd_its": 1000.0 / ms_rn_step,
                   "note": "PSM_FLAG_TOPK_RENORM: feature map sum_sel w f / sum_sel w and its backward"}
    del rn
    # screen-space low-pass filter (the 2DGS variant of the surfel kernel)
    lpf = Form(psm, t, cam, K, "ellipse", "topk", gout, device, launch=head_launch, flags=psm.FLAG_LOWPASS)
    ms_lp_step, _, st_lp = timed(lpf, True, args.steps, args.warmup)
    ms_lp_fwd, _, _ = timed(lpf, False, args.steps, args.warmup)
    print(f"[bench] low-pass filter fwd {ms_lp_fwd:.3f} ms, fwd+bwd {ms_lp_step:.3f} ms, pairs {st_lp.pairs}",
          file=sys.stderr, flush=True)
    lowpass = {"fwd_ms": ms_lp_fwd, "fwd_fps": 1000.0 / ms_lp_fwd, "fwd_bwd_ms": ms_lp_step,
               "fwd_bwd_its": 1000.0 / ms_lp_step, "pairs": int(st_lp.pairs),
               "note": "PSM_FLAG_LOWPASS: rho = min(u^2 + v^2, 2 |x - c|^2); footprint = union with the filter disk"}
    del lpf
    base = Form(psm, t, cam, K, "aabb", "full", gout, device, tune=launch is None)
    ms_base_step, stages_base, st_base = timed(base, True, max(3, args.steps // 2), 2)
    ms_base_fwd, _, _ = timed(base, False, max(3, args.steps // 2), 2)
    base_launch, base_tuned = base.launch(), base.tuned_ms
    print(f"[bench] full+aabb fwd+bwd {ms_base_step:.3f} ms, fwd {ms_base_fwd:.3f} ms, launch {base_launch}",
          file=sys.stderr, flush=True)
    del base

    ablation = {}
    if not args.no_ablation:
        rows = {"baseline (sphere, dense)": ("sphere", "full"), "w/ precise tile (ellipse, dense)": ("ellipse", "full"),
                "w/ top-k (sphere, top-k)": ("sphere", "topk"), "full method (ellipse, top-k)": ("ellipse", "topk")}
        for label, (tm, bl) in rows.items():
            f = Form(psm, t, cam, K, tm, bl, gout, device)
            ms, _, s2 = timed(f, False, max(3, args.steps // 2), 2)
            ablation[label] = {"fwd_ms": ms, "fps": 1000.0 / ms, "pairs": int(s2.pairs),
                               "pairs_per_tile": s2.pairs / s2.tiles}
            del f
            print(f"[bench] ablation {label}: {ms:.3f} ms", file=sys.stderr, flush=True)

    torch.cuda.empty_cache()
    line = {
        "metric": METRIC,
        "value": 1000.0 / ms_step,
        "unit": "it/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if dtype == "f32" else dtype,
        "data": "synthetic",
        "config": {"workload": f"{args.workload}: planes7 scene, {sc.n} surfels, {cam.width}x{cam.height}, "
                               f"{sc.c}-d {dtype} features, K={K}, exact-ellipse tiles, Top-K blend",
                   "surfels": sc.n, "width": cam.width, "height": cam.height, "feat_dim": sc.c, "k": K,
                   "tile_mode": "ellipse", "blend": "topk", "parallelism": "single-gpu"},
        "fwd_fps": 1000.0 / ms_fwd,
        "fwd_ms": ms_fwd,
        "dense_aabb_form": {"fwd_fps": 1000.0 / ms_base_fwd, "fwd_bwd_its": 1000.0 / ms_base_step,
                            "fwd_ms": ms_base_fwd, "fwd_bwd_ms": ms_base_step, "pairs": int(st_base.pairs),
                            "stages_ms": stages_base, "launch": base_launch, "tuned_ms": base_tuned},
        "speedup_vs_dense_aabb": {"fwd": ms_base_fwd / ms_fwd, "fwd_bwd": ms_base_step / ms_step},
        "opacity_footprint": opacity_footprint,
        "feature_only": feature_only,
        "topk_renorm": topk_renorm,
        "lowpass": lowpass,
        "pairs": int(st.pairs), "pairs_walked": int(st.pairs_walked), "contributors": int(st.contributors),
        "visible": int(st.visible),
        "stages_ms": stages,
        "launch": {"schedule": ["grid", "persistent"][head_launch[0]],
                   "bwd_schedule": ["grid", "persistent"][head_launch[1]], "blend_pass": head_launch[2],
                   "bwd_pass": head_launch[3], "tile": f"{head_launch[4]}x{256 // head_launch[4]}",
                   "source": "autotuner" if launch is None else "--launch",
                   "tuned_ms": head_tuned_ms},
        "selected_unique": int(st.selected_unique), "selections": int(st.selections),
        "selected_pairs": int(st.selected_pairs), "bwd_entries": int(st.bwd_entries),
        "roofline": roofline(stages, st, K, sc.c, S, fbytes, args.workload, head_launch),
        "stage_roofline": stage_table(stages, st, K, sc.c, fbytes, S),
        "step_hbm": {"algorithmic_bytes": step_bytes(st, K, sc.c, fbytes, S),
                     "gbs": step_bytes(st, K, sc.c, fbytes, S) / (ms_step * 1e-3) / 1e9,
                     "frac": step_bytes(st, K, sc.c, fbytes, S) / (ms_step * 1e-3) / 1e9 / HBM_PEAK_GBS},
        "ablation_fwd": ablation,
    }
    if not args.no_cpu_baseline:
        feat64 = t["feat"].float().cpu().numpy().astype(np.float64)
        line["cpu_baseline"] = cpu_baseline(sc, cam, K, feat64, args.cpu_tiles)
        print(f"[bench] cpu baseline {line['cpu_baseline']['value']:.4f} it/s", file=sys.stderr, flush=True)
    line["instance_labels"] = labels_workload(psm, t["means"], max(3, args.steps // 2), 2)
    line["geometry_loss"] = geometry_workload(psm, t["means"], t["scales"], t["quats"], sc, max(3, args.steps // 2), 2)
    print(f"[bench] geometry loss {line['geometry_loss']['ms']:.3f} ms "
          f"({line['geometry_loss']['alu_tflops']:.1f} TFLOP/s)", file=sys.stderr, flush=True)
    line["frustum_attention"] = attention_workload(psm, max(3, args.steps // 2), 2)
    fa = line["frustum_attention"]
    print(f"[bench] frustum attention {fa['ms']:.3f} ms, {fa['active']} active of {fa['surfels']}, "
          f"{fa['mfma_tflops']:.1f} TFLOP/s", file=sys.stderr, flush=True)
    print(f"[bench] labels fwd {line['instance_labels']['fwd_ms']:.3f} ms, bwd {line['instance_labels']['bwd_ms']:.3f} ms",
          file=sys.stderr, flush=True)
    if not args.no_batch:
        del t, gout
        torch.cuda.empty_cache()
        line["batch_8cam"] = batch_workload(psm, scenes, max(3, args.steps // 2), 2)
        print(f"[bench] batch 8 cameras fwd+bwd {line['batch_8cam']['fwd_bwd_ms']:.3f} ms, graph "
              f"{line['batch_8cam']['graph_replay_ms']:.3f} ms", file=sys.stderr, flush=True)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
