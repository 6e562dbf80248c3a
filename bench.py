"""Throughput benchmark of the gfx950 tetrahedron rasterizer.

One step = forward + backward of the whole rendering path (pre-filter,
projection, depth sort, tile binning and sort, compositing, reverse-order
backward, vertex chain) through the autograd Function, on the training-shaped
workload: a 64^3-cube Kuhn grid (1,572,864 tets, 274,625 vertices) with a
sphere/torus smooth-union SDF plus noise, per-vertex RGB, 4 orbit views at
512x512, s = 320.  Inputs are resident on the device before timing starts.

Prints one JSON line (rank 0, one GPU).  Besides the headline it reports the
plain path (one launch sequence per view), step latency percentiles, per-stage
times from HIP events on the rendering stream, the roofline of the dominant
compositing kernel and the CPU oracle timed on a bounded pixel sample.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "fwd+bwd Mpixels/s (64³ grid, 512², 4 views) + p99 latency vs plain path"
HBM_PEAK_GBS = 8000.0
CU_NUM, CLOCK_GHZ = 256, 2.4
LDS_PEAK_GBS = 128 * CU_NUM * CLOCK_GHZ   # 128 B per clock per CU
# Algorithmic bytes of the compositing kernels in the per-unit terms of the
# hot-path measurement plan: a record of R_B bytes plus its 4-byte list
# index per entry walked, 40 B per pixel (8 output channels + 8 B of state),
# and for the backward 2 x 92 B per (view, kept tet) for the per-tet gradient
# written and read back.
R_B = 96
ENTRY_INDEX_B = 4
PIXEL_B = 40
TET_GRAD_RW_B = 2 * 92
# HBM bytes per launch of the compositing kernels at the default workload and
# launch shape (8x8 tiles, 4 waves, chunks 64/32), from the rocprofv3
# FETCH_SIZE / WRITE_SIZE passes summarised under profiles/ (FETCH_SIZE scaled
# by 2.0, WRITE_SIZE by 1.0 against a 256 MiB copy); the backward is its two
# kernels (the walk with its recurrence, then the per-pair gradients), summed,
# and its shares below are weighted by their durations.  VALU issue share:
# wave instructions SQ_INSTS_VALU x 4 cycles over 1024 SIMDs x 2.4 GHz x the
# mean duration; LDS busy share (LdsUtil: SQ_LDS_IDX_ACTIVE over CU cycles),
# the LDS bytes that busy time carries at 128 B per clock with the
# bank-conflict cycles taken out, the conflict cycles' share of the LDS busy
# cycles, and the mean occupancy (OccupancyPercent: SQ_WAVE_CYCLES over 32
# waves per CU).  Valid only for the kernel sources with these digests;
# reported as null once they change.
MEASURED = {"sha256": {"paper_2406_01579_amd/csrc/raster_mw.hip":
                       "57f32e73266485e7c7d770940c8e4dab026883d8c463d4cbe158caf61350e308",
                       "paper_2406_01579_amd/csrc/ts_device.h":
                       "3efa48fcd06f1d44b1e5829b6a4cd555b858726d468a599dab0209f998398312",
                       "paper_2406_01579_amd/csrc/tile8.h":
                       "80399ecd7337f4b753b94c7beb97c827d2359253f7b90f247744d996997845fe",
                       "paper_2406_01579_amd/csrc/ts_internal.h":
                       "1e2cc2feb686279adb054a0a7bc7445ca8931d479ec02b1e34e50765eee98310"},
            "composite_bwd": {"traffic": 234.9e6, "valu_issue_frac": 0.539, "lds_util": 0.181,
                              "lds_active_bytes": 1.0923e9, "lds_bank_conflict_frac": 0.152, "occupancy_pct": 43.4},
            "composite": {"traffic": 110.6e6, "valu_issue_frac": 0.489, "lds_util": 0.155,
                          "lds_active_bytes": 0.6513e9, "lds_bank_conflict_frac": 0.191, "occupancy_pct": 42.5}}


def measured_counters(kernel, args):
    import hashlib
    if (args.tile, args.waves, args.s, args.chunk_fwd in (0, 64), args.chunk_bwd in (0, 32)) != \
            ("8x8", 4, 320.0, True, True):
        return None
    for path, digest in MEASURED["sha256"].items():
        with open(os.path.join(ROOT, path), "rb") as f:
            if hashlib.sha256(f.read()).hexdigest() != digest:
                return None
    return MEASURED.get(kernel)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--s", type=float, default=320.0)
    ap.add_argument("--tile", default="8x8")
    ap.add_argument("--waves", type=int, default=4, help="waves sharing one 8x8 tile")
    ap.add_argument("--chunk-fwd", type=int, default=0, help="forward LDS chunk length (32, 64; 0: 64)")
    ap.add_argument("--chunk-bwd", type=int, default=0, help="backward LDS chunk length (16, 32; 0: 32)")
    ap.add_argument("--check", default="lazy", choices=["sync", "lazy"])
    ap.add_argument("--record-grads", action="store_true",
                    help="backward with one gradient accumulator per record (RENDER_RECORD_GRADS)")
    ap.add_argument("--recompute-state", action="store_true",
                    help="no per-pixel state in the workspace; the backward recomputes it (RENDER_RECOMPUTE_STATE)")
    ap.add_argument("--deterministic", action="store_true", help="fixed-order sums (RENDER_DETERMINISTIC)")
    ap.add_argument("--mode", default="graph", choices=["graph", "eager"],
                    help="headline path: the whole fwd+bwd step captured once in a HIP graph and replayed, or "
                         "eager launches through the autograd Function")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-plain", action="store_true", help="skip the one-launch-per-view path")
    ap.add_argument("--window-bench", type=int, default=5,
                    help="also time the step with the per-pixel resort window of this size (0: skip)")
    ap.add_argument("--cpu-pixels", type=int, default=400000)
    ap.add_argument("--cpu-pixels-1core", type=int, default=25000,
                    help="pixels of the oracle timed on one host thread (a sample of the same workload)")
    ap.add_argument("--no-serve", action="store_true", help="skip the short serving trace of the default run")
    ap.add_argument("--serve-trace-rate", type=float, default=1000.0,
                    help="arrival rate of the default run's short serving trace (req/s)")
    ap.add_argument("--serve-trace-seconds", type=float, default=1.5)
    ap.add_argument("--workload", default="training", choices=["training", "batched", "multiscene"],
                    help="batched: 128^3 band grid, 8 views at 1024^2; multiscene: 32 scenes, 124 mixed views "
                         "(fwd+bwd of every view in one graph-captured launch sequence vs one per view)")
    ap.add_argument("--serve", action="store_true",
                    help="serving benchmark instead: 16 resident scenes, open-loop Poisson arrivals, "
                         "continuous batching vs the plain one-launch-per-view path")
    ap.add_argument("--serve-rates", default="50,200,500,1000,2000")
    ap.add_argument("--serve-seconds", type=float, default=8.0, help="trace length per rate")
    ap.add_argument("--serve-max-requests", type=int, default=4000)
    ap.add_argument("--serve-streams", type=int, default=2)
    ap.add_argument("--calib-copy-mib", type=int, default=0,
                    help="after the run, copy a device buffer of this many MiB three times (a plain copy "
                         "kernel of known size, to scale hardware byte counters)")
    return ap.parse_args()


def pct(a, q):
    return float(np.percentile(np.asarray(a), q))


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}); the renderer shards by view and scene "
              "with no exchange in the forward, and a multi-GPU run is not implemented", file=sys.stderr)
        sys.exit(2)

    if args.serve:
        return serve_bench(args)
    if args.workload != "training":
        return workload_bench(args)

    import torch

    import synth
    from paper_2406_01579_amd import Params, Renderer, SceneT, TetSplatFunction
    from paper_2406_01579_amd import _lib

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    tw, th = (int(x) for x in args.tile.split("x"))
    wl = synth.training(s=args.s)
    sc = wl.scenes[0]
    cams = wl.cams
    nv = cams.shape[0]
    W, H = int(cams[0, 0]), int(cams[0, 1])
    pixels = nv * W * H
    st = SceneT.from_numpy(sc, dev)
    verts = st.verts.clone().requires_grad_(True)
    sdf = st.sdf.clone().requires_grad_(True)
    colors = st.colors.clone().requires_grad_(True)
    gen = torch.Generator(device=dev)
    gen.manual_seed(0)
    dout = torch.randn((nv, 8, H, W), device=dev, generator=gen)
    params = Params(tile_w=tw, tile_h=th, waves=args.waves, record_grads=args.record_grads,
                    recompute_state=args.recompute_state, deterministic=args.deterministic,
                    chunk_fwd=args.chunk_fwd, chunk_bwd=args.chunk_bwd)
    renderer = Renderer(params, device=dev, check=args.check)

    def step(cam_subset=None):
        cs = cams if cam_subset is None else cams[cam_subset]
        out = TetSplatFunction.apply(verts, sdf, colors, st.tets, cs, args.s, renderer)
        g = dout if cam_subset is None else dout[cam_subset]
        torch.autograd.backward(out, g)
        verts.grad = None
        sdf.grad = None
        colors.grad = None

    # warm-up (also sizes the workspaces)
    for _ in range(max(1, args.warmup)):
        step()
    torch.cuda.synchronize()

    # timed region: K steps, HIP events per step and per pipeline stage
    _lib.profile(True)
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        evs[k][0].record()
        step()
        evs[k][1].record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    stages = _lib.profile_read()
    _lib.profile(False)
    step_ms = [a.elapsed_time(b) for a, b in evs]
    eager_ms = 1000.0 * wall / args.steps
    eager = {"ms_per_step": round(eager_ms, 4), "mpx_s": round(pixels / (eager_ms * 1e-3) / 1e6, 2),
             "p50_ms": round(pct(step_ms, 50), 4), "p99_ms": round(pct(step_ms, 99), 4)}
    ms_per_step, lat = eager_ms, step_ms

    graph = None
    if args.mode == "graph":
        from paper_2406_01579_amd import CapturedStep
        cstep = CapturedStep(verts.detach(), sdf.detach(), colors.detach(), st.tets, cams, args.s, params, dout)
        for _ in range(max(1, args.warmup)):
            cstep.replay()
        cstep.check()
        # throughput: the K replays back to back, nothing recorded between
        # them (a pair of timing events per step adds about 9 us of queue
        # work per step); per-step latency from a second, instrumented pass
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for k in range(args.steps):
            cstep.replay()
        torch.cuda.synchronize()
        gwall = time.perf_counter() - t0
        cstep.check()
        gev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
        for k in range(args.steps):
            gev[k][0].record()
            cstep.replay()
            gev[k][1].record()
        torch.cuda.synchronize()
        cstep.check()
        g_ms = [a.elapsed_time(b) for a, b in gev]
        ms_per_step, lat = 1000.0 * gwall / args.steps, g_ms
        graph = {"ms_per_step": round(ms_per_step, 4), "capacities": [cstep.kept_cap, cstep.entry_cap]}
        del cstep
    value = pixels / (ms_per_step * 1e-3) / 1e6

    # the same step with the per-pixel resort window (Sec. 3.3), graph-captured
    window = None
    if args.window_bench > 0 and args.mode == "graph" and (tw, th) == (8, 8):
        from paper_2406_01579_amd import CapturedStep
        wparams = Params(tile_w=8, tile_h=8, waves=args.waves, window=args.window_bench)
        wstep = CapturedStep(verts.detach(), sdf.detach(), colors.detach(), st.tets, cams, args.s, wparams, dout)
        for _ in range(max(1, args.warmup)):
            wstep.replay()
        wstep.check()
        n_w = max(5, args.steps // 2)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(n_w):
            wstep.replay()
        torch.cuda.synchronize()
        wms = 1000.0 * (time.perf_counter() - t0) / n_w
        wstep.check()
        window = {"window": args.window_bench, "ms_per_step": round(wms, 4),
                  "mpx_s": round(pixels / (wms * 1e-3) / 1e6, 2)}
        del wstep

    # workload facts of the last forward (for the roofline)
    # (the per-pixel state comes from a forward that keeps it)
    import dataclasses
    stats_r = renderer if not args.recompute_state else Renderer(
        dataclasses.replace(params, recompute_state=False), device=dev, check="sync")
    plan = stats_r.forward([SceneT(verts.detach(), st.tets, sdf.detach(), colors.detach(), args.s)], cams)
    stt = stats_r.read_status(plan)
    dbg = stats_r.debug(plan)
    E = int(stt.entries)
    tiles = dbg["ranges"].shape[0]
    last = dbg["last"]
    # entries each tile had to walk: up to its last blended entry (what the
    # backward reads); the forward walks the same prefix plus its final chunk
    rng_ = dbg["ranges"].astype(np.int64)
    # per-tile max last-blended position from the per-pixel state
    tile_of_pix = []
    tx_n, ty_n = (W + tw - 1) // tw, (H + th - 1) // th
    jj, ii = np.meshgrid(np.arange(H), np.arange(W), indexing="ij")
    tloc = (jj // th) * tx_n + (ii // tw)
    e_proc = 0
    for v in range(nv):
        lv = last[v * W * H:(v + 1) * W * H].reshape(H, W)
        mx = np.full(tx_n * ty_n, -1, np.int64)
        np.maximum.at(mx, tloc.ravel(), lv.ravel())
        base = v * tx_n * ty_n
        st_ = rng_[base:base + tx_n * ty_n, 0]
        e_proc += int(np.maximum(mx + 1 - st_, 0)[mx >= 0].sum())
    del plan

    comp_ms, comp_n = stages["composite"]
    bwd_ms, bwd_n = stages["composite_bwd"]
    pg_ms, pg_n = stages["pair_grads"]
    fwd_avg = comp_ms / max(comp_n, 1)
    # the backward compositing step runs as two kernels on the 8x8 multi-wave
    # path (the walk with its recurrence, then the per-pair gradients): its
    # duration is their sum per step
    bwd_avg = bwd_ms / max(bwd_n, 1) + (pg_ms / pg_n if pg_n else 0.0)
    # algorithmic HBM bytes per launch (one launch covers all 4 views): the
    # per-unit terms of the measurement plan times the entries (walked, for
    # the backward), pixels and (view, kept tet) records of this launch
    K_rec = int(stt.records)
    fwd_bytes = (R_B + ENTRY_INDEX_B) * E + PIXEL_B * pixels
    bwd_bytes = (R_B + ENTRY_INDEX_B) * e_proc + PIXEL_B * pixels + TET_GRAD_RW_B * K_rec
    kern = {
        "composite": dict(ms=fwd_avg, bytes=fwd_bytes),
        "composite_bwd": dict(ms=bwd_avg, bytes=bwd_bytes),
    }
    dom = max(kern, key=lambda k: kern[k]["ms"])
    ach = kern[dom]["bytes"] / (kern[dom]["ms"] * 1e-3) / 1e9
    meas = measured_counters(dom, args)

    def mget(key):
        return None if meas is None or key not in meas else meas[key]
    lds = None
    if mget("lds_util") is not None:
        lds_gbs = mget("lds_active_bytes") / (kern[dom]["ms"] * 1e-3) / 1e9
        lds = {"achieved": round(lds_gbs, 1), "peak": round(LDS_PEAK_GBS, 1), "unit": "GB/s",
               "frac": round(lds_gbs / LDS_PEAK_GBS, 4), "busy_frac": mget("lds_util"),
               "bank_conflict_frac": mget("lds_bank_conflict_frac")}
    roofline = {"bound": "hbm", "achieved": round(ach, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(ach / HBM_PEAK_GBS, 4), "traffic": None if meas is None else int(meas["traffic"]),
                "kernel": dom, "kernel_ms": round(kern[dom]["ms"], 4), "algorithmic_bytes": int(kern[dom]["bytes"]),
                "kernels": ({"k_composite_bwd_mw": round(bwd_ms / max(bwd_n, 1), 4),
                             "k_pair_grads": round(pg_ms / max(pg_n, 1), 4)}
                            if dom == "composite_bwd" and pg_n else None),
                "bytes_per_unit": {"entry_walked": R_B + ENTRY_INDEX_B, "pixel": PIXEL_B,
                                   "view_kept_tet": TET_GRAD_RW_B if dom == "composite_bwd" else 0},
                "valu_issue_frac": mget("valu_issue_frac"),
                "lds": lds,
                "occupancy_pct": mget("occupancy_pct"),
                "note": "the compositing kernels are bound by the per-tile sequential walk (dependent chunk phases) "
                        "and VALU issue, not HBM; traffic is the HBM bytes the counters saw per launch"}

    # plain path: one launch sequence per view
    plain = None
    if not args.no_plain:
        for _ in range(3):
            for v in range(nv):
                step([v])
        torch.cuda.synchronize()
        n_plain = max(5, args.steps // 2)
        t0 = time.perf_counter()
        pev = []
        for _ in range(n_plain):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for v in range(nv):
                step([v])
            b.record()
            pev.append((a, b))
        torch.cuda.synchronize()
        pw = (time.perf_counter() - t0) / n_plain
        pms = [a.elapsed_time(b) for a, b in pev]
        plain = {"ms_per_step": round(1000 * pw, 4), "mpx_s": round(pixels / pw / 1e6, 2),
                 "p50_ms": round(pct(pms, 50), 4), "p99_ms": round(pct(pms, 99), 4)}

    if args.calib_copy_mib > 0:
        n = args.calib_copy_mib * (1 << 20) // 4
        src = torch.ones(n, device=dev)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    serving = None
    if not args.no_serve:
        serving = serve_trace(args)

    cpu = None
    if not args.no_cpu:
        cpu = cpu_baseline(sc, cams, args.s, args.cpu_pixels, args.cpu_pixels_1core)

    line = {
        "metric": METRIC, "value": round(value, 2), "unit": "Mpixels/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 4), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "training-shaped: 64^3-cube Kuhn grid (1,572,864 tets), sphere+torus smooth-union "
                               "SDF + N(0,0.005), per-vertex RGB, 4 orbit views 512x512, s=320, fwd+bwd",
                   "views": nv, "width": W, "height": H, "tile": args.tile, "waves": args.waves,
                   "chunks": [args.chunk_fwd or 64, args.chunk_bwd or 32], "s": args.s,
                   "path": ("whole fwd+bwd step through the autograd Function captured in one HIP graph"
                            if args.mode == "graph" else "eager launches through the autograd Function"),
                   "status_check": args.check,
                   "flags": [k for k in ("record_grads", "recompute_state", "deterministic") if getattr(args, k)]},
        "p50_ms": round(pct(lat, 50), 4), "p99_ms": round(pct(lat, 99), 4),
        "eager_path": eager,
        "graph": graph,
        "plain_path": plain,
        "window_path": window,
        "roofline": roofline,
        "serving": serving,
        "cpu_baseline": cpu,
        "stages_ms_per_step": {k: round(v[0] / max(args.steps, 1), 4) for k, v in stages.items() if v[1]},
        "workload_stats": {"entries": E, "entries_walked_bwd": e_proc, "kept_tets": int(stt.kept),
                           "records": int(stt.records), "tiles": tiles},
    }
    print(json.dumps(line), flush=True)


def workload_bench(args):
    """fwd+bwd of every view of every scene in one launch sequence, captured
    once in a HIP graph and replayed, with the launch shape picked by the
    autotuner on this workload; against the plain path, one eager launch
    sequence (forward + backward) per view."""
    import torch

    import synth
    from paper_2406_01579_amd import Params, Renderer, SceneT
    from paper_2406_01579_amd.tune import Autotuner

    torch.cuda.set_device(0)
    dev = torch.device("cuda:0")
    t0 = time.perf_counter()
    wl = synth.batched(s=args.s) if args.workload == "batched" else synth.multiscene(s=args.s)
    scenes = [SceneT.from_numpy(sc, dev) for sc in wl.scenes]
    cams, vs = wl.cams, wl.view_scene
    nv = cams.shape[0]
    pixels = int(sum(int(c[0]) * int(c[1]) for c in cams))
    print(f"[{args.workload}] {len(scenes)} scenes, {nv} views, {pixels / 1e6:.2f} Mpx, "
          f"{sum(int(s.tets.shape[0]) for s in scenes)} tets, built in {time.perf_counter() - t0:.1f} s",
          file=sys.stderr, flush=True)
    gen = torch.Generator(device=dev)
    gen.manual_seed(0)
    douts = [torch.randn((8, int(c[1]), int(c[0])), device=dev, generator=gen) for c in cams]
    tuner = Autotuner(reps=2, base=Params())
    params = tuner.best(scenes, cams, vs, dout=douts)
    tuned = next(iter(tuner.cache.values()))
    print(f"[{args.workload}] autotuned {params.tile_w}x{params.tile_h} waves {params.waves} chunks "
          f"{params.chunk_fwd}/{params.chunk_bwd}: {tuned['ms']}",
          file=sys.stderr, flush=True)

    # exact sizes from one synchronous forward, then capture with headroom
    probe = Renderer(params, device=dev, check="sync")
    st = probe.forward(scenes, cams, vs).status
    kept, ent = int(int(st.kept) * 1.25) + 1024, int(int(st.entries_needed) * 1.3) + 4096
    r = Renderer(params, device=dev, check="none")
    r.set_capacity(scenes, cams, vs, kept, ent)
    side = torch.cuda.Stream(device=dev)
    side.wait_stream(torch.cuda.current_stream(dev))
    with torch.cuda.stream(side):
        for _ in range(2):
            r.backward(r.forward(scenes, cams, vs), douts)
    torch.cuda.current_stream(dev).wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan = r.forward(scenes, cams, vs)
        grads = r.backward(plan, douts)
    torch.cuda.synchronize()
    for _ in range(args.warmup):
        graph.replay()
    torch.cuda.synchronize()
    stt = r.read_status(plan)
    assert stt.overflow == 0, "capacities exceeded"
    # throughput from back-to-back replays; per-step latency from a second,
    # instrumented pass
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(args.steps):
        graph.replay()
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t1) / args.steps
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    for a, b in evs:
        a.record()
        graph.replay()
        b.record()
    torch.cuda.synchronize()
    lat = [a.elapsed_time(b) for a, b in evs]
    value = pixels / wall / 1e6

    plain = None
    if not args.no_plain:
        pr = Renderer(params, device=dev, check="sync")
        single = [(int(vs[v]), cams[v:v + 1], douts[v:v + 1]) for v in range(nv)]
        for sid, c, d in single:                       # sizes and warm-up
            pr.backward(pr.forward([scenes[sid]], c), d)
        pr.check = "lazy"
        torch.cuda.synchronize()
        pms = []
        t2 = time.perf_counter()
        for _ in range(max(1, args.steps // 5)):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for sid, c, d in single:
                pr.backward(pr.forward([scenes[sid]], c), d)
            b.record()
            torch.cuda.synchronize()
            pms.append(a.elapsed_time(b))
        pwall = (time.perf_counter() - t2) / max(1, args.steps // 5)
        plain = {"ms_per_step": round(pwall * 1e3, 4), "mpx_s": round(pixels / pwall / 1e6, 2),
                 "p50_ms": round(pct(pms, 50), 4), "p99_ms": round(pct(pms, 99), 4)}
    desc = ("128^3-cube blob grid pruned to the |f|<0.05 band (662,683 tets), 8 orbit views at 1024x1024, s=320, "
            "fwd+bwd" if args.workload == "batched" else
            "32 blob scenes (32^3..128^3 cube grids, |f|<0.05 band, 5.55 M tets), 124 views at 256..1024 square "
            "(1-8 per scene), s=320, fwd+bwd")
    line = {
        "metric": f"fwd+bwd Mpixels/s ({args.workload}) vs plain path", "value": round(value, 2),
        "unit": "Mpixels/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(wall * 1e3, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": desc, "views": nv, "scenes": len(scenes), "pixels": pixels,
                   "tile": f"{params.tile_w}x{params.tile_h}", "waves": params.waves,
                   "chunks": [params.chunk_fwd, params.chunk_bwd],
                   "path": "fwd+bwd of all views and scenes in one launch sequence, captured in one HIP graph"},
        "p50_ms": round(pct(lat, 50), 4), "p99_ms": round(pct(lat, 99), 4),
        "autotune_ms": tuned["ms"],
        "plain_path": plain,
        "workload_stats": {"entries": int(stt.entries), "kept_tets": int(stt.kept), "records": int(stt.records)},
    }
    del grads
    print(json.dumps(line), flush=True)


def serve_bench(args):
    """Forward-only serving: 16 resident blob scenes (32^3..128^3 cube grids,
    band-pruned), requests of 1-4 views at 256/512/1024 square, open-loop
    Poisson arrivals; continuous batching over several streams vs the plain
    path (FIFO, one launch sequence per view) on the same trace."""
    import torch

    import synth
    from paper_2406_01579_amd import Params
    from paper_2406_01579_amd.serve import SceneRegistry, Server

    torch.cuda.set_device(0)
    t0 = time.perf_counter()
    scenes = synth.serving_scenes(s=args.s)
    reg = SceneRegistry(Params(waves=args.waves))
    rng = np.random.default_rng(9)
    for sc in scenes:
        reg.add(sc, np.concatenate([synth.random_orbit_cameras(rng, 2, z) for z in (256, 512, 1024)], 0))
    print(f"[serve] {len(scenes)} scenes resident ({reg.bytes / 2**20:.0f} MiB) in {time.perf_counter() - t0:.1f} s",
          file=sys.stderr, flush=True)
    # warm-up trace (allocator pools, first launches of each shape)
    for batching in (True, False):
        Server(reg, streams=args.serve_streams if batching else 1, batching=batching, keep_outputs=False).run(
            synth.serving_requests(200, 1000.0, len(scenes), seed=99))
    rows = []
    for rate in (float(x) for x in args.serve_rates.split(",")):
        n = int(min(args.serve_max_requests, max(50, rate * args.serve_seconds)))
        trace = synth.serving_requests(n, rate, len(scenes))
        row = {"rate_per_s": rate, "requests": n}
        for name, batching in (("batched", True), ("plain", False)):
            srv = Server(reg, streams=args.serve_streams if batching else 1, batching=batching, keep_outputs=False)
            st = srv.run(trace)
            row[name] = {k: (round(v, 4) if isinstance(v, float) else v) for k, v in st.items()
                         if k in ("p50_ms", "p99_ms", "mean_ms", "mpix_per_s", "launches", "reruns", "batches",
                                  "mean_views_per_batch", "max_queue", "served", "rejected")}
            print(f"[serve] rate {rate:g}/s {name}: p50 {st['p50_ms']:.3f} ms p99 {st['p99_ms']:.3f} ms "
                  f"{st['mpix_per_s']:.0f} Mpx/s", file=sys.stderr, flush=True)
        rows.append(row)
    top = rows[-1]
    line = {
        "metric": "serving forward Mpixels/s + p50/p99 latency vs plain path (16 resident scenes, Poisson arrivals)",
        "value": top["batched"]["mpix_per_s"], "unit": "Mpixels/s", "n_gpus": 1, "steps": None, "warmup": None,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "16 blob scenes (32^3..128^3 cube grids, |f|<0.05 band), requests of 1-4 views at "
                               "256/512/1024 square, open-loop Poisson arrivals, forward only, s=320",
                   "streams": args.serve_streams, "rates": args.serve_rates, "tile": "8x8", "waves": args.waves},
        "rates": rows,
    }
    print(json.dumps(line), flush=True)


def serve_trace(args):
    """A short serving trace of the serving workload (16 resident blob scenes,
    32^3..128^3 cube grids; requests of 1-4 views at 256/512/1024 square;
    open-loop Poisson arrivals; forward only): continuous batching over two
    streams against the plain path (FIFO, one launch sequence per view) on
    the same trace."""
    import torch

    import synth
    from paper_2406_01579_amd import Params
    from paper_2406_01579_amd.serve import SceneRegistry, Server
    t0 = time.perf_counter()
    scenes = synth.serving_scenes(s=args.s)
    reg = SceneRegistry(Params(waves=args.waves))
    rng = np.random.default_rng(9)
    for sc in scenes:
        reg.add(sc, np.concatenate([synth.random_orbit_cameras(rng, 2, z) for z in (256, 512, 1024)], 0))
    for batching in (True, False):
        Server(reg, streams=args.serve_streams if batching else 1, batching=batching, keep_outputs=False).run(
            synth.serving_requests(200, 1000.0, len(scenes), seed=99))
    rate = args.serve_trace_rate
    n = int(max(50, rate * args.serve_trace_seconds))
    trace = synth.serving_requests(n, rate, len(scenes))
    out = {"rate_per_s": rate, "requests": n, "streams": args.serve_streams,
           "workload": "16 resident blob scenes (32^3..128^3), 1-4 views at 256/512/1024 square, Poisson "
                       "arrivals, forward only"}
    for name, batching in (("batched", True), ("plain", False)):
        srv = Server(reg, streams=args.serve_streams if batching else 1, batching=batching, keep_outputs=False)
        st = srv.run(trace)
        out[name] = {k: round(st[k], 4) for k in ("p50_ms", "p99_ms", "mpix_per_s")}
    out["setup_s"] = round(time.perf_counter() - t0, 1)
    del reg
    torch.cuda.empty_cache()
    return out


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(sc, cams, s, npix, npix1):
    """The oracle as it stands, float32, forward + backward on a bounded
    sample of pixels of the same workload (every k-th pixel of every view),
    on all host threads and on one."""
    import oracle
    g = oracle.Geometry.of(sc)
    P = oracle.params_array(s)
    pix = oracle.all_pixels(cams)

    def run(n):
        step = max(1, pix.shape[0] // n)
        sample = np.ascontiguousarray(pix[::step][:n])
        dout = np.random.default_rng(0).normal(size=(sample.shape[0], 8))
        t0 = time.perf_counter()
        oracle.render(g, cams, P, sample, prec=32)
        t1 = time.perf_counter()
        oracle.backward(g, cams, P, sample, dout, prec=32)
        t2 = time.perf_counter()
        return sample.shape[0], step, t1 - t0, t2 - t1

    threads = oracle.num_threads()
    n, step, tf, tb = run(npix)
    oracle.set_threads(1)
    n1, step1, tf1, tb1 = run(npix1)
    oracle.set_threads(threads)
    return {"value": round(n / (tf + tb) / 1e6, 6), "unit": "Mpixels/s", "cores": threads,
            "kind": "oracle",
            "sample": f"{n} pixels (every {step}th of the 4x512x512 views), float32 forward ({tf:.2f} s) + "
                      f"backward ({tb:.2f} s), per-pixel loop over every kept tet",
            "single_core": {"value": round(n1 / (tf1 + tb1) / 1e6, 6), "unit": "Mpixels/s", "cores": 1,
                            "sample": f"{n1} pixels (every {step1}th), forward {tf1:.2f} s + backward {tb1:.2f} s"},
            "cpu_model": cpu_model(), "nproc": os.cpu_count(),
            "omp_num_threads": os.environ.get("OMP_NUM_THREADS")}


if __name__ == "__main__":
    main()
