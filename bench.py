"""Benchmark of the StyleBlit hot path on one MI355X.

A step is one frame through the whole per-frame path (seed records, the
per-pixel level loop of Algorithm 2 and the voting blend), with the style
(padded exemplar, guide and lookup table) already resident, as it is across
frames in use.  The style's lookup-table build runs once before timing and is
reported separately.

Default workload: the 1920x1080 normal-guided frame (512x512 sphere
exemplar, 4 levels of spacing 64..8, threshold 32, radius 3).  Inputs and
outputs rotate over enough buffer sets (> 512 MB) that each step reads its
guide from HBM rather than from the 256 MB Infinity Cache.  The kernel
choice is the autotuner's pick for this frame shape (every choice computes
the same bits).

The roofline object is for the dominant kernel, the voting pass, timed per
launch with HIP events recorded between the passes on the launch stream.

Prints one JSON line.  ``--gpus`` above 1 is refused: this measures one GPU.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# VALU issue peak: 256 CUs x 4 SIMDs, each issuing one wave64 instruction
# every 4 cycles (16 lanes per cycle), at 2.4 GHz = 614.4 G wave instructions/s
VALU_PEAK_G_WAVE_INSTR = 256 * 2.4
# counter summaries per workload, valid for the kernel source they name: the
# voting kernel's FETCH_SIZE / WRITE_SIZE per dispatch with the copy-kernel
# calibration, and the per-frame kernels' instruction counts (SQ_INSTS_VALU
# etc. per dispatch)
PROFILES = os.path.join(ROOT, "profiles")


def traffic_file(workload_name):
    return os.path.join(PROFILES, f"k_blend_{workload_name}_traffic.json")


def instr_file(workload_name):
    return os.path.join(PROFILES, f"path_{workload_name}_instructions.json")


KERNEL_SRCS = [os.path.join(ROOT, "paper_1807_03249_amd", "csrc", f)
               for f in ("stylize.hip", "sb_device.h")]


def path_algorithmic_bytes(w, h, fmt, sw, sh, nseeds, nfallback):
    """Bytes the whole method must move per frame: target guide read, RGB and
    chunk map written, the exemplar (RGB + guide) read once, and one
    lookup-table entry per seed and per fallback pixel."""
    gb = 2 if fmt == 0 else 4
    return w * h * (gb + 3 + 4) + sw * sh * (3 + gb) + 4 * (nseeds + nfallback)


def vote_algorithmic_bytes(w, h, sw, sh):
    """Bytes the voting step must move per frame: the RGB output written and
    the exemplar RGB read once (its input offsets are an intermediate of the
    two-pass design, not of the method)."""
    return w * h * 3 + sw * sh * 3


def progress(msg):
    """A progress line on stderr (the JSON result alone goes to stdout)."""
    print(f"bench: {msg}", file=sys.stderr, flush=True)


def kernel_sha():
    """Hash of the frame kernels' sources (the kernels and the device helpers
    they include), which the counter summaries record."""
    h = hashlib.sha256()
    for path in KERNEL_SRCS:
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def traffic_per_launch(workload_name):
    """HBM bytes per voting launch from the committed counter summary, or
    None when it is missing, for another workload, or for older kernel
    source."""
    try:
        with open(traffic_file(workload_name)) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if t.get("kernel_source_sha256_16") != kernel_sha() or t.get("workload") != workload_name:
        return None
    fetch = t["fetch_kib_per_dispatch"] * 1024.0 / t["copy_fetch_factor"]
    write = t["write_kib_per_dispatch"] * 1024.0 / t["copy_write_factor"]
    return fetch + write


def cpu_model():
    """The host CPU's model name (from /proc/cpuinfo), or None."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def valu_issue(workload_name, kernel_prefix, kernel_ms):
    """Vector-ALU issue rate of one per-frame kernel: its wave instructions
    per launch from the committed counter summary over the live kernel time,
    against the issue peak; None when the summary is missing, for another
    workload, or for older kernel source."""
    try:
        with open(instr_file(workload_name)) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if t.get("kernel_source_sha256_16") != kernel_sha() or t.get("workload") != workload_name:
        return None
    for name, k in t["kernels"].items():
        if name.startswith(kernel_prefix):
            g = k["valu_wave_instructions"] / (kernel_ms * 1e-3) / 1e9
            return {"kernel": name, "valu_wave_instructions": k["valu_wave_instructions"],
                    "lane_ops_per_px": round(k["valu_wave_instructions"] * 64 / t["pixels"], 1),
                    "achieved": round(g, 1), "peak": VALU_PEAK_G_WAVE_INSTR,
                    "unit": "G wave instructions/s", "frac": round(g / VALU_PEAK_G_WAVE_INSTR, 4)}
    return None


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", type=int, default=2, choices=[1, 2, 3])
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--streams", type=int, default=2,
                    help="streams the timed frames are enqueued on, round robin")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--rotate-mb", type=float, default=600.0)
    ap.add_argument("--tune", action="store_true",
                    help="autotune the frame's kernel choice (default: the library default, "
                         "whose voting kernel the committed counter summary covers)")
    ap.add_argument("--no-tune", action="store_true", help="batch leg: library default choice")
    ap.add_argument("--no-batch", action="store_true", help="skip the 64-frame batch leg")
    ap.add_argument("--no-serve", action="store_true", help="skip the serving leg")
    ap.add_argument("--no-seg", action="store_true", help="skip the segmentation-guide leg")
    ap.add_argument("--no-anim", action="store_true", help="skip the animation leg")
    ap.add_argument("--no-channels", action="store_true",
                    help="skip the three-channel (appearance) guide leg")
    ap.add_argument("--no-search", action="store_true",
                    help="skip the many-channel (exact search) leg")
    ap.add_argument("--serve-requests", type=int, default=10000)
    ap.add_argument("--serve-qps", type=str, default="2000,12000,24000,36000,48000",
                    help="comma-separated request rates of the serving sweep")
    ap.add_argument("--calibrate-copy-mb", type=float, default=0.0,
                    help="after timing, run one plain device copy of this many MB "
                         "(the counter calibration kernel for rocprofv3 --pmc runs)")
    args = ap.parse_args()

    if args.gpus != 1:
        print(f"bench.py measures one GPU; --gpus {args.gpus} is not supported "
              "(frames are independent, so several GPUs would each run their own share of "
              "the frames with no exchange between them)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_1807_03249_amd as sb
    import paper_1807_03249_amd.autotune as at
    import workloads

    torch.cuda.set_device(0)
    styles, frames = workloads.config(args.workload)
    st_np, fr = styles[0], frames[0]
    p = fr.params
    prm = sb.params(p.levels, p.finest, p.threshold, p.radius, seed=fr.seed)
    w, h = fr.w, fr.h
    wname = workloads.CONFIG_NAMES[args.workload]

    # style registration (upload, padded exemplar, lookup table on the device),
    # timed on its second run (the first also loads the code objects)
    style = sb.Style(st_np.rgb, st_np.guide, st_np.lut_bits)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    style = sb.Style(st_np.rgb, st_np.guide, st_np.lut_bits)
    torch.cuda.synchronize()
    lut_ms = (time.perf_counter() - t0) * 1e3

    # rotating buffer sets
    g_np = fr.guide.view(np.int16) if fr.guide.dtype == np.uint16 else fr.guide
    guide0 = torch.from_numpy(g_np).cuda()
    jit = None  # the seeds come from the jitter hash of prm.seed
    wsb = sb.workspace_bytes(w, h, prm)
    per_set = guide0.numel() * guide0.element_size() + w * h * 3 + w * h * 4 + wsb
    nsets = max(2, int(args.rotate_mb * 1e6 // per_set) + 1)
    nsets += nsets % args.streams  # a buffer set is always reused on the same stream
    sets = []
    for _ in range(nsets):
        sets.append((guide0.clone(), torch.empty((h, w, 3), dtype=torch.uint8, device="cuda"),
                     torch.empty((h, w), dtype=torch.int32, device="cuda"),
                     torch.empty(wsb, dtype=torch.uint8, device="cuda")))
    torch.cuda.synchronize()

    tune = None
    if args.tune:
        tune = at.tune_frame(style, guide0, jit, prm)["tune"]

    # frames are enqueued round robin on `--streams` streams (each with its
    # own buffer sets), so one frame's level loop overlaps the previous
    # frame's vote: both kernels are latency-bound and leave issue slots idle
    streams = [torch.cuda.Stream() for _ in range(args.streams)]

    def step(k, events=None, stream=None):
        g, o_rgb, o_chunk, ws = sets[k % nsets]
        with torch.cuda.stream(stream if stream is not None else streams[k % args.streams]):
            sb.stylize(style, g, jit, prm, out_rgb=o_rgb, out_chunk=o_chunk, workspace=ws,
                       tune=tune, events=events)

    # the timed loop launches prepared calls (arguments marshalled once per
    # buffer set), so the host adds only the C call per frame
    plans = [sb.FramePlan(style, g, jit, prm, o_rgb, o_chunk, ws, tune=tune)
             for g, o_rgb, o_chunk, ws in sets]
    handles = [s.cuda_stream for s in streams]

    def timed(nsteps, nstreams):
        for k in range(args.warmup):
            plans[k % nsets].launch(handles[k % nstreams])
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for k in range(nsteps):
            plans[k % nsets].launch(handles[k % nstreams])
        torch.cuda.synchronize()
        return time.perf_counter() - t0

    # one stream alone first (context for the per-frame latency), then the
    # timed region: exactly K steps on all streams
    single_s = timed(args.steps, 1)
    elapsed = timed(args.steps, args.streams)
    ms_per_step = elapsed * 1e3 / args.steps
    mpx_s = w * h * args.steps / elapsed / 1e6

    # per-pass durations: fence-free HIP timing events recorded by the
    # library between the passes, on one stream (frames one after another)
    evs = [sb.TimingEvents() for _ in range(args.steps)]
    for k in range(args.steps):
        step(k, evs[k], stream=streams[0])
    torch.cuda.synchronize()
    passes = np.array([e.pass_ms() for e in evs])
    for e in evs:
        e.close()
    frame_ms = np.sort(passes.sum(axis=1))
    seeds_ms, assign_ms, vote_ms = passes.mean(axis=0)

    # outputs of the last step: fallback pixels for the byte count
    chunk = sets[(args.steps - 1) % nsets][2].cpu().numpy().view(np.uint32)
    nfallback = int(((chunk >> 26) == p.levels).sum())
    nseeds = sb.jitter_len(w, h, p.levels, p.finest)
    pbytes = path_algorithmic_bytes(w, h, st_np.fmt, st_np.sw, st_np.sh, nseeds, nfallback)
    vbytes = vote_algorithmic_bytes(w, h, st_np.sw, st_np.sh)
    vote_gbs = vbytes / (vote_ms * 1e-3) / 1e9
    traffic = traffic_per_launch(wname)

    # a streaming device copy of 1 GiB on this GPU: what HBM sustains for
    # plain reads and writes (reported beside the 8 TB/s peak)
    csrc = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    cdst = torch.empty_like(csrc)
    cdst.copy_(csrc)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(10):
        cdst.copy_(csrc)
    e1.record()
    e1.synchronize()
    copy_gbs = round(2 * 10 * csrc.numel() / (e0.elapsed_time(e1) * 1e-3) / 1e9, 1)
    del csrc, cdst

    cpu = None
    if not args.no_cpu:
        import oracle

        lut = oracle.lut_build(st_np.guide, st_np.lut_bits)
        nthreads = oracle.set_threads(0)
        n = 0
        c0 = time.perf_counter()
        while True:
            oracle.stylize(st_np.rgb, st_np.guide, lut, st_np.lut_bits, fr.guide, fr.jitter,
                           p.levels, p.finest, p.threshold, p.radius, seed=fr.seed)
            n += 1
            if time.perf_counter() - c0 >= args.cpu_seconds or n >= 200:
                break
        csec = time.perf_counter() - c0
        cpu = {"value": round(w * h * n / csec / 1e6, 3), "unit": "Mpixel/s", "cores": nthreads,
               "kind": "oracle",
               "sample": f"{n} full {w}x{h} frames of this workload (lookup table built once, "
                         f"not timed), OpenMP over rows"}
        # the same oracle on one thread (the paper-like single-core figure)
        oracle.set_threads(1)
        n1 = 0
        c0 = time.perf_counter()
        while True:
            oracle.stylize(st_np.rgb, st_np.guide, lut, st_np.lut_bits, fr.guide, fr.jitter,
                           p.levels, p.finest, p.threshold, p.radius, seed=fr.seed)
            n1 += 1
            if time.perf_counter() - c0 >= args.cpu_seconds / 4 or n1 >= 20:
                break
        c1 = time.perf_counter() - c0
        oracle.set_threads(nthreads)
        cpu["single_thread"] = {"value": round(w * h * n1 / c1 / 1e6, 3),
                                "sample": f"{n1} full {w}x{h} frames on one thread"}
        cpu["cpu_model"] = cpu_model()
        cpu["host_cpus"] = os.cpu_count()

    progress("main leg and CPU baseline done")
    seg = None if args.no_seg else seg_leg(sb, torch, np, workloads, st_np, fr, prm, ms_per_step)
    progress("segmentation leg done")
    anim = None if args.no_anim else anim_leg(sb, torch, np, workloads, style, w, h, p)
    progress("animation leg done")
    chan = None if args.no_channels else channels_leg(sb, torch, np, workloads, ms_per_step)
    progress("three-channel leg done")
    search = None if args.no_search else search_leg(sb, torch, np, workloads, ms_per_step,
                                                    cpu_frame=not args.no_cpu)
    progress("many-channel leg done")
    batch = None if args.no_batch else batch_leg(sb, at, torch, workloads, args.no_tune)
    progress("batch leg done")
    serve = None
    if not args.no_serve:
        serve = []
        for q in args.serve_qps.split(","):
            serve.append(serve_leg(sb, torch, np, workloads, args.serve_requests, float(q)))
            progress(f"serving at {q} QPS done")

    if args.calibrate_copy_mb > 0:
        nb = int(args.calibrate_copy_mb * 1e6) // 4 * 4
        src = torch.empty(nb, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        torch.add(src, 0, out=dst)  # one elementwise kernel: reads and writes nb bytes
        torch.cuda.synchronize()

    line = {
        "metric": "stylized Mpixel/s at 1080p (HBM GB/s and p50/p99 frame latency alongside)",
        "value": round(mpx_s, 3),
        "unit": "Mpixel/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 6),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u8" if st_np.fmt == 0 else "u16",
        "data": "synthetic",
        "config": {"workload": wname, "width": w, "height": h,
                   "source": f"{st_np.sw}x{st_np.sh}", "levels": p.levels, "finest": p.finest,
                   "threshold": p.threshold, "radius": p.radius, "buffer_sets": nsets,
                   "tune": list(tune) if tune else "default", "streams": args.streams},
        "single_stream": {"ms_per_step": round(single_s * 1e3 / args.steps, 6),
                          "value": round(w * h * args.steps / single_s / 1e6, 3)},
        "frame_latency_ms": {"p50": round(float(frame_ms[len(frame_ms) // 2]), 6),
                             "p99": round(float(frame_ms[min(len(frame_ms) - 1,
                                                             int(0.99 * len(frame_ms)))]), 6)},
        "pass_ms": {"seeds": round(float(seeds_ms), 6), "assign": round(float(assign_ms), 6),
                    "vote": round(float(vote_ms), 6)},
        "hbm_gbs_algorithmic": round(pbytes / (ms_per_step * 1e-3) / 1e9, 2),
        "algorithmic_bytes_per_frame": pbytes,
        "style_registration_ms": round(lut_ms, 3),
        "roofline": {"bound": "hbm", "kernel": "k_blend (voting pass)",
                     "achieved": round(vote_gbs, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(vote_gbs / HBM_PEAK_GBS, 5),
                     "traffic": round(traffic) if traffic is not None else None,
                     "traffic_gbs": (round(traffic / (vote_ms * 1e-3) / 1e9, 2)
                                     if traffic is not None else None),
                     "kernel_ms": round(float(vote_ms), 6), "algorithmic_bytes": vbytes},
        "hbm_stream_copy_gbs": copy_gbs,
        "valu_issue": {"vote": valu_issue(wname, "k_blend<", float(vote_ms)),
                       "level_loop": valu_issue(wname, "k_assign<", float(assign_ms))},
        "cpu_baseline": cpu,
        "segmentation": seg,
        "animation": anim,
        "three_channels": chan,
        "many_channels": search,
        "batch": batch,
        "serve": serve,
    }
    print(json.dumps(line), flush=True)


def seg_leg(sb, torch, np, workloads, st_np, fr, prm, plain_ms, nlabels=6, steps=100):
    """The same frame with the segmentation guide: seeded Voronoi label maps
    (nlabels labels over 40 exemplar and 60 target regions), per-label
    lookup tables resident with the style."""
    ls = workloads.voronoi_labels(st_np.sw, st_np.sh, nlabels, 40, 11)
    lt = workloads.voronoi_labels(fr.w, fr.h, nlabels, 60, 12)
    style = sb.Style(st_np.rgb, st_np.guide, st_np.lut_bits, labels=ls, nlabels=nlabels)
    g_np = fr.guide.view(np.int16) if fr.guide.dtype == np.uint16 else fr.guide
    g = torch.from_numpy(g_np).cuda()
    jit = None  # the seeds come from the jitter hash of prm.seed
    ltd = torch.from_numpy(lt).cuda()
    rgb = torch.empty((fr.h, fr.w, 3), dtype=torch.uint8, device="cuda")
    chunk = torch.empty((fr.h, fr.w), dtype=torch.int32, device="cuda")
    ws = torch.empty(sb.workspace_bytes(fr.w, fr.h, prm), dtype=torch.uint8, device="cuda")

    def run():
        sb.stylize(style, g, jit, prm, out_rgb=rgb, out_chunk=chunk, workspace=ws, tgt_labels=ltd)

    for _ in range(10):
        run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        run()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    lv = chunk.cpu().numpy().view(np.uint32) >> 26
    return {"labels": nlabels, "ms_per_frame": round(ms, 6),
            "mpixel_per_s": round(fr.w * fr.h / (ms * 1e-3) / 1e6, 2),
            "vs_plain": round(plain_ms / ms, 3),
            "fallback_fraction": round(float((lv == prm.levels).mean()), 4),
            "label_tables_mib": round(style.label_luts.numel() * 4 / 2**20, 2)}


def channels_leg(sb, torch, np, workloads, plain_ms, steps=100):
    """The appearance workload: a 1080p target with two normal channels plus
    an appearance channel, the 512x512 style's exact table over 2^24 bins
    (three 8-bit channels).  Style registration (table build included) and
    the frame, against the two-channel frame of the main leg."""
    styles, frames = workloads.config(6)
    st_np, fr = styles[0], frames[0]
    p = fr.params
    prm = sb.params(p.levels, p.finest, p.threshold, p.radius, seed=fr.seed)
    style = sb.Style(st_np.rgb, st_np.guide, st_np.lut_bits)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    style = sb.Style(st_np.rgb, st_np.guide, st_np.lut_bits)
    torch.cuda.synchronize()
    reg_ms = (time.perf_counter() - t0) * 1e3
    g = torch.from_numpy(fr.guide).cuda()
    jit = None  # the seeds come from the jitter hash of prm.seed
    rgb = torch.empty((fr.h, fr.w, 3), dtype=torch.uint8, device="cuda")
    chunk = torch.empty((fr.h, fr.w), dtype=torch.int32, device="cuda")
    ws = torch.empty(sb.workspace_bytes(fr.w, fr.h, prm), dtype=torch.uint8, device="cuda")

    def run():
        sb.stylize(style, g, jit, prm, out_rgb=rgb, out_chunk=chunk, workspace=ws)

    for _ in range(10):
        run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        run()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    lv = chunk.cpu().numpy().view(np.uint32) >> 26
    return {"workload": workloads.CONFIG_NAMES[6], "ms_per_frame": round(ms, 6),
            "mpixel_per_s": round(fr.w * fr.h / (ms * 1e-3) / 1e6, 2),
            "vs_two_channel": round(plain_ms / ms, 3),
            "fallback_fraction": round(float((lv == p.levels).mean()), 4),
            "table_mib": round(style.lut.numel() * 4 / 2**20, 1),
            "style_registration_ms": round(reg_ms, 3)}


def search_leg(sb, torch, np, workloads, plain_ms, steps=50, cpu_frame=True):
    """Guides of many channels, each lookup the exact search on the k-d tree
    built on the GPU: the features workload at 1080p with five 8-bit channels
    (normals, appearance, chroma) and with four 16-bit ones (texture
    coordinates, normals); tree build, frame and passes, searches per frame.
    Also the three-channel appearance frame through the search instead of
    its 2^24-bin table, and one oracle frame for scale."""
    import oracle

    def frame_stats(style, guide_np, p, seed):
        prm = sb.params(p.levels, p.finest, p.threshold, p.radius, seed=seed)
        g = torch.from_numpy(guide_np.view(np.int16) if guide_np.dtype == np.uint16
                             else guide_np).cuda()
        h, w = guide_np.shape[:2]
        bufs = [(torch.empty((h, w, 3), dtype=torch.uint8, device="cuda"),
                 torch.empty((h, w), dtype=torch.int32, device="cuda"),
                 torch.empty(sb.workspace_bytes(w, h, prm), dtype=torch.uint8, device="cuda"))
                for _ in range(2)]
        plans = [sb.FramePlan(style, g, None, prm, o_rgb, o_chunk, o_ws)
                 for o_rgb, o_chunk, o_ws in bufs]
        rgb, chunk, ws = bufs[0]
        streams = [torch.cuda.current_stream().cuda_stream, torch.cuda.Stream().cuda_stream]

        def timed(nstreams):
            for k in range(5):
                plans[k % 2].launch(streams[k % nstreams])
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for k in range(steps):
                plans[k % 2].launch(streams[k % nstreams])
            torch.cuda.synchronize()
            return (time.perf_counter() - t0) * 1e3 / steps

        ms = timed(1)
        ms2 = timed(2)
        ev = sb.TimingEvents()
        passes = []
        for _ in range(20):
            sb.stylize(style, g, None, prm, out_rgb=rgb, out_chunk=chunk, workspace=ws, events=ev)
            torch.cuda.synchronize()
            passes.append(ev.pass_ms())
        ev.close()
        med = np.median(np.array(passes), axis=0)
        lv = chunk.cpu().numpy().view(np.uint32) >> 26
        nfb = int((lv == p.levels).sum())
        nseeds = int(sum(-(-w // (p.finest << k)) * -(-h // (p.finest << k))
                         for k in range(p.levels)))
        return {"ms_per_frame": round(ms, 6), "mpixel_per_s": round(w * h / (ms * 1e-3) / 1e6, 2),
                "two_streams": {"ms_per_frame": round(ms2, 6),
                                "mpixel_per_s": round(w * h / (ms2 * 1e-3) / 1e6, 2)},
                "pass_ms": {"seeds": round(float(med[0]), 6), "level_loop": round(float(med[1]), 6),
                            "vote": round(float(med[2]), 6)},
                "fallback_fraction": round(nfb / (w * h), 4),
                "searches_per_frame": nseeds + nfb,
                "searches_per_us": round((nseeds + nfb) / ((med[0] + med[1]) * 1e3), 1)}

    out = {}
    for depth, ch in ((8, 5), (16, 4)):
        styles, frames = workloads.config(7, depth=depth)
        st_np, fr = styles[0], frames[0]
        style = sb.Style(st_np.rgb, st_np.guide, channels=ch)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        style = sb.Style(st_np.rgb, st_np.guide, channels=ch)
        torch.cuda.synchronize()
        reg_ms = (time.perf_counter() - t0) * 1e3
        hdr = style.tree[:16].cpu().numpy().view(np.uint32)
        r = {"workload": workloads.CONFIG_NAMES[7], "channels": ch, "depth": depth,
             "threshold": fr.params.threshold, "style_registration_ms": round(reg_ms, 3),
             "tree_nodes": int(hdr[0]), "tree_mib": round(style.tree.numel() / 2**20, 1)}
        r.update(frame_stats(style, fr.guide, fr.params, fr.seed))
        r["vs_two_channel"] = round(plain_ms / r["ms_per_frame"], 3)
        if cpu_frame and depth == 8:
            p = fr.params
            c0 = time.perf_counter()
            oracle.stylize_n(st_np.rgb, st_np.guide, ch, fr.guide, None, p.levels, p.finest,
                             p.threshold, p.radius, seed=fr.seed)
            r["oracle_frame_s"] = round(time.perf_counter() - c0, 3)
            r["oracle_threads"] = oracle.set_threads(0)
        out[f"u{depth}x{ch}"] = r
    # the appearance workload (three 8-bit channels) through the search
    styles, frames = workloads.config(6)
    st_np, fr = styles[0], frames[0]
    style = sb.Style(st_np.rgb, st_np.guide, channels=3)
    r = {"workload": workloads.CONFIG_NAMES[6], "channels": 3, "depth": 8,
         "tree_mib": round(style.tree.numel() / 2**20, 1)}
    r.update(frame_stats(style, fr.guide, fr.params, fr.seed))
    out["u8x3_search"] = r
    return out


def anim_leg(sb, torch, np, workloads, style, w, h, p, nframes=12, reps=5):
    """The per-frame seed schedule on a static and on an animated target
    (drifting bumps): the fraction of pixels whose source coordinate / chunk
    code changes between consecutive frames as a function of the threshold
    t -- static target with seeds re-drawn every frame (the flicker alone),
    moving target with seeds held (the motion alone) and moving target with
    seeds re-drawn; 12-frame sequences as one batch; then sessions of
    60 fps frames served with in-order completion."""
    import paper_1807_03249_amd.serve as sv

    guides_np = workloads.animated_bump_guides(w, h, 64, nframes, 3.0, 601)
    guides = [torch.from_numpy(g).cuda() for g in guides_np]
    pool = [torch.from_numpy(workloads.jitter_table(w, h, p.levels, p.finest, 610 + k)
                             .view(np.int32)).cuda() for k in range(16)]
    held = [pool[0]] * nframes
    redrawn = pool[:nframes]
    base = int(p.threshold)
    ts = sorted({0, base // 4, base // 2, base, 2 * base, 4 * base, 16 * base, 64 * base})
    b = sb.Batch(use_graph=True)
    outs = [(torch.empty((h, w, 3), dtype=torch.uint8, device="cuda"),
             torch.empty((h, w), dtype=torch.int32, device="cuda"),
             torch.empty((h, w), dtype=torch.int32, device="cuda")) for _ in range(nframes)]
    ws = None
    cws = torch.empty(sb.lib().sb_change_workspace_bytes(), dtype=torch.uint8, device="cuda")
    counts = torch.empty((nframes - 1, 2), dtype=torch.int64, device="cuda")
    sweep = []
    seq_ms = None
    for t in ts:
        prm = sb.params(p.levels, p.finest, t, p.radius)
        row = {"t": t}
        cases = (("static_redrawn", [guides[0]] * nframes, redrawn),
                 ("moving_held", guides, held), ("moving_redrawn", guides, redrawn))
        for name, gs, jits in cases:
            jobs = [sb.FrameJob(style, g, j, prm, o[0], o[1], o[2])
                    for g, j, o in zip(gs, jits, outs)]
            if ws is None:
                ws = torch.empty(b.workspace_bytes(jobs), dtype=torch.uint8, device="cuda")
            b.run(jobs, workspace=ws)
            for k in range(nframes - 1):
                sb.frame_change(outs[k][1], outs[k + 1][1], outs[k][2], outs[k + 1][2],
                                counts=counts[k], workspace=cws)
            c = counts.cpu().numpy().astype(np.float64) / (w * h)
            lv = (outs[0][1].cpu().numpy().view(np.uint32) >> 26)
            row[name] = {"src_changed": round(float(c[:, 1].mean()), 4),
                         "chunk_changed": round(float(c[:, 0].mean()), 4),
                         "fallback": round(float((lv == p.levels).mean()), 4)}
            if t == base and name == "moving_redrawn":
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                for _ in range(reps):
                    b.run(jobs, workspace=ws)
                torch.cuda.synchronize()
                seq_ms = (time.perf_counter() - t0) * 1e3 / reps
        sweep.append(row)
    b.close()
    res = {"frames": nframes, "size": f"{w}x{h}", "drift_px_per_frame": 3.0, "sweep": sweep,
           "sequence_ms": round(seq_ms, 4),
           "sequence_mpixel_per_s": round(nframes * w * h / (seq_ms * 1e-3) / 1e6, 2)}

    # sessions: S viewers at 60 fps for one second, random phases; frame k of
    # session s shows guide (k + s) mod nframes with a fresh jitter table
    prm = sb.params(p.levels, p.finest, p.threshold, p.radius)
    rng = np.random.default_rng(620)
    res["sessions"] = []
    for nses in (32, 128, 256):
        phase = rng.uniform(0.0, 1.0, nses)
        reqs = []
        for k in range(60):
            for s in range(nses):
                reqs.append(((k + phase[s]) / 60.0, s, k))
        reqs.sort()
        rq = [sv.Request(a, style, guides[(k + s) % nframes], pool[(s * 13 + k) % len(pool)],
                         prm, session=s) for a, s, k in reqs]
        ent = {"sessions": nses, "fps": 60, "frames": len(rq)}
        for name, kw in (("batched", dict(slots=8, max_batch=4, use_graph=False)),
                         ("plain", dict(plain=True))):
            out = sv.run(rq, budget_bytes=1 << 30, **kw)
            summ = sv.summarize(out, pixels=np.full(len(rq), float(w * h)))
            order = all(np.all(np.diff(out["completed"][out["session"] == s]) >= 0)
                        for s in range(nses))
            ent[name] = {"p50_ms": round(summ["p50_ms"], 4), "p99_ms": round(summ["p99_ms"], 4),
                         "frames_per_s": round(summ["req_per_s"], 1),
                         "mean_batch": round(summ["mean_batch"], 2), "in_order": bool(order)}
        res["sessions"].append(ent)
    return res


def batch_leg(sb, at, torch, workloads, no_tune, reps=5):
    """64 frames of uneven size, half normal- and half UV-guided, 4 resident
    styles: one autotuned batch plan run per batch vs the same 64 frames through
    the per-frame kernels, launched from one C call (sb_stylize_frames) with
    the same kernel choice."""
    import numpy as np

    styles_np, frames_np = workloads.config(4)
    styles = [sb.Style(s.rgb, s.guide, s.lut_bits) for s in styles_np]
    jobs = []
    for f in frames_np:
        p = f.params
        jobs.append(sb.FrameJob(styles[f.style], f.guide, f.jitter,
                                sb.params(p.levels, p.finest, p.threshold, p.radius, seed=f.seed)))
    px = sum(j.w * j.h for j in jobs)
    probe = sb.Batch(use_graph=True)
    ws = torch.empty(probe.workspace_bytes(jobs), dtype=torch.uint8, device="cuda")
    probe.close()
    if no_tune:
        pick = {"tune": None, "blocks_per_cu": 0, "cached": False}
    else:
        pick = at.tune_batch(jobs, workspace=ws)
    b = sb.Batch(use_graph=True, tune=pick["tune"], blocks_per_cu=pick["blocks_per_cu"])
    plain_ws = torch.empty(max(sb.workspace_bytes(j.w, j.h, j.params) for j in jobs),
                           dtype=torch.uint8, device="cuda")

    def run_batch():
        b.run(jobs, workspace=ws)

    def run_plain():
        sb.stylize_frames(jobs, workspace=plain_ws, tune=pick["tune"])

    # the same per-frame launches split over two streams (halves of the list)
    side = torch.cuda.Stream()
    plain_ws2 = torch.empty_like(plain_ws)
    half = len(jobs) // 2

    def run_plain2():
        side.wait_stream(torch.cuda.current_stream())
        sb.stylize_frames(jobs[:half], workspace=plain_ws, tune=pick["tune"])
        with torch.cuda.stream(side):
            sb.stylize_frames(jobs[half:], workspace=plain_ws2, tune=pick["tune"])
        torch.cuda.current_stream().wait_stream(side)

    out = {}
    for name, fn in (("graph", run_batch), ("plain", run_plain), ("plain_2_streams", run_plain2)):
        fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / reps
        out[name] = {"ms_per_batch": round(ms, 4), "mpixel_per_s": round(px / (ms * 1e-3) / 1e6, 2)}
    b.close()
    # algorithmic bytes of the whole batch: every frame's own bytes (guide,
    # RGB, chunk map, touched table entries) and each distinct style's
    # exemplar once per launch
    nbytes = 0
    for j, f in zip(jobs, frames_np):
        p = f.params
        chunk = j.out_chunk.cpu().numpy().view(np.uint32)
        nfb = int(((chunk >> 26) == p.levels).sum())
        nseeds = sb.jitter_len(j.w, j.h, p.levels, p.finest)
        nbytes += path_algorithmic_bytes(j.w, j.h, j.style.fmt, 0, 0, nseeds, nfb)
    for st in styles_np:
        nbytes += st.sw * st.sh * (3 + (2 if st.fmt == 0 else 4))
    gms = out["graph"]["ms_per_batch"]
    out["algorithmic_bytes"] = nbytes
    out["hbm_gbs_algorithmic"] = round(nbytes / (gms * 1e-3) / 1e9, 2)
    out["roofline_frac"] = round(nbytes / (gms * 1e-3) / 1e9 / HBM_PEAK_GBS, 5)
    out["frames"] = len(jobs)
    out["mpixel"] = round(px / 1e6, 3)
    out["speedup"] = round(out["plain"]["ms_per_batch"] / out["graph"]["ms_per_batch"], 3)
    out["tune"] = list(pick["tune"]) if pick["tune"] else "default"
    out["blocks_per_cu"] = pick["blocks_per_cu"] or "default"
    out["plain_launch"] = ("sb_stylize_frames (one C call, per-frame kernels, same tune); "
                           "plain_2_streams: the two halves of the list on two streams")
    return out


def serve_leg(sb, torch, np, workloads, nreq, qps):
    """Poisson trace at a fixed QPS over 8 resident styles and three frame
    sizes: continuous batching (4 streams) vs the plain per-request path."""
    import paper_1807_03249_amd.serve as sv

    trace = workloads.config(5, requests=nreq, qps=qps, pool=2)
    styles = [sb.Style(s.rgb, s.guide, s.lut_bits) for s in trace["styles"]]
    guides = {}
    reqs, px = [], []
    for i in range(nreq):
        si, st = int(trace["size_idx"][i]), int(trace["style_idx"][i])
        fmt = trace["styles"][st].fmt
        key = (si, fmt, int(trace["pool_idx"][i]))
        if key not in guides:
            g = trace["guides"][key]
            guides[key] = torch.from_numpy(g.view(np.int16) if g.dtype == np.uint16 else g).cuda()
        g = guides[key]
        h, w = int(g.shape[0]), int(g.shape[1])
        p = trace["params"][fmt]
        # every request its own jitter hash seed (per-frame seeds, no table)
        reqs.append(sv.Request(float(trace["arrivals"][i]), styles[st], g, None,
                               sb.params(p.levels, p.finest, p.threshold, p.radius,
                                         seed=int(trace["seeds"][i]))))
        px.append(w * h)
    px = np.array(px, dtype=np.float64)
    res = {"qps": qps, "requests": nreq, "budget_mib": 1024}
    # continuous batching: 8 slots (streams), each taking up to 4 admitted
    # requests per launch as direct launches with exact grids; the same on 4
    # slots as captured graphs of up to 16 (the grid given, so that every
    # batch replays one); per-request launches on 8 slots
    # (no batching, same overlap); one stream, one request per launch, in
    # arrival order (the plain path)
    for name, kw in (("batched", dict(slots=8, max_batch=4, use_graph=False)),
                     ("batched_graph_4", dict(slots=4, max_batch=16, use_graph=True,
                                             blocks_per_cu=16)),
                     ("per_request_8", dict(slots=8, max_batch=1)),
                     ("plain", dict(plain=True))):
        out = sv.run(reqs, budget_bytes=1 << 30, **kw)
        summ = sv.summarize(out, pixels=px)
        is1080 = np.array([r.w == 1920 for r in reqs])
        k = int(nreq * 0.05)
        lat = out["latency"][k:][is1080[k:]] * 1e3
        summ["p50_ms_1080p"] = float(np.percentile(lat, 50)) if lat.size else None
        summ["p99_ms_1080p"] = float(np.percentile(lat, 99)) if lat.size else None
        res[name] = {k2: (round(v, 4) if isinstance(v, float) else v) for k2, v in summ.items()}
    return res


if __name__ == "__main__":
    main()
