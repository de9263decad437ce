"""The routes of a batch: replays of the plan's graph with every kind of frame and a
frame set that changes from replay to replay, direct launches from pageable
descriptors, and the rule that chooses between graph and direct launches.  Every
frame equals the frame alone.  Tolerance 0."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1807_03249_amd as m

    m.lib()
    return m


def _guide(gen, fmt, h, w):
    """Smooth random channels of a guide format."""
    import torch

    k, top = {"u8x2": (2, 255), "u16x2": (2, 65535), "u8x3": (4, 255), "u8xn": (8, 255)}[fmt]
    lat = torch.rand(1, k, h // 12 + 2, w // 12 + 2, generator=gen, device="cuda")
    v = torch.nn.functional.interpolate(lat, (h, w), mode="bilinear")[0].permute(1, 2, 0) * top
    v = v.to(torch.int32)
    return (v.to(torch.int16) if fmt == "u16x2" else v.to(torch.uint8)).contiguous()


def _style(sb, gen, fmt, size=48, labels=0):
    import torch

    rgb = (torch.rand(size, size, 3, generator=gen, device="cuda") * 255).byte()
    kw = {}
    if labels:
        kw = {"labels": torch.randint(0, labels, (size, size), generator=gen, device="cuda").byte(),
              "nlabels": labels}
    if fmt == "u8xn":
        return sb.Style(rgb, _guide(gen, fmt, size, size), channels=5)
    return sb.Style(rgb, _guide(gen, fmt, size, size), 6, **kw)


# (format, w, h, levels, finest, threshold, radius, labels)
FRAMES = [("u8x2", 200, 90, 3, 8, 48, 3, 0), ("u16x2", 97, 61, 4, 8, 1 << 20, 7, 0),
          ("u8x3", 130, 70, 3, 8, 200, 4, 0), ("u8x2", 75, 131, 9, 8, 64, 1, 0),
          ("u8x2", 160, 120, 3, 16, 90, 2, 4), ("u16x2", 64, 48, 2, 4, 1 << 18, 0, 0),
          ("u8xn", 90, 75, 3, 8, 160, 3, 0), ("u8x3", 33, 200, 1, 8, 300, 6, 0),
          ("u8x2", 17, 9, 0, 8, 48, 5, 0)]


def _jobs(sb, gen, seed=0):
    import torch

    jobs = []
    for i, (fmt, w, h, levels, finest, threshold, radius, labels) in enumerate(FRAMES):
        lab = torch.randint(0, labels, (h, w), generator=gen, device="cuda").byte() if labels else None
        jobs.append(sb.FrameJob(_style(sb, gen, fmt, labels=labels), _guide(gen, fmt, h, w), None,
                                sb.params(levels, finest, threshold, radius, seed=seed + i),
                                tgt_labels=lab))
    return jobs


def _check(sb, jobs):
    import torch

    for i, j in enumerate(jobs):
        kw = {"tgt_labels": j.tgt_labels} if j.tgt_labels is not None else {}
        rgb, chunk = sb.stylize(j.style, j.guide, None, j.params, **kw)[:2]
        assert torch.equal(j.out_chunk, chunk), f"frame {i} chunk"
        assert torch.equal(j.out_rgb, rgb), f"frame {i} rgb"


def _mark_tail(sb, plan):
    """A word past every batch's frames in the next descriptor half: the copy of
    a graph takes it to the device, a direct launch reads only what it uses."""
    half = plan.desc_dev.numel() // 2
    at = half * plan._k + half - 8
    plan.desc_host[at:at + 8] = 0x5A
    plan.desc_dev[at:at + 8] = 0
    return at


def _replayed(plan, at):
    return bool((plan.desc_dev[at:at + 8] == 0x5A).all())


@pytest.mark.parametrize("graph,bpc", [(True, 16), (True, 1), (True, 0), (False, 0)])
def test_every_kind_of_frame(sb, graph, bpc):
    """Labels, three channels, radius 4 to 7, nine levels, cells smaller than
    blocks and searched frames, in sets that change from run to run with eager
    work and synchronisation between the runs."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    jobs = _jobs(sb, gen)
    plan = sb.Batch(use_graph=graph, blocks_per_cu=bpc)
    print(f"[gpu-case] every kind of frame graph={graph} blocks_per_cu={bpc}", flush=True)
    for run, pick in enumerate([range(9), (4, 1, 7), (6, 3), (2,), (8, 5, 0, 6), range(8, -1, -1)]):
        some = [jobs[i] for i in pick]
        for j in some:
            j.out_rgb.fill_(0x5A)
            j.out_chunk.fill_(-1)
        at = _mark_tail(sb, plan)
        plan.run(some)
        torch.cuda.synchronize()
        assert _replayed(plan, at) == (graph and bpc > 0), "route"
        _check(sb, some)
    # back to back, both descriptor halves in flight
    sets = [[0, 1, 2, 4], [3, 5, 7], [6, 4, 0], [8, 7, 1]]
    for pick in sets:
        plan.run([jobs[i] for i in pick])
    torch.cuda.synchronize()
    _check(sb, jobs)
    plan.close()


def test_searched_frames_do_not_count(sb):
    """A searched frame of 26 Mpixel beside a small one of a table format: the
    graph would run only the small one."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    w, h = 8192, 3200
    big = sb.FrameJob(_style(sb, gen, "u8xn", 8),
                      torch.zeros(h, w, 8, dtype=torch.uint8, device="cuda"), None,
                      sb.params(1, 64, 1 << 30, 0, seed=3))
    small = _jobs(sb, gen)[0]
    plan = sb.Batch()
    print("[gpu-case] searched frames do not count", flush=True)
    at = _mark_tail(sb, plan)
    plan.run([small, big])
    torch.cuda.synchronize()
    assert not _replayed(plan, at)
    _check(sb, [small, big])
    plan.close()


def test_large_batch_replays(sb):
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    st = _style(sb, gen, "u8x2")
    g = _guide(gen, "u8x2", 2160, 3840)
    plan = sb.Batch()
    print("[gpu-case] large batch replays", flush=True)
    for frames, graph in ((3, False), (4, True)):
        jobs = [sb.FrameJob(st, g, None, sb.params(4, 8, 48, 2, seed=f)) for f in range(frames)]
        at = _mark_tail(sb, plan)
        plan.run(jobs)
        torch.cuda.synchronize()
        assert _replayed(plan, at) == graph
        _check(sb, jobs)
    plan.close()


def test_pageable_descriptors(sb):
    """Descriptors in host memory that kernels cannot read, or at an odd address
    in memory they can: uploaded by a copy."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(10)
    jobs = _jobs(sb, gen)
    L = sb.lib()
    nb = L.sb_batch_desc_bytes()
    dev = torch.empty(nb, dtype=torch.uint8, device="cuda")
    pinned = torch.zeros(nb + 4, dtype=torch.uint8).pin_memory()
    pageable = np.zeros(nb, np.uint8)
    arr = (sb.SbFrame * len(jobs))(*[j.c() for j in jobs])
    wsb = L.sb_batch_workspace_bytes(arr, len(jobs))
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for name, host in (("pageable", pageable.ctypes.data), ("odd", pinned.data_ptr() + 4)):
        print(f"[gpu-case] descriptors {name}", flush=True)
        plan = ctypes.c_void_p()
        stream = torch.cuda.current_stream().cuda_stream
        assert L.sb_batch_create(dev.data_ptr(), host, 0, None, 0, stream,
                                 ctypes.byref(plan)) == sb.SB_OK
        for run in range(3):
            for j in jobs:
                j.out_rgb.fill_(0x5A)
                j.out_chunk.fill_(-1)
            assert L.sb_batch_run(plan, arr, len(jobs), ws.data_ptr(), wsb, stream) == sb.SB_OK
            torch.cuda.synchronize()
            _check(sb, jobs)
        assert L.sb_batch_destroy(plan) == sb.SB_OK


@pytest.mark.filterwarnings("ignore:The CUDA Graph is empty")
def test_small_batch_while_capturing(sb):
    """A graph plan's run on a stream that is being captured runs at once, for
    small batches as for large: recorded, its replays would read a descriptor
    half that later runs have filled for other frames."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    jobs = _jobs(sb, gen)[:6]
    plan = sb.Batch()
    ws = torch.empty(plan.workspace_bytes(jobs), dtype=torch.uint8, device="cuda")
    plan.run(jobs, ws)
    torch.cuda.synchronize()
    want = [(j.out_rgb.clone(), j.out_chunk.clone()) for j in jobs]
    for j in jobs:
        j.out_rgb.fill_(0x5A)
    torch.cuda.synchronize()
    print("[gpu-case] small batch while capturing", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.run(jobs, ws)
    torch.cuda.synchronize()
    for j, (rgb, chunk) in zip(jobs, want):
        assert torch.equal(j.out_rgb, rgb) and torch.equal(j.out_chunk, chunk)
    for _ in range(3):  # and the plan goes on
        for j in jobs:
            j.out_rgb.fill_(0x5A)
        plan.run(jobs, ws)
        torch.cuda.synchronize()
        for j, (rgb, chunk) in zip(jobs, want):
            assert torch.equal(j.out_rgb, rgb) and torch.equal(j.out_chunk, chunk)
    plan.close()
