"""The default kernel choice of a frame follows its size, format and threshold;
on both sides of every line the default's outputs equal an explicit choice's
(which other tests compare with the oracle).  Tolerance 0."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1807_03249_amd as m

    m.lib()
    return m


# 2^18 and 2^19 pixels, 3 * 2^20 with thresholds about the uniform-window rule
@pytest.mark.parametrize("fmt,w,h,size,threshold,radius", [
    ("u8x2", 512, 512, 64, 32, 3), ("u8x2", 513, 512, 64, 32, 3), ("u8x2", 1024, 512, 64, 32, 2),
    ("u8x2", 1025, 512, 64, 32, 7), ("u8x2", 2048, 1536, 64, 1024, 3),
    ("u8x2", 2048, 1536, 64, 1023, 3), ("u8x2", 2047, 1536, 64, 1024, 3),
    ("u16x2", 2048, 1537, 128, 1 << 20, 3), ("u16x2", 2048, 1537, 128, (1 << 20) - 1, 3),
    ("u8x3", 2048, 1536, 64, 4096, 1), ("u8x3", 300, 200, 64, 192, 4)])
def test_default_choice(sb, fmt, w, h, size, threshold, radius):
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(w * 10 + h)

    def guide(rows, cols, period):
        # smooth random channels: chunks of every size
        k, top = (4 if fmt == "u8x3" else 2), (65535 if fmt == "u16x2" else 255)
        lat = torch.rand(1, k, rows // period + 2, cols // period + 2, generator=gen, device="cuda")
        v = torch.nn.functional.interpolate(lat, (rows, cols), mode="bilinear")[0]
        v = (v * top).to(torch.int32).permute(1, 2, 0).contiguous()
        return v.to(torch.int16) if fmt == "u16x2" else v.to(torch.uint8)

    rgb = (torch.rand(size, size, 3, generator=gen, device="cuda") * 255).to(torch.uint8)
    st = sb.Style(rgb, guide(size, size, 16), 6)
    tgt = guide(h, w, 64)
    p = sb.params(4, 8, threshold, radius, seed=w)
    print(f"[gpu-case] default choice {fmt} {w}x{h} t={threshold} r={radius}", flush=True)
    got = sb.stylize(st, tgt, None, p, want_nnf=True)
    want = sb.stylize(st, tgt, None, p, want_nnf=True, tune=(4, 16, 4, 4, 1))
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# below and above the size from which a plan with a default grid replays its
# graph, and either side of it with the grid given (a graph) or no graph at all
@pytest.mark.parametrize("frames,graph,bpc", [(2, True, 0), (3, True, 0), (4, True, 0),
                                              (2, True, 4), (4, False, 0)])
def test_batch_routes(sb, frames, graph, bpc):
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(frames)
    size, w, h = 64, 3840, 2160
    styles = [sb.Style((torch.rand(size, size, 3, generator=gen, device="cuda") * 255).byte(),
                       (torch.rand(size, size, 2, generator=gen, device="cuda") * 255).byte(), 6)
              for _ in range(2)]
    lat = torch.rand(frames, 2, h // 40 + 2, w // 40 + 2, generator=gen, device="cuda")
    v = torch.nn.functional.interpolate(lat, (h, w), mode="bilinear")
    guides = (v * 255).byte().permute(0, 2, 3, 1).contiguous()
    print(f"[gpu-case] batch of {frames} graph={graph} blocks_per_cu={bpc}", flush=True)
    plan = sb.Batch(use_graph=graph, blocks_per_cu=bpc)
    for run in range(3):  # both descriptor halves, and one again
        jobs = [sb.FrameJob(styles[f % 2], guides[f], None, sb.params(4, 8, 48, 3, seed=run * 9 + f))
                for f in range(frames)]
        plan.run(jobs)
        for j in jobs:
            rgb, chunk = sb.stylize(j.style, j.guide, None, j.params)
            assert torch.equal(j.out_rgb, rgb) and torch.equal(j.out_chunk, chunk)
