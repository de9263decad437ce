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
