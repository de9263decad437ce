"""Style registration on the GPU (lookup tables and search trees) at the sizes
where the build kernels change their split, against the oracle.  Tolerance 0:
every entry is a source coordinate."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1807_03249_amd as m

    m.lib()
    return m


# sides around one scan block (4^6 buckets from 128 x 128 pixels on), several
# blocks, fewer pixels than a wave, and a last wave with one pixel
@pytest.mark.parametrize("sw,sh,bits,spread", [(1, 1, 3, "noise"), (13, 5, 8, "noise"),
                                               (129, 127, 8, "smooth"), (130, 131, 9, "runs"),
                                               (256, 256, 9, "noise"), (301, 260, 11, "smooth"),
                                               (256, 257, 4, "one")])
def test_16bit_table(sb, sw, sh, bits, spread):
    """The bucket sort behind a 16-bit table: runs of equal buckets within and
    across waves, every pixel in one bucket, and a label no pixel holds."""
    rng = np.random.default_rng(sw * 1000 + sh)
    if spread == "smooth":  # neighbours share buckets, as in texture coordinates
        y, x = np.mgrid[0:sh, 0:sw]
        g = np.stack([x * 65536 // sw, y * 65536 // sh], -1)
    elif spread == "runs":
        g = np.repeat(rng.integers(0, 65536, (sh, (sw + 9) // 10, 2)), 10, 1)[:, :sw]
    else:
        g = rng.integers(0, 65536 if spread == "noise" else 1, (sh, sw, 2)) + (spread == "one") * 777
    g = np.ascontiguousarray(g.astype(np.uint16))
    rgb = rng.integers(0, 256, (sh, sw, 3)).astype(np.uint8)
    labels = rng.integers(0, 2, (sh, sw)).astype(np.uint8)  # label 2 is absent
    print(f"[gpu-case] 16-bit table {sw}x{sh} bits={bits} {spread}", flush=True)
    st = sb.Style(rgb, g, bits, labels=labels, nlabels=3)
    np.testing.assert_array_equal(st.lut.cpu().numpy().view(np.uint32), oracle.lut_build(g, bits))
    np.testing.assert_array_equal(st.label_luts.cpu().numpy().view(np.uint32),
                                  oracle.lut_build_labels(g, labels, 3, bits))


# texel counts around a run of eight, a power of eight, one workgroup's sort
# (2048), and the splits over the chip (an odd remainder, a last segment of one
# texel, a full one); "few": most texels are duplicates, "one": all are,
# "outlier": the histogram of every split has nearly all texels in one bin
@pytest.mark.parametrize("depth,channels,sw,sh,spread,queries", [
    (8, 5, 8, 1, "noise", 400), (8, 3, 3, 3, "noise", 400), (16, 4, 16, 4, "noise", 400),
    (16, 7, 13, 5, "few", 400), (8, 8, 64, 32, "noise", 600), (8, 5, 683, 3, "few", 600),
    (16, 2, 64, 64, "outlier", 600), (16, 4, 241, 17, "outlier", 600),
    (8, 5, 128, 128, "one", 600), (8, 2, 257, 255, "few", 600), (16, 8, 300, 219, "noise", 600),
    (8, 6, 512, 513, "smooth", 500), (8, 5, 50, 41, "smooth", 70001)])
def test_search_tree(sb, depth, channels, sw, sh, spread, queries):
    """The many-channel tree at every kind of size its build tells apart, and
    queries on either side of the change from eight lanes a query to four."""
    rng = np.random.default_rng(depth * 1000 + sw)
    top, dt = (1 << depth) - 1, np.uint8 if depth == 8 else np.uint16
    elems = oracle.texel_bytes(depth, channels) * 8 // depth
    if spread == "smooth":
        y, x = np.mgrid[0:sh, 0:sw]
        g = np.stack([(np.sin(x / (7 + k)) + np.cos(y / (5 + k)) + 2) * top / 4
                      for k in range(elems)], -1)
    else:
        g = rng.integers(0, top + 1, (sh, sw, elems))
        if spread == "few":
            g = g[:1, :5][np.zeros((sh, sw), int), rng.integers(0, min(sw, 5), (sh, sw))]
        elif spread == "one":
            g[:] = g[0, 0]
        elif spread == "outlier":
            g = np.where(rng.random((sh, sw, elems)) < 0.002, g, g & 7)
    g = np.ascontiguousarray(g.astype(dt))
    q = rng.integers(0, top + 1, (queries, elems)).astype(dt)
    q[::3] = g.reshape(-1, elems)[rng.integers(0, sw * sh, len(q[::3]))]  # exact hits: ties
    print(f"[gpu-case] search tree {depth}x{channels} {sw}x{sh} {spread} {queries}", flush=True)
    import torch

    st = sb.Style(np.zeros((sh, sw, 3), np.uint8), g, channels=channels)
    qt = torch.from_numpy(q.view(np.int16) if depth == 16 else q).cuda()
    got = st.query(qt).cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, oracle.nn_query_n(g, channels, q))


# bits around the first bins' spacing (1 to 64 bins apart), one site, one value
# along a channel, lines without any, dense noise, and zero and large weights
@pytest.mark.parametrize("channels,bits,spread,weights", [
    (2, 1, "noise", None), (2, 4, "line", None), (2, 7, "sphere", None), (2, 8, "one", None),
    (2, 8, "noise", None), (3, 1, "noise", None), (3, 2, "one", [127, 1, 3]),
    (3, 4, "sphere", [1, 0, 127]), (3, 5, "line", [2, 3, 5]), (3, 6, "noise", None)])
def test_8bit_table(sb, channels, bits, spread, weights):
    """The separable passes: every bin's minimum found between its neighbours'."""
    rng = np.random.default_rng(channels * 100 + bits)
    sh, sw = 67, 61
    g = rng.integers(0, 256, (sh, sw, 4 if channels == 3 else 2)).astype(np.uint8)
    if spread == "one":
        g[:] = g[0, 0]
    elif spread == "line":  # one channel constant: whole planes hold no site
        g[..., channels - 1] = 77
    elif spread == "sphere":
        y, x = np.mgrid[0:sh, 0:sw]
        g[..., 0], g[..., 1] = np.clip(x * 4, 20, 200), np.clip(y * 4, 20, 200)
    rgb = np.zeros((sh, sw, 3), np.uint8)
    print(f"[gpu-case] 8-bit table channels={channels} bits={bits} {spread} {weights}", flush=True)
    st = sb.Style(rgb, g, bits, weights=weights)
    want = oracle.lut_build(g, bits, weights) if channels == 3 else oracle.lut_build(g, bits)
    np.testing.assert_array_equal(st.lut.cpu().numpy().view(np.uint32), want)


# source widths on and off multiples of four, one texel, rows shorter than four
@pytest.mark.parametrize("sw,sh,offset", [(1, 1, 0), (3, 2, 0), (4, 3, 0), (5, 4, 0), (64, 5, 0),
                                          (62, 33, 0), (64, 9, 1)])
def test_padded_exemplar(sb, sw, sh, offset):
    """The packed exemplar: texels R | G << 8 | B << 16 | 1 << 24 inside an
    empty margin of 8, zero rows after it; `offset`: the bytes start unaligned."""
    import torch

    rng = np.random.default_rng(sw * 100 + sh)
    buf = torch.from_numpy(rng.integers(0, 256, sw * sh * 3 + offset).astype(np.uint8)).cuda()
    n = int(sb.lib().sb_exemplar_texels(sw, sh))
    out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    print(f"[gpu-case] padded exemplar {sw}x{sh} +{offset}", flush=True)
    rc = sb.lib().sb_pack_exemplar(buf.data_ptr() + offset, sw, sh, out.data_ptr(), None)
    assert rc == sb.SB_OK
    torch.cuda.synchronize()
    rgb = buf.cpu().numpy()[offset:].reshape(sh, sw, 3).astype(np.uint32)
    want = np.zeros(n, np.uint32)
    rows = want[:n // (sw + 16) * (sw + 16)].reshape(-1, sw + 16)
    rows[8:8 + sh, 8:8 + sw] = rgb[..., 0] | rgb[..., 1] << 8 | rgb[..., 2] << 16 | 1 << 24
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)


# one level, more records than lanes (9 x 11), frames of a block and a pixel
# more, cells smaller than blocks, and no level at all
@pytest.mark.parametrize("depth,channels,w,h,levels,finest", [
    (8, 5, 97, 61, 1, 8), (16, 4, 97, 61, 11, 8), (8, 3, 8, 8, 4, 8), (8, 7, 17, 9, 9, 16),
    (16, 7, 40, 33, 3, 8), (16, 2, 70, 50, 3, 4), (8, 5, 41, 23, 0, 8)])
def test_search_level_loop(sb, depth, channels, w, h, levels, finest):
    """Many-channel frames on both level loops, every output against the oracle."""
    import torch

    rng = np.random.default_rng(w * 100 + levels)
    elems, dt = oracle.texel_bytes(depth, channels) * 8 // depth, np.uint8 if depth == 8 else np.uint16
    top = (1 << depth) - 1

    def guide(rows, cols):
        y, x = np.mgrid[0:rows, 0:cols]
        g = [(np.sin(x / (9 + k)) + np.cos(y / (7 + k)) + 2) * top / 4 for k in range(elems)]
        return np.ascontiguousarray(np.stack(g, -1).astype(dt))

    src, tgt = guide(48, 52), guide(h, w)
    rgb = rng.integers(0, 256, (48, 52, 3)).astype(np.uint8)
    t = (top // 16) ** 2
    print(f"[gpu-case] search level loop {depth}x{channels} {w}x{h} L={levels} finest={finest}",
          flush=True)
    st = sb.Style(rgb, src, channels=channels)
    tg = torch.from_numpy(tgt.view(np.int16) if depth == 16 else tgt).cuda()
    got = sb.stylize(st, tg, None, sb.params(levels, finest, t, 2, seed=5), want_nnf=True)
    want = oracle.stylize_n(rgb, src, channels, tgt, None, levels, finest, t, 2, seed=5)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a.cpu().numpy().view(b.dtype).reshape(b.shape), b)
