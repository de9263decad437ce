"""The search tree that a registration leaves in device memory: equal texels are one,
every box and key that of the texels below it, so a guide of few values is as cheap
to search as one of few texels.  Tolerance 0."""
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


def _start(level):
    return (8 ** level - 1) // 7


def _up256(x):
    return (x + 255) // 256 * 256


def _guide(rng, depth, channels, sw, sh, spread):
    top, dt = (1 << depth) - 1, np.uint8 if depth == 8 else np.uint16
    elems = oracle.texel_bytes(depth, channels) * 8 // depth
    y, x = np.mgrid[0:sh, 0:sw]
    if spread == "noise":
        g = rng.integers(0, top + 1, (sh, sw, elems))
    elif spread == "one":
        g = np.zeros((sh, sw, elems)) + rng.integers(0, top + 1, elems)
    elif spread == "few":
        g = rng.integers(0, top + 1, (5, elems))[rng.integers(0, 5, (sh, sw))]
    elif spread == "steps":  # smooth, in eighths of the range
        g = np.stack([(np.sin(x / (9 + k)) + np.cos(y / (7 + k)) + 2) * top / 4
                      for k in range(elems)], -1) // (top // 8) * (top // 8)
    else:  # "half": a constant left half beside noise
        g = rng.integers(0, top + 1, (sh, sw, elems))
        g[:, : sw // 2] = top // 3
    g = np.ascontiguousarray(g.astype(dt))
    g[..., channels:] = rng.integers(0, top + 1, g[..., channels:].shape)  # to be ignored
    return g


# fewer texels than a node, one more than a power of eight, one workgroup's merge
# and more, one sort's block and more, and every kind of duplicates
@pytest.mark.parametrize("depth,channels,sw,sh,spread", [
    (8, 5, 1, 1, "one"), (8, 3, 5, 1, "few"), (16, 4, 13, 5, "noise"), (8, 2, 64, 48, "noise"),
    (16, 7, 33, 31, "few"), (8, 5, 129, 127, "one"), (8, 5, 160, 150, "steps"),
    (16, 4, 200, 90, "steps"), (8, 8, 150, 161, "half"), (16, 2, 100, 97, "half")])
def test_tree_of_distinct_texels(sb, depth, channels, sw, sh, spread):
    rng = np.random.default_rng(depth * 1000 + sw)
    g = _guide(rng, depth, channels, sw, sh, spread)
    n, t = sw * sh, g.shape[2] * depth // 8
    print(f"[gpu-case] tree shape {depth}x{channels} {sw}x{sh} {spread}", flush=True)
    st = sb.Style(np.zeros((sh, sw, 3), np.uint8), g, channels=channels)
    raw = st.tree.cpu().numpy()
    levels = 1
    while 8 ** levels < n:
        levels += 1
    entries, m, texel, chans = (int(v) for v in raw[:16].view(np.uint32))

    values, first = np.unique(g.reshape(n, -1)[:, :channels], axis=0, return_index=True)
    assert m == len(values), "one texel per distinct value"
    assert (entries, texel, chans) == (_start(levels) + m, t, channels)

    padded = (n + 7) // 8 * 8
    at_vals = 256 + _up256(_start(levels - 1) * 16 * t)
    at_keys = at_vals + _up256(padded * t)
    vals = raw[at_vals:at_vals + m * t].view(g.dtype).reshape(m, -1)[:, :channels].astype(np.int64)
    keys = raw[at_keys:at_keys + (_start(levels) + padded) * 4].view(np.uint32)
    boxes = raw[256:256 + _start(levels - 1) * 16 * t].view(g.dtype)
    boxes = boxes.reshape(-1, 2, 8, g.shape[2])[..., :channels].astype(np.int64)

    leaf = keys[_start(levels):]
    assert np.all(leaf[m:] == 0xFFFFFFFF)
    raster = (leaf[:m] >> 16).astype(np.int64) * sw + (leaf[:m] & 0xFFFF)
    np.testing.assert_array_equal(np.sort(raster), np.sort(first))  # the first of its value
    np.testing.assert_array_equal(vals, g.reshape(n, -1)[raster, :channels])
    for level in range(levels - 1, 0, -1):
        per = 8 ** (levels - level)
        for p in range((m + per - 1) // per):
            below = slice(p * per, min((p + 1) * per, m))
            e = _start(level) + p
            assert keys[e] == leaf[below].min()
            box = boxes[(e - 1) >> 3, :, (e - 1) & 7]
            np.testing.assert_array_equal(box[0], vals[below].min(0))
            np.testing.assert_array_equal(box[1], vals[below].max(0))

    # and the lookups, on values the guide holds and beside them
    top = (1 << depth) - 1
    q = g.reshape(n, -1)[rng.integers(0, n, 600)].astype(np.int64)
    q[::2] = np.clip(q[::2] + rng.integers(-4, 5, q[::2].shape), 0, top)
    q = np.ascontiguousarray(q.astype(g.dtype))
    import torch

    qt = torch.from_numpy(q.view(np.int16) if depth == 16 else q).cuda()
    got = st.query(qt).cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, oracle.nn_query_n(g, channels, q))


def _leaves(vals, depth):
    """The order that median splits leave the texels in: every run of 2^k texels
    sorted along its widest element, texels at one value of it by the next widest
    (its upper four bits of a 16-bit one's range), then by their index."""
    at = np.arange(len(vals))
    for lg in range(11, 3, -1):
        for first in range(0, len(at), 1 << lg):
            run = at[first:first + (1 << lg)]
            ext = vals[run].max(0) - vals[run].min(0)
            axis = int(ext.argmax())
            ext[axis] = -1
            near = int(ext.argmax())
            low = vals[run, near].min()
            shift = 0 if depth == 8 else max(int(vals[run, near].max() - low).bit_length() - 4, 0)
            at[first:first + (1 << lg)] = run[np.lexsort((run, (vals[run, near] - low) >> shift,
                                                          vals[run, axis]))]
    return at


# few values of every element, so that medians fall among texels they cannot tell
# apart: without a second element these are split at random, and boxes overlap
@pytest.mark.parametrize("depth,channels,steps", [(8, 3, 9), (8, 5, 3), (16, 4, 5), (16, 2, 30)])
def test_equal_values_of_an_axis(sb, depth, channels, steps):
    rng = np.random.default_rng(depth * 100 + channels)
    elems = oracle.texel_bytes(depth, channels) * 8 // depth
    values = np.stack(np.meshgrid(*[np.arange(steps)] * channels), -1).reshape(-1, channels)
    values = values[rng.permutation(len(values))[:1000]] * (((1 << depth) - 1) // steps)
    values[:, 1:] = values[:, 1:] * 3 // 4  # one element is the widest
    n = len(values)
    g = np.zeros((1, n, elems), np.uint8 if depth == 8 else np.uint16)
    g[0, :, :channels] = values
    print(f"[gpu-case] tree order {depth}x{channels} {n}", flush=True)
    st = sb.Style(np.zeros((1, n, 3), np.uint8), g, channels=channels)
    levels = 1
    while 8 ** levels < n:
        levels += 1
    t = elems * depth // 8
    at_keys = 256 + _up256(_start(levels - 1) * 16 * t) + _up256((n + 7) // 8 * 8 * t)
    keys = st.tree.cpu().numpy()[at_keys:at_keys + (_start(levels) + n) * 4].view(np.uint32)
    np.testing.assert_array_equal(keys[_start(levels):], _leaves(values.astype(np.int64), depth))


@pytest.mark.parametrize("depth,channels", [(16, 8), (16, 5), (8, 8)])
def test_values_of_the_guide(sb, depth, channels):
    """Lookups of every value of a guide of noise, those that a median put beside
    equal ones among them: each its own texel."""
    import torch

    rng = np.random.default_rng(depth + channels)
    size, top = 150, (1 << depth) - 1
    elems = oracle.texel_bytes(depth, channels) * 8 // depth
    g = rng.integers(0, top + 1, (size, size, elems)).astype(np.uint8 if depth == 8 else np.uint16)
    print(f"[gpu-case] values of the guide {depth}x{channels}", flush=True)
    st = sb.Style(np.zeros((size, size, 3), np.uint8), g, channels=channels)
    order = rng.permutation(size * size)
    q = np.ascontiguousarray(g.reshape(-1, elems)[order])
    values, first, back = np.unique(q[:, :channels], axis=0, return_index=True, return_inverse=True)
    least = np.full(len(values), size * size)
    np.minimum.at(least, back.ravel(), order)
    want = least[back.ravel()]
    want = (want // size << 16 | want % size).astype(np.uint32)
    t = torch.from_numpy(q.view(np.int16) if depth == 16 else q).cuda()
    np.testing.assert_array_equal(st.query(t).cpu().numpy().view(np.uint32), want)
    t = torch.cat([t] * 4)  # more than 65536: four lanes a lookup
    np.testing.assert_array_equal(st.query(t).cpu().numpy().view(np.uint32), np.tile(want, 4))


def test_cost_of_exact_lookups(sb):
    """The values of a guide of eight channels of noise cost little more than those
    of a guide of four (7 times when searches bounded by a far texel went on)."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def ms(channels):
        v = torch.randint(0, 65536, (200, 200, channels), generator=gen, device="cuda")
        g = v.to(torch.int16).contiguous()
        st = sb.Style(torch.zeros(200, 200, 3, dtype=torch.uint8, device="cuda"), g, channels=channels)
        q = torch.cat([g.reshape(-1, channels)] * 3)
        best = float("inf")
        for _ in range(7):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            for _ in range(5):
                st.query(q)
            t[1].record()
            t[1].synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
        return best

    print("[gpu-case] cost of exact lookups", flush=True)
    assert ms(8) < 4 * ms(4)


def _places(words):
    """The first place that equal texels of two words meet at."""
    h = np.zeros(len(words), np.uint32)
    for w in words.T:
        h = (h ^ w) * np.uint32(0x9E3779B1)
        h ^= h >> np.uint32(15)
    h *= np.uint32(0x9E3779B1)
    h ^= h >> np.uint32(16)
    return (h >> np.uint32(16)) % 1024


def test_cost_of_values_of_one_place(sb):
    """Two values that meet at one place register in the time of two that do not."""
    import torch

    values = np.random.default_rng(8).integers(0, 65536, (200, 4)).astype(np.uint16)
    place = _places(values.view(np.uint32))
    same = np.argwhere((place[:, None] == place) & (np.arange(200)[:, None] < np.arange(200)))
    assert len(same) and place[0] != place[1]
    pick = torch.randint(0, 2, (512, 512), generator=torch.Generator().manual_seed(8)).cuda()
    rgb = torch.zeros(512, 512, 3, dtype=torch.uint8, device="cuda")

    def ms(two):
        g = torch.from_numpy(values[two].astype(np.int32)).cuda()[pick].to(torch.int16).contiguous()
        best = float("inf")
        for _ in range(7):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            st = sb.Style(rgb, g, channels=4)
            t[1].record()
            t[1].synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
            del st
        return best

    print("[gpu-case] cost of values of one place", flush=True)
    apart, together = ms([0, 1]), ms(list(same[0]))
    print(f"{apart * 1e3:.0f} us, {together * 1e3:.0f} us of one place")
    assert together < 2 * apart
