"""Timed cases: the calls a program makes of this library, over the sizes it makes them at.

A case is one of four kinds of work:

* ``frame``: one frame through a prepared call (``FramePlan``) or, with labels,
  ``stylize``: what an interactive renderer does for every image;
* ``anim``: one step of an animation: the frame's jitter table drawn on the
  device, the frame stylised with its source coordinates, and the change
  counts against the previous frame;
* ``batch``: many frames of uneven size and mixed guidance in one call
  (a captured graph, direct launches, or frame by frame);
* ``register``: a style made resident (padded exemplar and the exact lookup
  table or search tree), for a search style with the lookups of a set of
  guide values.

The guide kinds are the library's: ``normal`` (two 8-bit channels, sphere
exemplar, bump-mapped target), ``uv`` (two 16-bit channels, texture
coordinates), ``appearance`` (three 8-bit channels), ``features8`` (five 8-bit
channels, searched) and ``features16`` (four 16-bit channels, searched).
Sizes and parameters are those of the workloads and tests of this repository;
the inputs follow the same recipes, made on the device with torch.

Every output is an integer the method defines exactly (bytes, coordinates,
chunk codes, counts), so nothing here is rounded and ``exact`` has no 64-bit
value to add: a result is right only if it is equal.
"""
import math
import random

import torch

import paper_1807_03249_amd as sb

DEV = "cuda"
KINDS = ("normal", "uv", "appearance", "features8", "features16")
GUIDE_BYTES = {"normal": 2, "uv": 4, "appearance": 4, "features8": 8, "features16": 8}
# levels, finest spacing, threshold and radius of each kind's workload
PARAMS = {"normal": (4, 8, 32, 3), "uv": (5, 8, 4096, 3), "appearance": (4, 8, 192, 3),
          "features8": (4, 8, 160, 3), "features16": (4, 8, 1 << 22, 3)}


def _frame_case(guide, w, h, style, **kw):
    levels, finest, threshold, radius = PARAMS[guide]
    c = {"kind": "frame", "guide": guide, "w": w, "h": h, "style": style, "lut_bits": 0,
         "levels": levels, "finest": finest, "threshold": threshold, "radius": radius, "labels": 0}
    if guide in ("normal", "appearance"):
        c["lut_bits"] = 8
    elif guide == "uv":
        c["lut_bits"] = max(4, int(math.log2(style)))
    c.update(kw)
    return c


def _register_case(guide, style, lut_bits, labels=0, queries=0):
    return {"kind": "register", "guide": guide, "style": style, "lut_bits": lut_bits,
            "labels": labels, "queries": queries}


def listed():
    return [
        # the smallest call: a 256 x 256 preview frame, where launches count
        dict(_frame_case("normal", 256, 256, 256, levels=3, threshold=48, radius=2),
             name="frame_normal_256"),
        # the ordinary frame: a normal-guided full-HD render
        dict(_frame_case("normal", 1920, 1080, 512), name="frame_normal_1080p"),
        # the largest frame: 4K with 16-bit texture coordinates and a 2048 x 2048 exemplar
        dict(_frame_case("uv", 3840, 2160, 2048), name="frame_uv_4k"),
        # normals plus an appearance channel (the 2^24-bin table)
        dict(_frame_case("appearance", 1920, 1080, 512), name="frame_appearance_1080p"),
        # the segmentation guide: six labels as a hard constraint
        dict(_frame_case("normal", 1920, 1080, 512, labels=6), name="frame_labels_1080p"),
        # guides of many channels, looked up by exact search: normals, appearance and chroma
        dict(_frame_case("features8", 1920, 1080, 512), name="frame_features8_1080p"),
        # ... and texture coordinates with normals at 16 bits
        dict(_frame_case("features16", 1920, 1080, 512), name="frame_features16_1080p"),
        # one step of a 480p animation, odd-sized: fresh table, coordinates, change counts
        dict(_frame_case("normal", 853, 481, 512, kind="anim"), name="anim_853x481"),
        # offline or serving batches: 64 frames of uneven size, half normal- and half UV-guided
        {"name": "batch_64", "kind": "batch", "frames": 64, "api": "graph", "style": 512,
         "mix": 401},
        # registering a style when a user picks an exemplar: 8-bit normals
        dict(_register_case("normal", 512, 8), name="register_normal_512"),
        # ... a large texture with 16-bit coordinates
        dict(_register_case("uv", 2048, 11), name="register_uv_2048"),
        # ... and a many-channel style, with the lookups of a small image's guide values
        dict(_register_case("features8", 512, 0, queries=65536), name="register_features8_512"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("frame", "frame", "frame", "frame", "anim", "batch", "register"))
    if kind == "batch":
        return {"kind": "batch", "frames": _log_int(rng, 2, 64),
                "api": rng.choice(("graph", "direct", "frames")), "style": rng.choice((256, 512)),
                "mix": rng.randint(0, 1 << 30)}
    guide = rng.choice(KINDS)
    if kind == "register":
        search = guide.startswith("features")
        style = _log_int(rng, 64, 512 if search or guide == "appearance" else 2048)
        bits = (0 if search else rng.randint(5, 8) if guide == "appearance"
                else rng.randint(6, 8) if guide == "normal" else rng.randint(6, 11))
        labels = rng.choice((0, 0, 4)) if guide == "normal" else 0
        return _register_case(guide, style, bits, labels, _log_int(rng, 1, 65536) if search else 0)
    if kind == "anim":
        guide = rng.choice(("normal", "uv", "appearance"))
    w, h = _log_int(rng, 64, 1920), _log_int(rng, 64, 1080)
    if kind == "frame" and guide in ("normal", "uv", "appearance") and rng.random() < 0.25:
        w, h = rng.randint(1920, 3840), rng.randint(1080, 2160)
    c = _frame_case(guide, w, h, rng.randint(128, 512), kind=kind)
    if guide == "uv":
        c["lut_bits"] = rng.randint(7, 11)
    c["levels"] = rng.choice((1, 2, 3, 4, 4, 5))
    c["finest"] = rng.choice((4, 8, 8, 8, 16))
    c["threshold"] = int(c["threshold"] * rng.choice((0.25, 1, 1, 4)))
    c["radius"] = rng.choice((0, 1, 2, 3, 3, 4, 5, 7))
    if kind == "frame" and guide == "normal":
        c["labels"] = rng.choice((0, 0, 0, 2, 6))
    return c


# ---------------------------------------------------------------- inputs


def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, device=DEV)


def _noise(gen, n, w, h, period):
    """n smoothstep-interpolated lattice noise images (n, h, w) in [0, 1)."""
    lat = _rand(gen, n, math.ceil(h / period) + 2, math.ceil(w / period) + 2)

    def axis(m):
        g = (torch.arange(m, device=DEV) + 0.5) / period
        i = g.floor().long()
        f = g - i
        return i, f * f * (3 - 2 * f)

    ix, fx = axis(w)
    iy, fy = axis(h)
    rows = lat[:, :, ix] * (1 - fx) + lat[:, :, ix + 1] * fx
    return rows[:, iy] * (1 - fy[:, None]) + rows[:, iy + 1] * fy[:, None]


def _texture(gen, w, h):
    """Stochastic RGB texture: three octaves per channel, rescaled to bytes."""
    v = sum(a * _noise(gen, 3, w, h, p) for p, a in ((16, 1.0), (8, 0.5), (4, 0.25)))
    lo, hi = v.amin((1, 2), True), v.amax((1, 2), True)
    return (255 * (v - lo) / (hi - lo) + 0.5).byte().permute(1, 2, 0).contiguous()


def _encode(nx, ny):
    return torch.stack([(nx + 1) * 127.5 + 0.5, (ny + 1) * 127.5 + 0.5], -1).clamp(0, 255).byte()


def _sphere(size):
    x = (torch.arange(size, device=DEV) + 0.5 - size / 2) / (size / 2)
    dx, dy = x[None, :].expand(size, size), x[:, None].expand(size, size)
    r = (dx * dx + dy * dy).sqrt().clamp_min(1.0)
    return _encode(dx / r, dy / r)


def _bumps(gen, w, h, n):
    """Normals of a heightfield of n Gaussian bumps, signed."""
    m = min(w, h)
    cx, cy = _rand(gen, n) * w, _rand(gen, n) * h
    sig = (0.03 + 0.09 * _rand(gen, n)) * m
    amp = (0.5 + _rand(gen, n)) * sig * torch.where(_rand(gen, n) < 0.5, -1.0, 1.0)
    x = torch.arange(w, device=DEV) + 0.5
    y = torch.arange(h, device=DEV) + 0.5
    gx = torch.zeros(h, w, device=DEV)
    gy = torch.zeros(h, w, device=DEV)
    for k in range(n):
        ex = torch.exp(-(x - cx[k]) ** 2 / (2 * sig[k] ** 2))
        ey = amp[k] * torch.exp(-(y - cy[k]) ** 2 / (2 * sig[k] ** 2))
        gx += ey[:, None] * (ex * (cx[k] - x) / sig[k] ** 2)
        gy += (ey * (cy[k] - y) / sig[k] ** 2)[:, None] * ex
    norm = (gx * gx + gy * gy + 1).sqrt()
    return _encode(-gx / norm, -gy / norm)


def _u16(t):
    return t.clamp(0, 65535).to(torch.int32).to(torch.int16)


def _identity_uv(size):
    c = (torch.arange(size, device=DEV) + 0.5) * 65536 / size
    return torch.stack(torch.meshgrid(c, c, indexing="xy"), -1).floor()


def _warped_uv(gen, w, h, size):
    """Texture coordinates at texel scale, tiled and warped by smooth noise."""
    d = (2 * _noise(gen, 2, w, h, 256) - 1) * 12
    x = torch.arange(w, device=DEV)[None, :] + d[0] + 0.5
    y = torch.arange(h, device=DEV)[:, None] + d[1] + 0.5
    return torch.stack([torch.remainder(x, size), torch.remainder(y, size)], -1) * 65536 / size


def _blur(v):
    p = torch.nn.functional.pad(v[None, None], (4, 4, 4, 4), mode="replicate")
    return torch.nn.functional.avg_pool2d(p, 9, 1)[0, 0].add(0.5).clamp(0, 255).byte()


def _colours(rgb):
    """Blurred luma and two opponent-colour channels of an image."""
    r, g, b = rgb.float().unbind(-1)
    return [_blur((77 * r + 150 * g + 29 * b) / 256), _blur((r - g + 255) / 2),
            _blur((r + g - 2 * b + 510) / 4)]


def _texels(chans, elements):
    out = torch.zeros(*chans[0].shape, elements, dtype=chans[0].dtype, device=DEV)
    for k, c in enumerate(chans):
        out[..., k] = c
    return out


def _widen(n):
    return [_u16(n[..., k].int() * 257) for k in range(2)]


def _source(gen, guide, size):
    """(rgb, guide) of an exemplar of size x size."""
    rgb = _texture(gen, size, size)
    if guide == "normal":
        return rgb, _sphere(size)
    if guide == "uv":
        return rgb, _u16(_identity_uv(size))
    n = _sphere(size)
    if guide == "appearance":
        return rgb, _texels([n[..., 0], n[..., 1], _colours(rgb)[0]], 4)
    if guide == "features8":
        return rgb, _texels([n[..., 0], n[..., 1]] + _colours(rgb), 8)
    uv = _u16(_identity_uv(size))
    return rgb, _texels([uv[..., 0], uv[..., 1]] + _widen(n), 4)


def _target(gen, guide, w, h, size, rgb, bumps):
    if guide == "normal":
        return _bumps(gen, w, h, bumps)
    if guide == "uv":
        return _u16(_warped_uv(gen, w, h, size))
    n = _bumps(gen, w, h, bumps)
    if guide == "appearance":
        return _texels([n[..., 0], n[..., 1], _colours(_texture(gen, w, h))[0]], 4)
    # an object textured with the exemplar: its normals there plus bump detail
    uv = _warped_uv(gen, w, h, size)
    at = (uv * size / 65536).long().clamp(0, size - 1)
    n = (_sphere(size)[at[..., 1], at[..., 0]].int() + (n.int() - 128) // 8).clamp(0, 255).byte()
    if guide == "features8":
        return _texels([n[..., 0], n[..., 1]] + _colours(rgb[at[..., 1], at[..., 0]]), 8)
    uv = _u16(uv)
    return _texels([uv[..., 0], uv[..., 1]] + _widen(n), 4)


def _labels(gen, w, h, nlabels, sites):
    """Voronoi regions: every pixel labelled by its nearest site."""
    sx, sy = _rand(gen, sites) * w, _rand(gen, sites) * h
    x = torch.arange(w, device=DEV)[None, :]
    y = torch.arange(h, device=DEV)[:, None]
    best = torch.full((h, w), 1e12, device=DEV)
    lab = torch.zeros(h, w, dtype=torch.uint8, device=DEV)
    for k in range(sites):
        d = (x - sx[k]) ** 2 + (y - sy[k]) ** 2
        lab[d < best] = k % nlabels
        best = torch.minimum(best, d)
    return lab


def _channels(guide):
    return {"features8": 5, "features16": 4}.get(guide)


def _register(s):
    """The registration call of a program that has an exemplar on the device."""
    return sb.Style(s["rgb"], s["guide"], s["lut_bits"], labels=s["labels"],
                    nlabels=s["nlabels"], channels=s["channels"])


def _style_inputs(gen, guide, size, lut_bits, labels):
    rgb, g = _source(gen, guide, size)
    lab = _labels(gen, size, size, labels, 40) if labels else None
    return {"rgb": rgb, "guide": g, "lut_bits": lut_bits, "labels": lab,
            "nlabels": labels or None, "channels": _channels(guide)}


def _batch_sides(case):
    rng = random.Random(case["mix"])
    return [(rng.randint(320, 1920), rng.randint(240, 1080)) for _ in range(case["frames"])]


def _batch_jobs(gen, case, seed):
    """Half normal-, half UV-guided frames of 320..1920 x 240..1080 on four
    styles, their outputs one after another in two buffers."""
    n, size = case["frames"], case["style"]
    styles = [_register(_style_inputs(gen, g, size, 8, 0)) for g in ("normal", "normal", "uv", "uv")]
    sides = _batch_sides(case)
    total = sum(w * h for w, h in sides)
    rgb = torch.empty(total, 3, dtype=torch.uint8, device=DEV)
    chunk = torch.empty(total, dtype=torch.int32, device=DEV)
    jobs, at = [], 0
    for i, (w, h) in enumerate(sides):
        guide = "normal" if i < (n + 1) // 2 else "uv"
        style = styles[(0 if guide == "normal" else 2) + i % 2]
        levels, finest, threshold, radius = PARAMS[guide]
        p = sb.params(levels, finest, threshold, radius, seed=seed + i)
        jobs.append(sb.FrameJob(style, _target(gen, guide, w, h, size, None, 16), None, p,
                                rgb[at:at + w * h], chunk[at:at + w * h]))
        at += w * h
    return jobs, rgb, chunk


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    s = {"case": case, "seed": seed}
    if case["kind"] == "batch":
        s["jobs"], s["rgb"], s["chunk"] = _batch_jobs(gen, case, seed)
        if case["api"] == "frames":
            n = max(sb.workspace_bytes(j.w, j.h, j.params) for j in s["jobs"])
        else:
            s["plan"] = sb.Batch(use_graph=case["api"] == "graph")
            n = s["plan"].workspace_bytes(s["jobs"])
        s["workspace"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        return s
    guide, size = case["guide"], case["style"]
    inputs = _style_inputs(gen, guide, size, case["lut_bits"], case["labels"])
    if case["kind"] == "register":
        s["inputs"] = inputs
        if case["queries"]:
            side = max(1, math.ceil(math.sqrt(case["queries"])))
            t = _target(gen, guide, side, side, size, inputs["rgb"], 8)
            s["texels"] = t.reshape(-1, t.shape[-1])[:case["queries"]].contiguous()
        return s
    w, h = case["w"], case["h"]
    s["style"] = _register(inputs)
    s["target"] = _target(gen, guide, w, h, size, inputs["rgb"],
                          8 if w * h < 300000 else 64).contiguous()
    s["rgb"] = torch.empty(h, w, 3, dtype=torch.uint8, device=DEV)
    s["chunk"] = torch.empty(h, w, dtype=torch.int32, device=DEV)
    p = sb.params(case["levels"], case["finest"], case["threshold"], case["radius"],
                  seed=None if case["kind"] == "anim" else seed)
    s["params"] = p
    s["workspace"] = torch.empty(sb.workspace_bytes(w, h, p), dtype=torch.uint8, device=DEV)
    if case["kind"] == "anim":
        s["table"] = sb.jitter_fill(w, h, case["levels"], case["finest"], seed, 0)
        _, chunk, nnf = sb.stylize(s["style"], s["target"], s["table"], p, want_nnf=True)
        s["previous"] = (chunk, nnf)
    elif case["labels"]:
        s["map"] = _labels(gen, w, h, case["labels"], 60)
    else:
        s["plan"] = sb.FramePlan(s["style"], s["target"], None, p, s["rgb"], s["chunk"],
                                 s["workspace"])
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        jobs = state["jobs"]
        if case["api"] == "frames":
            sb.stylize_frames(jobs, state["workspace"])
        else:
            state["plan"].run(jobs, state["workspace"])
        return state["rgb"], state["chunk"]
    if case["kind"] == "register":
        style = _register(state["inputs"])
        if case["queries"]:
            return style.rgba, style.query(state["texels"])
        return style.rgba, style.lut if style.label_luts is None else (style.lut, style.label_luts)
    if case["kind"] == "anim":
        sb.jitter_fill(case["w"], case["h"], case["levels"], case["finest"], state["seed"], 1,
                       out=state["table"])
        rgb, chunk, nnf = sb.stylize(state["style"], state["target"], state["table"],
                                     state["params"], state["rgb"], state["chunk"], want_nnf=True,
                                     workspace=state["workspace"])
        changed = sb.frame_change(state["previous"][0], chunk, state["previous"][1], nnf)
        return rgb, chunk, nnf, changed
    if case["labels"]:
        return sb.stylize(state["style"], state["target"], None, state["params"], state["rgb"],
                          state["chunk"], workspace=state["workspace"], tgt_labels=state["map"])
    state["plan"].launch()
    return state["rgb"], state["chunk"]


def _frame_bytes(guide, w, h, size):
    """Guide in, RGB and chunk map out, the exemplar (RGB and guide) once."""
    g = GUIDE_BYTES[guide]
    return w * h * (g + 7) + size * size * (3 + g)


def work(case):
    """Integer work throughout: the operations a pass cannot do without are
    one guide error per pixel and one sum per channel and texel voted (at
    least the pixel's own); a registration looks at every texel and bin once."""
    if case["kind"] == "batch":
        px = sum(w * h for w, h in _batch_sides(case))
        return {"bytes": px * 10 + 4 * case["style"] ** 2 * 6, "flops": px * 9}
    guide, size = case["guide"], case["style"]
    if case["kind"] == "register":
        chans = {"normal": 2, "uv": 2, "appearance": 3}.get(guide, 0)
        table = 4 * (case["labels"] + 1) * (1 << (chans * case["lut_bits"])) if chans else 0
        q = case["queries"] * (GUIDE_BYTES[guide] + 4)
        return {"bytes": size * size * (3 + GUIDE_BYTES[guide] + 4) + table + q,
                "flops": size * size + table // 4}
    w, h = case["w"], case["h"]
    b = _frame_bytes(guide, w, h, size) + (w * h + size * size if case["labels"] else 0)
    if case["kind"] == "anim":  # coordinates out, two pairs of maps compared
        b += w * h * (4 + 16)
    return {"bytes": b, "flops": w * h * 9}


def exact(case, seed):
    return None
