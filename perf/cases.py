"""Performance cases of the spatial model checker: what its users have it do,
through the public entry points of the Python binding.

A case names a kind of work and its sizes; `prepare` makes what a program
holds before the call (context, resident images, compiled formulas, output
buffers), `run` is one pass.  All outputs are bit masks or integer labels, so
they are compared exactly.

Kinds
  check    check_all of one formula on one resident image
  stream   load_image of a new image from device memory, then check_all
  batch    check_batch of one formula on many images of uneven sizes
  volume   check_all on a volume
  labels   ccl_labels (2-D) or ccl_labels3 (depth > 1) of a packed mask
  pj       ccl_labels_pj, the paper's own labelling algorithm
  serve    a burst of requests through the serving loop
"""
import math
import random

import numpy as np
import torch

import paper_2010_07284_amd as vlg

DEV = "cuda:0"
TYPES = {"f32": torch.float32, "u8": torch.uint8, "u16": torch.uint16}
BYTES = {"f32": 4, "u8": 1, "u16": 2}


# ------------------------------------------------------------------ formulas
# Texts in the tool's language; image values lie in [0, 1] (f32), 0..255 (u8)
# or 0..65535 (u16), thresholds are scaled to the type.

PLAIN = """
let A  = intensity(img) >. {0.65}
let B  = intensity(img) >. {0.35}
let C  = intensity(img) <. {0.45}
let D  = B & !A
let E  = D | C
let G  = near(E)
let R1 = reach(A, B)
let R2 = reach(C, !A)
output "G" G
output "R2" R2
output "O" R1 | surrounded(near(A), B)
"""

# the paper's segmentation: grow from a high threshold into a low one
GROW = """
let hI = intensity(img) >. {0.95}
let vI = intensity(img) >. {0.86}
output "segmentation" grow(hI, vI)
"""

# arithmetic atoms over two channels, touch and grow on them
ARITH = """
let A = (intensity(img, 0) + intensity(img, 1)) * 0.5 >. {0.55}
let B = intensity(img, 0) - intensity(img, 1) <. -{0.2}
let C = abs(intensity(img, 1) - {0.5}) * 2 <=. {0.35}
let D = intensity(img, 0) / (intensity(img, 1) + {0.25}) >=. 1
let E = min(intensity(img, 0), intensity(img, 1)) >. max({0.2}, percentile(img, 1, 0.4) - {0.1})
let F = intensity(img, 0) >. percentile(img, 0, 0.6)
output "a" A
output "b" B & !C
output "d" D | E
output "touch" touch(A, C)
output "touch2" touch(!B, F & D)
output "mix" grow(E, A | B) & near(touch(C, D))
output "neg" -intensity(img, 1) <. -{0.4}
"""

# percentile thresholds on four channels, a region grown on each, and their
# combinations
SEGMENT = """
let h0 = intensity(img, 0) >. percentile(img, 0, 0.95)
let l0 = intensity(img, 0) >. percentile(img, 0, 0.86)
let h1 = intensity(img, 1) >. percentile(img, 1, 0.95)
let l1 = intensity(img, 1) >. percentile(img, 1, 0.86)
let h2 = intensity(img, 2) >. percentile(img, 2, 0.95)
let l2 = intensity(img, 2) >. percentile(img, 2, 0.86)
let h3 = intensity(img, 3) >. percentile(img, 3, 0.95)
let l3 = intensity(img, 3) >. percentile(img, 3, 0.86)
let d0 = intensity(img, 0) <. percentile(img, 0, 0.3)
let d1 = intensity(img, 1) <. percentile(img, 1, 0.3)
let m2 = intensity(img, 2) >. percentile(img, 2, 0.5)
let m3 = intensity(img, 3) >. percentile(img, 3, 0.7)
let g0 = grow(h0, l0)
let g1 = grow(h1, l1)
let g2 = grow(h2, l2)
let g3 = grow(h3, l3)
let core = (g0 | g1) & !d0
let rim = near(core) & !interior(core)
let back = reach(d0, d1 | !m2)
let hole = surrounded(!core, rim | g2)
let mix = (near(g2) & m3) | interior(l1 | l3)
let tail = touch(mix, core)
output "core" core
output "rim" rim
output "back" back & !g3
output "hole" hole
output "tail" tail | (near(near(g3)) & !back)
output "all" grow(core, mix | tail)
"""

# a segmentation on volumes: percentiles, arithmetic, N and every
# reach-type operator
VOLUME = """
let A = intensity(img, 0) >. percentile(img, 0, 0.95)
let B = intensity(img, 0) >. percentile(img, 0, 0.86)
let C = intensity(img, 1) >. {0.5}
let M = (intensity(img, 0) + intensity(img, 1)) * 0.5 >. {0.45}
let core = grow(A, B)
output "core" core
output "edema" grow(core, B | (C & M)) & !core
output "shell" near(core) & !interior(core)
output "enclosed" surrounded(C, near(core))
output "contact" touch(C, core)
output "reach" reach(A, M)
"""

# one atom, one N, one connective: the streaming operators alone
PIXELWISE = """
let A = intensity(img) >. {0.7}
let N1 = near(A)
output "atom" A
output "ring" N1 & !A
"""


def random_text(seed, nodes, reach):
    """About `nodes` operators over one channel, `reach` of them reach-type,
    each reading nodes made shortly before; up to 8 outputs."""
    rng = random.Random(seed)
    lines, recent, outs = [], [], []

    def add(e):
        recent.append("n%d" % len(lines))
        lines.append("let %s = %s" % (recent[-1], e))
        return recent[-1]

    def atom():
        return add("intensity(img) %s {%.4f}" % (rng.choice((">.", "<.", ">=.", "<=.")), rng.uniform(0.1, 0.9)))

    for _ in range(3):
        atom()
    every = max(2, nodes // (reach + 1)) if reach else nodes + 1
    while len(lines) < nodes:
        a, b = rng.sample(recent[-min(len(recent), 12):], 2)
        if reach and len(lines) % every == every - 1:
            outs.append(add("%s(%s, %s)" % (rng.choice(("reach", "surrounded", "grow")), a, b)))
        elif rng.random() < 0.15:
            atom()
        else:
            add(rng.choice(("%s & %s" % (a, b), "%s | %s" % (a, b), "%s & !%s" % (a, b), "near(%s)" % a,
                            "interior(%s)" % a, "!%s" % a, "near(%s) | %s" % (a, b))))
    outs = sorted(set(outs[-7:] + [recent[-1]]))
    return "\n".join(lines + ['output "%s" %s' % (o, o) for o in outs])


def chain_text(seed, steps, reach):
    """A long sequence N, &, !, N, ... over a 0/1 mask with `reach` reach
    elements spread over it: the paper's sequential formulas."""
    rng = random.Random(seed)
    lines, partners = ["let x0 = intensity(img) >. 0"], [0]
    every = max(1, steps // max(1, reach))
    rot = outs = 0
    for i in range(1, steps + reach + 1):
        near_by = [j for j in partners[-40:] if j <= i - 2] or [0]
        if i % (every + 1) == 0:
            lines.append("let x%d = reach(x%d, x%d)" % (i, i - 1, rng.choice(near_by)))
            rot = 1
            continue
        e = ("near(x%d)" % (i - 1), "x%d & x%d" % (i - 1, rng.choice(near_by)), "!x%d" % (i - 1))[rot % 3]
        if rot % 3:
            partners.append(i)
        rot += 1
        lines.append("let x%d = %s" % (i, e))
    n = len(lines)
    outs = sorted({n - 1} | set(range(n // 6, n, max(1, n // 6))))[-8:]
    return "\n".join(lines + ['output "x%d" x%d' % (k, k) for k in outs])


def windows_text(seed):
    """Intensity windows of single ellipses on channel 0 of the ellipse and
    maze image, a corridor search on channels 1 and 2, and regions grown,
    reached and surrounded from them."""
    rng = random.Random(seed)
    lines = ["let maze = intensity(img, 1) >. 0.5", "let seed = intensity(img, 2) >. 0.5",
             "let walk = reach(seed, maze)", "let corridor = grow(seed, maze)"]
    for k in range(8):
        v = 0.5 + 0.5 * (rng.randrange(100) + 1) / 100
        lines.append("let w%d = (intensity(img) >. %.4f) & (intensity(img) <. %.4f)" % (k, v - 0.0025, v + 0.0025))
    for k, t in enumerate((0.12, 0.25, 0.4)):
        lines.append("let t%d = intensity(img) <. %.2f" % (k, t))
    lines.append("let e = intensity(img) >. 0.5")
    lines += ["let u%d = near(near(w%d)) | interior(w%d)" % (k, k, (k + 1) % 8) for k in range(8)]
    lines += ["let g0 = grow(w0 | w1, e)", "let g1 = grow(t0, t1)", "let r0 = reach(w2 | w3, e | t0)",
              "let r1 = reach(u4, t2 & !u5)", "let s0 = surrounded(t0 | u6, !t1)", "let s1 = surrounded(u7, e)",
              "let g2 = grow(g0 & near(u0), t2 | u1)", "let r2 = reach(interior(g1), !s0 & !e)"]
    lines += ['output "o%d" %s' % (k, e) for k, e in enumerate(
        ("walk", "corridor", "g0 & !u2", "g1 | u3", "r0 & near(r1)", "r1", "s0 | s1", "g2", "r2 & !near(g0)",
         "interior(near(u0 | u1 | u2))"))]
    return "\n".join(lines)


def formula_text(case):
    name, t = case["formula"], case["dtype"]
    texts = {"plain": PLAIN, "grow": GROW, "arith": ARITH, "segment": SEGMENT, "volume": VOLUME,
             "pixelwise": PIXELWISE}
    if name == "random":
        text = random_text(case["text_seed"], case["nodes"], case["reach"])
    elif name == "chain":
        text = chain_text(case["text_seed"], case["nodes"], case["reach"])
    elif name == "windows":
        text = windows_text(case["text_seed"])
    else:
        text = texts[name]
    top = {"f32": 1.0, "u8": 255.0, "u16": 65535.0}[t]
    parts = text.split("{")  # {x}: the fraction x of the type's range
    return parts[0] + "".join("%.6g%s" % (float(p.split("}", 1)[0]) * top, p.split("}", 1)[1]) for p in parts[1:])


def formula_channels(name):
    return {"arith": 2, "segment": 4, "volume": 2, "windows": 3}.get(name, 1)


# ------------------------------------------------------------------ images

def smooth(gen, shape, cell):
    """Smooth random fields in [0, 1] (..., H, W): a coarse grid of normals,
    interpolated."""
    h, w = shape[-2:]
    lead = shape[:-2]
    n = int(np.prod(lead)) if lead else 1
    coarse = torch.randn((n, 1, h // cell + 2, w // cell + 2), generator=gen, device=DEV)
    f = torch.nn.functional.interpolate(coarse, size=(h, w), mode="bicubic", align_corners=False)
    return torch.sigmoid(1.6 * f).reshape(*lead, h, w)


def typed(t, dtype):
    if dtype == "f32":
        return t.contiguous()
    if dtype == "u8":
        return (t * 255.0).round_().clamp_(0, 255).to(torch.uint8)
    return (t * 65535.0).round_().clamp_(0, 65535).to(torch.int32).to(torch.uint16)


def scan_image(gen, channels, h, w, dtype):
    """Smooth regions with Rician-like acquisition noise, as an MRI slice."""
    out = torch.empty((channels, h, w), dtype=TYPES[dtype], device=DEV)
    for c in range(channels):
        t = smooth(gen, (h, w), 24)
        t = torch.sqrt((t + 0.04 * torch.randn((h, w), generator=gen, device=DEV)) ** 2 +
                       (0.04 * torch.randn((h, w), generator=gen, device=DEV)) ** 2).clamp_(0, 1)
        out[c] = typed(t, dtype)
    return out


def noise_image(gen, h, w, dtype):
    """Smoothed noise without acquisition noise."""
    return typed(smooth(gen, (1, h, w), 8), dtype)


def big_image(gen, h, w):
    """A very large channel: a smooth field repeated with per-row offsets."""
    base = smooth(gen, (1024, w), 64)
    out = torch.empty((1, h, w), dtype=torch.float32, device=DEV)
    for y in range(0, h, 1024):
        n = min(1024, h - y)
        torch.add(base[:n], 0.2 * torch.rand((n, 1), generator=gen, device=DEV) - 0.1, out=out[0, y:y + n])
    return out


def ellipse_maze_image(gen, rng, h, w):
    """Channel 0: noise in [0, 0.5] under ellipses of distinct intensities;
    channel 1: a one-pixel serpentine corridor; channel 2: its start."""
    out = torch.zeros((3, h, w), dtype=torch.float32, device=DEV)
    out[0] = 0.5 * smooth(gen, (h, w), 8)
    levels = list(range(100))
    rng.shuffle(levels)
    side = min(h, w)
    for k in levels:
        ry, rx = (side * rng.uniform(0.006, 0.06) for _ in range(2))
        cy, cx, th = rng.uniform(0, h), rng.uniform(0, w), rng.uniform(0, math.pi)
        r = max(ry, rx)
        y0, y1, x0, x1 = max(0, int(cy - r)), min(h, int(cy + r) + 2), max(0, int(cx - r)), min(w, int(cx + r) + 2)
        if y0 >= y1 or x0 >= x1:
            continue
        dy = torch.arange(y0, y1, device=DEV, dtype=torch.float32)[:, None] - cy
        dx = torch.arange(x0, x1, device=DEV, dtype=torch.float32)[None] - cx
        c, s = math.cos(th), math.sin(th)
        inside = ((dx * c + dy * s) / rx) ** 2 + ((dy * c - dx * s) / ry) ** 2 <= 1
        out[0, y0:y1, x0:x1].masked_fill_(inside, 0.5 + 0.5 * (k + 1) / 100)
    out[1, 0::2] = 1
    out[1, 1::4, w - 1] = 1
    out[1, 3::4, 0] = 1
    out[2, 0, 0] = 1
    return out


def make_image(case, gen, rng, h=None, w=None):
    h, w = h or case["h"], w or case["w"]
    kind = case["image"]
    if kind == "maze":
        return ellipse_maze_image(gen, rng, h, w)
    if kind == "coin":
        return (torch.rand((1, h, w), generator=gen, device=DEV) < 0.5).to(torch.uint8)
    if kind == "big":
        return big_image(gen, h, w)
    if kind == "noise":
        return noise_image(gen, h, w, case["dtype"])
    return scan_image(gen, formula_channels(case["formula"]), h, w, case["dtype"])


def pack_bits(m):
    """A boolean [..., W] device tensor as packed int64 words (bit x % 64)."""
    w = m.shape[-1]
    m = torch.nn.functional.pad(m, (0, -w % 64)).reshape(*m.shape[:-1], -1, 64).to(torch.int64)
    weights = torch.ones(64, dtype=torch.int64, device=DEV) << torch.arange(64, device=DEV)
    return (m * weights).sum(-1)


def sides(case):
    """The image sizes of a batch or request stream: part of the case."""
    rng = random.Random(case["size_seed"])
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    pick = (lambda: round(math.exp(rng.uniform(lo, hi)))) if case["kind"] == "serve" else \
        (lambda: rng.randint(case["lo"], case["hi"]))
    return [(pick(), pick()) for _ in range(case["n"])]


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest call: a small image, launches and latency
        {"name": "plain_256", "kind": "check", "formula": "plain", "image": "noise", "dtype": "f32", "h": 256,
         "w": 256, "fmt": "packed"},
        # images arriving one by one, each loaded, segmented and dropped
        {"name": "stream_u16_1000x750", "kind": "stream", "formula": "grow", "image": "scan", "dtype": "u16",
         "h": 750, "w": 1000, "fmt": "u8"},
        # the serving loop: a burst of mixed requests on resident images
        {"name": "serve_burst", "kind": "serve", "formula": "random", "image": "noise", "dtype": "f32", "n": 6,
         "lo": 256, "hi": 3000, "size_seed": 5, "requests": 24, "slots": 4, "text_seed": 5},
        # a long sequential formula on a small image: many small kernels
        {"name": "chain_1024", "kind": "check", "formula": "chain", "image": "coin", "dtype": "u8", "h": 1024,
         "w": 1024, "fmt": "packed", "nodes": 2000, "reach": 100, "text_seed": 3, "fuse_halo": 16},
        # labels of a mask for use outside the checker
        {"name": "labels_2048", "kind": "labels", "depth": 1, "h": 2048, "w": 2048, "cell": 8},
        # the paper's labelling algorithm, reconnect every 8 as in its figure
        {"name": "pj_2048", "kind": "pj", "h": 2048, "w": 2048, "cell": 8, "reconnect": 8},
        # the paper's segmentation on its slice size and pixel type
        {"name": "grow_7680_u16", "kind": "check", "formula": "grow", "image": "scan", "dtype": "u16", "h": 7680,
         "w": 7680, "fmt": "u8"},
        # a large formula on one image, labellings run together
        {"name": "windows_4096", "kind": "check", "formula": "windows", "image": "maze", "dtype": "f32", "h": 4096,
         "w": 4096, "fmt": "packed", "text_seed": 2, "ccl_lanes": 4},
        # arithmetic atoms and percentiles on two channels
        {"name": "arith_4096", "kind": "check", "formula": "arith", "image": "scan", "dtype": "f32", "h": 4096,
         "w": 4096, "fmt": "packed"},
        # a volume
        {"name": "volume_256", "kind": "volume", "formula": "volume", "dtype": "f32", "depth": 256, "h": 256,
         "w": 256, "fmt": "packed"},
        # many images of uneven sizes in one call
        {"name": "batch_128", "kind": "batch", "formula": "segment", "image": "scan", "dtype": "f32", "n": 128,
         "lo": 128, "hi": 2048, "size_seed": 4, "fmt": "packed"},
        # the largest: streaming operators on an image far beyond the caches
        {"name": "pixelwise_32000", "kind": "check", "formula": "pixelwise", "image": "big", "dtype": "f32",
         "h": 32000, "w": 32000, "fmt": "packed"},
    ]


def draw(rng):
    def side(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("check", "check", "check", "check", "stream", "batch", "volume", "labels", "labels3", "pj",
                       "serve"))
    dtype = rng.choice(("f32", "f32", "u8", "u16"))
    fmt = rng.choice(("packed", "packed", "u8"))
    seed = rng.randrange(1 << 20)
    if kind == "check":
        f = rng.choice(("plain", "grow", "arith", "segment", "random", "chain", "windows", "pixelwise"))
        c = {"kind": kind, "formula": f, "dtype": dtype, "fmt": fmt, "h": side(48, 6000), "w": side(48, 6000),
             "image": {"plain": "noise", "random": "noise", "pixelwise": "noise"}.get(f, "scan")}
        if f == "chain":
            c.update(image="coin", dtype="u8", h=side(200, 1500), w=side(200, 1500), nodes=rng.randint(200, 1500),
                     reach=rng.randint(5, 60), text_seed=seed)
            if rng.random() < 0.5:
                c["fuse_halo"] = rng.choice((4, 8, 16))
        elif f == "windows":
            c.update(image="maze", dtype="f32", text_seed=seed)
        elif f == "random":
            n = side(20, 400)
            c.update(nodes=n, reach=rng.randint(0, n // 12), text_seed=seed)
        if f in ("windows", "random", "segment") and rng.random() < 0.5:
            c["ccl_lanes"] = rng.choice((2, 4))
        return c
    if kind == "stream":
        return {"kind": kind, "formula": rng.choice(("grow", "plain")), "image": "scan", "dtype": dtype,
                "h": side(96, 3000), "w": side(96, 3000), "fmt": fmt}
    if kind == "batch":
        lo = side(40, 400)
        return {"kind": kind, "formula": rng.choice(("segment", "plain", "grow")), "image": "scan", "dtype": dtype,
                "n": rng.randint(2, 96), "lo": lo, "hi": lo * rng.randint(2, 4), "size_seed": seed, "fmt": fmt}
    if kind == "volume":
        return {"kind": kind, "formula": "volume", "dtype": dtype, "depth": side(6, 200), "h": side(24, 256),
                "w": side(24, 256), "fmt": fmt}
    if kind == "labels3":
        return {"kind": "labels", "depth": side(4, 200), "h": side(24, 256), "w": side(24, 256), "cell": 8}
    if kind in ("labels", "pj"):
        c = {"kind": kind, "h": side(64, 4096), "w": side(64, 4096), "cell": rng.choice((2, 8, 32))}
        c.update({"depth": 1} if kind == "labels" else {"reconnect": rng.choice((8, 16))})
        return c
    return {"kind": "serve", "formula": "random", "image": "noise", "dtype": dtype, "n": rng.randint(2, 6), "lo": 128,
            "hi": side(512, 3000), "size_seed": seed, "requests": rng.randint(4, 24), "slots": rng.choice((2, 4)),
            "text_seed": seed}


def outputs_of(f, heights_widths, fmt):
    """One buffer per image holding every output mask of it, and the masks."""
    n = vlg.formula_info(f)["outputs"]
    bufs, masks = [], []
    for h, w in heights_widths:
        shape, t = ((n, h, (w + 63) // 64), torch.int64) if fmt == "packed" else ((n, h, w), torch.uint8)
        bufs.append(torch.zeros(shape, dtype=t, device=DEV))
        masks.append(list(bufs[-1].unbind(0)))
    return bufs, masks


def serve_formula(case, k):
    nodes = (20, 60, 120, 250)[k % 4]
    return dict(case, nodes=nodes, reach=nodes // 16, text_seed=case["text_seed"] + k)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = random.Random(seed)
    kind = case["kind"]
    s = {"case": case}
    if kind == "serve":
        s["server"] = vlg.Server(slots=case["slots"], budget_bytes=4 << 30)
        s["ctx"] = ctx = vlg.create(0)
        images = [vlg.load_image(ctx, make_image(case, gen, rng, h, w)) for h, w in sides(case)]
        fs = [vlg.compile_formula(ctx, formula_text(serve_formula(case, k))) for k in range(4)]
        pick = random.Random(case["size_seed"])
        s["requests"], s["bufs"] = [], []
        for _ in range(case["requests"]):
            im, f = pick.choice(images), pick.choice(fs)
            bufs, masks = outputs_of(f, [im.shape[1:]], "packed")
            s["requests"].append((f, im, masks[0]))
            s["bufs"] += bufs
        return s
    s["ctx"] = ctx = vlg.create(0)
    if kind in ("labels", "pj"):
        d, h, w = case.get("depth", 1), case["h"], case["w"]
        s["mask"] = pack_bits(smooth(gen, (d, h, w), case["cell"]).reshape(d * h, w) > 0.5)
        s["out"] = torch.empty((d, h, w) if d > 1 else (h, w), dtype=torch.int32, device=DEV)
        return s
    for name in ("ccl_lanes", "fuse_halo"):
        if name in case:
            vlg.set_tunable(ctx, name, case[name])
    s["f"] = f = vlg.compile_formula(ctx, formula_text(case))
    if kind == "batch":
        s["images"] = [vlg.load_image(ctx, make_image(case, gen, rng, h, w)) for h, w in sides(case)]
        # one buffer for all masks of the batch
        n = vlg.formula_info(f)["outputs"]
        per = [(h, (w + 63) // 64 if case["fmt"] == "packed" else w) for h, w in sides(case)]
        s["buf"] = torch.zeros(n * sum(h * w for h, w in per),
                               dtype=torch.int64 if case["fmt"] == "packed" else torch.uint8, device=DEV)
        at, s["outs"] = 0, []
        for h, w in per:
            s["outs"].append([s["buf"][at + k * h * w:at + (k + 1) * h * w].view(h, w) for k in range(n)])
            at += n * h * w
        return s
    if kind == "volume":
        d, h, w = case["depth"], case["h"], case["w"]
        t = torch.empty((2, d, h, w), dtype=TYPES[case["dtype"]], device=DEV)
        for c in range(2):
            a = smooth(gen, (1, d * h, w), 24).reshape(d, h, w)
            # smooth along the slices too: a slowly turning mix of two fields
            b = smooth(gen, (1, h, w), 24)
            z = torch.linspace(0, 1, d, device=DEV)[:, None, None]
            f3 = b * (1 - z) + b.flip(-1) * z
            t[c] = typed((0.8 * f3 + 0.2 * a + 0.03 * torch.randn((d, h, w), generator=gen, device=DEV)).clamp_(0, 1),
                         case["dtype"])
        s["im"] = vlg.load_volume(ctx, t)
        s["bufs"], m = outputs_of(f, [(d * h, w)], case["fmt"])
        s["outs"] = m[0]
        return s
    t = make_image(case, gen, rng)
    s["bufs"], m = outputs_of(f, [(case["h"], case["w"])], case["fmt"])
    s["outs"] = m[0]
    if kind == "stream":
        s["pixels"] = t
    else:
        s["im"] = vlg.load_image(ctx, t)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("check", "volume"):
        vlg.check_all(s["ctx"], s["f"], s["im"], s["outs"], fmt=case["fmt"])
        return s["bufs"]
    if kind == "stream":
        im = vlg.load_image(s["ctx"], s["pixels"])
        vlg.check_all(s["ctx"], s["f"], im, s["outs"], fmt=case["fmt"])
        return s["bufs"]
    if kind == "batch":
        vlg.check_batch(s["ctx"], s["f"], s["images"], s["outs"], fmt=case["fmt"])
        return s["buf"]
    if kind == "labels":
        if case["depth"] > 1:
            return vlg.ccl_labels3(s["ctx"], s["mask"], case["depth"], case["h"], case["w"], out=s["out"])
        return vlg.ccl_labels(s["ctx"], s["mask"], case["h"], case["w"], out=s["out"])
    if kind == "pj":
        labels, stats = vlg.ccl_labels_pj(s["ctx"], s["mask"], case["h"], case["w"], case["reconnect"], out=s["out"])
        return [labels, stats["main_iterations"], stats["rounds"]]
    ids = [s["server"].submit(f, im, outs) for f, im, outs in s["requests"]]
    for i in ids:
        s["server"].wait(i)
    return s["bufs"]


def work(case):
    """Bytes: each channel read once, each output written once; no product
    of matrices is on this path, so the operations counted are the formula's
    pixel-wise operators on 64-bit words."""
    kind = case["kind"]
    if kind in ("labels", "pj"):
        n = case.get("depth", 1) * case["h"] * case["w"]
        return {"bytes": n / 8 + 4 * n, "flops": 0}
    if kind == "serve":
        size, pick, total = sides(case), random.Random(case["size_seed"]), 0
        counts = [formula_text(serve_formula(case, k)).count("output ") for k in range(4)]
        for _ in range(case["requests"]):
            (h, w), n = pick.choice(size), pick.choice(counts)
            total += h * w * BYTES[case["dtype"]] + n * h * ((w + 63) // 64) * 8
        return {"bytes": total, "flops": 0}
    outs = formula_text(case).count("output ")
    size = sides(case) if kind == "batch" else [(case.get("depth", 1) * case["h"], case["w"])]
    total = 0
    for h, w in size:
        total += h * w * BYTES[case["dtype"]] * formula_channels(case["formula"])
        total += outs * (h * ((w + 63) // 64) * 8 if case["fmt"] == "packed" else h * w)
    return {"bytes": total, "flops": 0}
