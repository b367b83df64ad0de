"""What the library is asked to do in use: the calls, their sizes and their inputs.

Every case is one call of a program that holds a resident G-buffer and renders
screen-space lighting from it: whole multi-resolution frames of the three
effects, the naive full-resolution pass they are weighed against, a served
frame on a resident mask pyramid, a batch of uneven frames, the steps called
one by one, and the two SSAO variants (bilateral blur with a foveated mask,
sub-images at full resolution with fewer samples).

`listed` names the common ones, `draw` spreads further ones over the same
ranges, `prepare` makes a call's inputs on the GPU, `run` is one call, `work`
what it cannot do without, and `exact` the same result in 64-bit torch.
"""
import math

import numpy as np
import torch

from paper_1906_04576_amd import mr

# blur variances and blend weights per level and effect (Table 1 of the paper)
SIGMA2 = {"ssao": (0.924, 1.848, 3.696, 0.0), "shadow": (0.924, 1.848, 3.696, 0.0), "ssgi": (0.924, 0.0, 0.924, 0.0)}
WEIGHT = {"ssao": (100.0, 50.0, 20.0, 1.0), "shadow": (1000.0, 1000.0, 1000.0, 1.0),
          "ssgi": (1000.0, 1.0, 100.0, 1.0)}
BIAS_REL, SHADOW_BIAS, LIGHT_SIZE, LIGHT_NEAR, SHADOW_MAP = 0.02, 0.05, 0.5, 1.0, 2048
LIGHT_EYE = (6.0, 14.0, 4.0)
DEPTH_RATIO, NORMAL_COS = 0.05, math.cos(math.radians(25.0))
FAR = 100.0
# frame sizes of a mixed stream of requests
SIZES = ((640, 360), (1280, 720), (1920, 1080), (2560, 1440), (3840, 2160))


def _case(name, call, effect, width, height, levels, enable, samples, radius, **more):
    c = {"call": call, "effect": effect, "width": width, "height": height, "levels": levels, "enable": enable,
         "samples": samples, "radius": radius, "boxes": 200, "spheres": 50, "half_normals": False, "half_levels": False,
         "frames": 1}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # a thumbnail or an inset view: the smallest frame, where launches count
        _case("frame_ssao_256", "frame", "ssao", 256, 256, 3, 0b111, 16, 0.5, boxes=8, spheres=0),
        # a game's frame at a common window size, with a larger sample set
        _case("frame_ssao_720p", "frame", "ssao", 1280, 720, 4, 0b1111, 64, 1.0),
        # the main workload: a 4K frame with 32 samples
        _case("frame_ssao_4k", "frame", "ssao", 3840, 2160, 4, 0b1111, 32, 1.0),
        # the full-resolution pass, for a reference image or without masks
        _case("naive_ssao_4k", "naive", "ssao", 3840, 2160, 4, 0b1111, 32, 1.0),
        # soft shadows at 4K from a G-buffer with FP16 normals
        _case("frame_shadow_4k", "frame", "shadow", 3840, 2160, 4, 0b1111, 32, 1.0, half_normals=True),
        # one bounce of indirect light; half resolution is left out for it
        _case("frame_ssgi_1440p", "frame", "ssgi", 2560, 1440, 4, 0b1101, 64, 2.0),
        # the full-resolution pass of the indirect light
        _case("naive_ssgi_1080p", "naive", "ssgi", 1920, 1080, 4, 0b1101, 64, 2.0),
        # a serving loop's most frequent request: the scene's masks are resident
        _case("served_ssao_1080p", "served", "ssao", 1920, 1080, 4, 0b1111, 32, 1.0),
        # uneven frames of several clients rendered together
        _case("batch_ssgi_8", "batch", "ssgi", 3840, 2160, 4, 0b1101, 64, 2.0, frames=8),
        # the steps one by one on a width that no vector load divides
        _case("steps_ssao_1366", "steps", "ssao", 1366, 768, 2, 0b11, 32, 1.0),
        # a headset's frame: foveated masks, blurred sub-images in FP16
        _case("blur_ssao_1440p", "blur", "ssao", 2560, 1440, 4, 0b1111, 32, 1.0, half_normals=True, half_levels=True),
        # sub-images at full resolution with fewer samples, masks included
        _case("fullres_ssao_1080p", "fullres", "ssao", 1920, 1080, 4, 0b1111, 32, 1.0),
    ]


def draw(rng):
    call = rng.choice(("frame",) * 6 + ("naive",) * 2 + ("served", "served", "batch", "steps", "steps", "blur", "fullres"))
    effect = "ssao" if call in ("blur", "fullres") else rng.choice(("ssao", "ssao", "shadow", "ssgi"))
    if call == "batch" and effect == "shadow":
        effect = "ssao"
    levels = rng.choice((3, 4, 4, 4)) if call != "steps" else rng.choice((1, 2, 3, 4, 5))
    # width and height over 128 .. 3840 and 72 .. 2160, odd multiples among them
    w = 128.0 * 30.0 ** rng.random()
    h = w * rng.choice((9 / 16, 9 / 16, 3 / 4, 1.0))
    # resident pyramids, batches and the blur take widths that 128 divides
    step = 128 if call in ("served", "batch", "blur") or rng.random() < 0.5 else 1 << (levels - 1)
    width = min(3840, max(step, int(w) // step * step))
    hs = 1 << (levels - 1)
    height = min(2160, max(hs, int(h) // hs * hs))
    enable = (1 << levels) - 1
    if effect == "ssgi" and levels >= 3:
        enable &= ~0b10
    samples = {"ssao": rng.choice((8, 16, 24, 32, 32, 50, 64, 128)), "shadow": rng.choice((16, 25, 32, 64)),
               "ssgi": rng.choice((24, 32, 64, 80))}[effect]
    if call in ("naive", "fullres") or effect == "ssgi":
        samples = min(samples, 64)
    return _case(None, call, effect, width, height, levels, enable, samples, rng.choice((0.5, 1.0, 2.0)),
                 boxes=rng.choice((8, 50, 200)), spheres=rng.choice((0, 20, 50)), half_normals=rng.random() < 0.4,
                 half_levels=call == "served" and rng.random() < 0.3, frames=rng.randint(2, 8) if call == "batch" else 1)


def frame_sizes(case):
    """(width, height) of each frame of a case; a batch takes its first frame's size and sizes below it in turn."""
    first = (case["width"], case["height"])
    if case["call"] != "batch":
        return [first]
    below = [s for s in SIZES if s[0] * s[1] <= first[0] * first[1]] or [first]
    return [first] + [below[(3 * k) % len(below)] for k in range(case["frames"] - 1)]


# ---------------------------------------------------------------------------
# inputs: a ground plane with boxes and spheres seen from an orbit camera,
# ray cast on the GPU in 64 bits and rounded to the G-buffer's types
# ---------------------------------------------------------------------------
def _look_at(eye, target=(0.0, 0.0, 0.0)):
    eye = np.asarray(eye, np.float64)
    back = eye - np.asarray(target, np.float64)
    back /= np.linalg.norm(back)
    right = np.cross((0.0, 1.0, 0.0), back)
    right /= np.linalg.norm(right)
    return eye, right, np.cross(back, right), back


def _focal(height):
    return float(np.float32(0.5 * height / math.tan(math.radians(30.0))))


def _scene(case, rs):
    nb, ns = case["boxes"], case["spheres"]
    c, size = rs.uniform(-5.0, 5.0, (nb, 2)), rs.uniform(0.5, 2.0, (nb, 3))
    lo = np.stack([c[:, 0] - size[:, 0] / 2, np.zeros(nb), c[:, 1] - size[:, 2] / 2], 1)
    sc, r = rs.uniform(-5.0, 5.0, (ns, 2)), rs.uniform(0.2, 1.5, ns)
    ball = np.stack([sc[:, 0], r, sc[:, 1], r], 1)
    albedo = np.concatenate([[[0.8, 0.8, 0.8]], rs.uniform(0.2, 1.0, (nb + ns, 3))])
    return np.concatenate([lo, lo + size], 1), ball, albedo


def _render(scene, view, width, height, focal, device):
    """(depth, world normal [3], object) of every pixel in 64 bits; depth is inf where nothing lies before FAR."""
    boxes, balls, _ = scene
    eye, right, up, back = view
    f64 = dict(dtype=torch.float64, device=device)
    X = ((torch.arange(width, **f64) + 0.5 - 0.5 * width) / focal)[None, :]
    Y = ((0.5 * height - (torch.arange(height, **f64) + 0.5)) / focal)[:, None]
    d = [X * float(right[a]) + Y * float(up[a]) - float(back[a]) for a in range(3)]
    t = torch.where(d[1] < 0, -float(eye[1]) / d[1], torch.full_like(d[1], math.inf))
    n = torch.zeros((3, height, width), **f64)
    n[1] = 1.0
    ident = torch.zeros((height, width), dtype=torch.int64, device=device)
    bounds = np.concatenate([boxes, np.concatenate([balls[:, :3] - balls[:, 3:], balls[:, :3] + balls[:, 3:]], 1)])
    for k, b in enumerate(bounds):
        corner = np.array([[b[0 if i & 1 else 3], b[1 if i & 2 else 4], b[2 if i & 4 else 5]] for i in range(8)]) - eye
        z = -(corner @ back)
        if z.min() < 1e-3:
            x0, x1, y0, y1 = 0, width, 0, height
        else:
            u, v = 0.5 * width + focal * (corner @ right) / z, 0.5 * height - focal * (corner @ up) / z
            x0, x1 = max(0, int(u.min()) - 1), min(width, int(u.max()) + 2)
            y0, y1 = max(0, int(v.min()) - 1), min(height, int(v.max()) + 2)
            if x0 >= x1 or y0 >= y1:
                continue
        at = (slice(y0, y1), slice(x0, x1))
        e = [d[a][at] for a in range(3)]
        if k < len(boxes):
            near, axis = None, None
            far = None
            for a in range(3):
                p, q = (float(b[a]) - float(eye[a])) / e[a], (float(b[a + 3]) - float(eye[a])) / e[a]
                lo, hi = torch.minimum(p, q), torch.maximum(p, q)
                if near is None:
                    near, far, axis = lo, hi, torch.zeros_like(lo)
                else:
                    axis = torch.where(lo > near, torch.full_like(lo, float(a)), axis)
                    near, far = torch.maximum(near, lo), torch.minimum(far, hi)
            hit = (near <= far) & (near > 0) & (near < t[at])
            m = [torch.where(axis == a, -torch.sign(e[a]), torch.zeros_like(near)) for a in range(3)]
        else:
            c, r = balls[k - len(boxes)][:3], float(balls[k - len(boxes)][3])
            o = [float(eye[a] - c[a]) for a in range(3)]
            A = e[0] * e[0] + e[1] * e[1] + e[2] * e[2]
            B = e[0] * o[0] + e[1] * o[1] + e[2] * o[2]
            D = B * B - A * (sum(v * v for v in o) - r * r)
            near = (-B - D.clamp(min=0).sqrt()) / A
            hit = (D >= 0) & (near > 0) & (near < t[at])
            m = [(o[a] + near * e[a]) / r for a in range(3)]
        t[at] = torch.where(hit, near, t[at])
        ident[at] = torch.where(hit, torch.full_like(ident[at], k + 1), ident[at])
        for a in range(3):
            n[a][at] = torch.where(hit, m[a], n[a][at])
    return torch.where(t < FAR, t, torch.full_like(t, math.inf)), n, ident


def _hemisphere(samples, rs):
    u = rs.uniform(size=(samples, 3))
    cz, phi = 0.1 + 0.9 * u[:, 0], 2.0 * math.pi * u[:, 1]
    ln, sz = 0.1 + 0.9 * ((np.arange(samples) + u[:, 2]) / samples) ** 2, np.sqrt(1.0 - cz * cz)
    return np.stack([ln * sz * np.cos(phi), ln * sz * np.sin(phi), ln * cz], 1).astype(np.float32)


def _disk(n, rs):
    r, a = np.sqrt(rs.uniform(size=n)), 2.0 * math.pi * rs.uniform(size=n)
    return np.stack([r * np.cos(a), r * np.sin(a)], 1).astype(np.float32)


def _inputs(case, seed, k, device):
    """One frame's G-buffer and effect inputs."""
    rs = np.random.RandomState((int(seed) * 64 + k) % (1 << 32))
    width, height = frame_sizes(case)[k]
    scene = _scene(case, rs)
    a = rs.uniform(0.0, 2.0 * math.pi)
    view = _look_at((11.0 * math.sin(a), rs.uniform(5.0, 9.0), 11.0 * math.cos(a)))
    _, right, up, back = view
    focal = _focal(height)
    depth, world, ident = _render(scene, view, width, height, focal, device)
    sky = ~torch.isfinite(depth)
    axes = (right, up, back)
    normal = torch.stack([sum(world[j] * float(axes[i][j]) for j in range(3)) for i in range(3)])
    normal = torch.where(sky[None], torch.zeros_like(normal), normal)
    g = {"focal": focal, "depth": depth.float().contiguous(),
         "normal": normal.to(torch.float16 if case["half_normals"] else torch.float32).contiguous()}
    if case["effect"] == "ssgi":
        l = np.asarray(LIGHT_EYE) / np.linalg.norm(LIGHT_EYE)
        ndl = sum(world[j] * float(l[j]) for j in range(3)).clamp(min=0)
        lit = torch.from_numpy(scene[2]).to(device)[ident].permute(2, 0, 1) * (0.1 + 0.9 * ndl)
        g["color"] = torch.where(sky[None], torch.zeros_like(lit), lit).half().contiguous()
    if case["effect"] == "shadow":
        lv = _look_at(LIGHT_EYE)
        lf = _focal(SHADOW_MAP)
        g["map"] = _render(scene, lv, SHADOW_MAP, SHADOW_MAP, lf, device)[0].float().contiguous()
        to_light = np.stack(lv[1:]) @ np.stack([right, up, back], 1)
        g["to_light"] = np.concatenate([to_light, (np.stack(lv[1:]) @ (view[0] - lv[0]))[:, None]], 1).astype(np.float32)
        g["light_focal"] = lf
    return g


def _samples(case, seed, device):
    """The effect's sample sets: random directions and offsets of the program's own."""
    rs = np.random.RandomState((int(seed) * 64 + 63) % (1 << 32))
    S = case["samples"]
    if case["effect"] == "shadow":
        return {"blocker": torch.from_numpy(_disk(max(1, S // 2), rs)).to(device),
                "pcf": torch.from_numpy(_disk(S, rs)).to(device)}
    if case["call"] == "fullres":  # each coarser level takes half the samples
        return {i: torch.from_numpy(_hemisphere(max(1, S >> (i - 1)), rs)).to(device) for i in _levels(case)}
    return {"kernel": torch.from_numpy(_hemisphere(S, rs)).to(device)}


def _levels(case):
    return [i for i in range(1, case["levels"] + 1) if (case["enable"] >> (i - 1)) & 1]


def _fovea(case):
    if case["call"] != "blur":
        return None
    w, h = case["width"], case["height"]
    return (w / 2.0, h / 2.0, 0.15 * h, 0.45 * h)


def _mask_params(case):
    n, e = case["levels"], case["effect"]
    pad = (0.924,) * 6
    return mr.MaskParams(num_levels=n, level_enable=case["enable"], depth_ratio=DEPTH_RATIO, normal_cos=NORMAL_COS,
                         sigma2=(SIGMA2[e] + pad)[:n], weight=(WEIGHT[e] + (20.0,) * 6)[:n], fovea=_fovea(case))


def prepare(case, seed):
    dev = torch.device("cuda")
    gs = [_inputs(case, seed, k, dev) for k in range(len(frame_sizes(case)))]
    smp = _samples(case, seed, dev)
    mp, g, effect, call = _mask_params(case), gs[0], case["effect"], case["call"]
    depth, normal, color, focal = g["depth"], g["normal"], g.get("color"), g["focal"]
    if effect == "shadow":
        params = mr.shadow_params(g["map"], g["to_light"], g["light_focal"], LIGHT_SIZE, LIGHT_NEAR, SHADOW_BIAS,
                                  smp["blocker"], smp["pcf"])
    elif call != "fullres":
        params = mr.ssao_params(smp["kernel"], case["radius"], BIAS_REL)
    st = {"call": call, "keep": (gs, smp, mp)}
    half = torch.float16 if case["half_levels"] else torch.float32
    if call in ("frame", "naive", "blur"):
        st["go"] = mr.FrameRunner(effect, depth, normal, focal, mp, call != "naive", color, params, level_dtype=half,
                                  bilateral=mr.Bilateral(0b1110 & case["enable"], 2) if call == "blur" else None)
    elif call == "served":
        npyr, _ = mr.mr_pyramid_bytes(case["width"], case["height"], focal, mp, mr.EFFECTS[effect])
        pyramid = torch.empty(npyr, dtype=torch.uint8, device=dev)
        st["go"] = mr.CachedFrameRunner(effect, depth, normal, focal, mp, pyramid, color, params, level_dtype=half)
        st["go"](build=True)
    elif call == "batch":
        st["go"] = mr.Batch(effect, [{k: x.get(k) for k in ("depth", "normal", "focal", "color")} for x in gs], mp, params)
    elif call == "steps":
        st.update(effect=effect, g=g, mp=mp, params=params, radius=case["radius"], kernel=smp.get("kernel"),
                  masks=mr.alloc_masks(case["width"], case["height"], focal, mp, dev))
        C = 3 if effect == "ssgi" else 1
        st["levels"] = {i: torch.empty(((C,) if C > 1 else ()) + tuple(reversed(mr.level_dims(
            case["width"], case["height"], i))), dtype=torch.float32, device=dev) for i in _levels(case)}
        st["image"] = torch.empty_like(st["levels"][1])
        st["hard"] = torch.empty(depth.shape, dtype=torch.uint8, device=dev) if effect == "shadow" else None
    else:
        masks = mr.alloc_masks(case["width"], case["height"], focal, mp, dev, level_map=False)
        st["masks"] = mr.prepare_build_masks(depth, normal, focal, mp, masks)
        st["go"] = mr.FullresRunner(depth, normal, focal, mp, masks,
                                    {i: mr.ssao_params(t, case["radius"], BIAS_REL) for i, t in smp.items()})
    return st


def run(state):
    call = state["call"]
    if call == "served":
        return state["go"](build=False)
    if call == "steps":
        g, mp, m, lv = state["g"], state["mp"], state["masks"], state["levels"]
        hard = None
        if state["effect"] == "shadow":
            hard = mr.mr_shadow_hard(g["depth"], g["focal"], state["params"], hard=state["hard"])
        mr.mr_build_masks(g["depth"], g["normal"], g["focal"], mp, hard_shadow=hard, masks=m)
        if state["effect"] == "shadow":
            mr.mr_eval_shadow(g["depth"], g["focal"], state["params"], mp, m, out=lv)
        elif state["effect"] == "ssgi":
            mr.mr_eval_ssgi(g["depth"], g["normal"], g["color"], g["focal"], state["kernel"], state["radius"], BIAS_REL,
                            mp, m, out=lv)
        else:
            mr.mr_eval_ssao(g["depth"], g["normal"], g["focal"], state["kernel"], state["radius"], BIAS_REL, mp, m, out=lv)
        mr.mr_upsample_merge(g["focal"], mp, m, lv, 3 if state["effect"] == "ssgi" else 1, out=state["image"])
        return {"image": state["image"], "edge": m.edge, "level_map": m.level_map, "count": m.count[:6],
                "alpha": {str(i): t for i, t in m.alpha.items()}, "stencil": {str(i): t for i, t in m.stencil.items()},
                "depth": {str(i): t for i, t in m.level_depth.items()}}
    if call == "fullres":
        state["masks"]()
    return state["go"]()


def work(case):
    """Inputs read and outputs written once; the arithmetic of the texels that have to be evaluated (every pixel of a
    naive pass; else the share of the texels near edges, which grows as a frame gets smaller)."""
    per_sample, per_texel = {"ssao": (28, 31), "shadow": (12, 45), "ssgi": (45, 31)}[case["effect"]]
    nbytes = flops = 0.0
    for (w, h) in frame_sizes(case):
        n = float(w * h)
        c = 3 if case["effect"] == "ssgi" else 1
        masks = case["call"] not in ("naive", "served")
        share = 1.0 if case["call"] in ("naive", "fullres") else min(1.0, 0.086 * 2160.0 / h)
        gbuf = 4.0 + (2.0 if case["half_normals"] else 4.0) * 3
        if case["effect"] == "shadow" and not masks:
            gbuf = 4.0
        nbytes += n * (gbuf if masks or case["call"] == "naive" else gbuf * share) + 4.0 * c * n
        if case["effect"] == "ssgi":
            nbytes += 6.0 * n * (1.0 if case["call"] == "naive" else share)
        if case["effect"] == "shadow":
            nbytes += 4.0 * SHADOW_MAP * SHADOW_MAP * min(1.0, n / (SHADOW_MAP * SHADOW_MAP))
        if case["call"] == "steps":  # edges, level map, a_i, stencils and level depth are outputs too
            nbytes += 2.0 * n + sum((5.0 + (4.0 if i > 1 else 0.0)) * n / 4 ** (i - 1) for i in _levels(case)[:-1])
        s = case["samples"] * (1.5 if case["effect"] == "shadow" else 1.0)
        flops += n * share * (s * per_sample + per_texel) + (20.0 * n if masks else 0.0)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def _valid(z):
    return torch.isfinite(z) & (z > 0)


def _f32(v):
    return float(np.float32(v))


def _camera(width, height, focal, i):
    return focal / (1 << (i - 1)), 0.5 * width, 0.5 * height


def _position(x, y, z, f, cx, cy):
    return ((x + 0.5) - cx) / f * z, (cy - (y + 0.5)) / f * z, -z


def _at_level(plane, i):
    s = 1 << (i - 1)
    return plane if s == 1 else plane[..., s // 2::s, s // 2::s].contiguous()


def _blocks(n, most=1 << 21):
    return [(a, min(n, a + most)) for a in range(0, n, most)]


def _gather_effect(zl, nl, cl, i, focal, ys, xs, kernel, radius):
    """SSAO (cl is None) or SSGI at the texels (ys, xs) of a level: [1 or 3][texels]."""
    H, W = zl.shape
    f, cx, cy = _camera(W, H, focal, i)
    r, b = _f32(radius), _f32(BIAS_REL)
    S = kernel.shape[0]
    C = 1 if cl is None else 3
    out = torch.zeros((C, ys.numel()), dtype=torch.float64, device=zl.device)
    for a, e in _blocks(ys.numel()):
        y, x = ys[a:e], xs[a:e]
        z = zl[y, x]
        n = [nl[j][y, x] for j in range(3)]
        P = _position(x, y, z, f, cx, cy)
        sg = torch.copysign(torch.ones_like(z), n[2])
        q = -1.0 / (sg + n[2])
        p = n[0] * n[1] * q
        T = (1.0 + sg * n[0] * n[0] * q, sg * p, -sg * n[0])
        B = (p, sg + n[1] * n[1] * q, -n[1])
        acc = torch.zeros((C, y.numel()), dtype=torch.float64, device=zl.device)
        for kx, ky, kz in kernel.tolist():
            Q = [P[j] + kx * r * T[j] + ky * r * B[j] + kz * r * n[j] for j in range(3)]
            d = -Q[2]
            u, v = cx + Q[0] / d * f, cy - Q[1] / d * f
            m = (d > 0) & (u >= 0) & (u < W) & (v >= 0) & (v < H)
            tx, ty = torch.where(m, u, 0.0).floor().long(), torch.where(m, v, 0.0).floor().long()
            zs = zl[ty, tx]
            m &= _valid(zs) & (zs < d - b * d) & ((z - zs).abs() < r)
            if cl is None:
                acc[0] += m
                continue
            X = _position(tx, ty, zs, f, cx, cy)
            vv = [X[j] - P[j] for j in range(3)]
            dd = vv[0] * vv[0] + vv[1] * vv[1] + vv[2] * vv[2]
            m &= dd > 0
            il = 1.0 / dd.sqrt()
            cr = (sum(n[j] * vv[j] for j in range(3)) * il).clamp(min=0)
            ce = (-sum(nl[j][ty, tx] * vv[j] for j in range(3)) * il).clamp(min=0)
            w = torch.where(m, cr * ce / dd.clamp(min=(0.1 * r) ** 2), 0.0)
            for c in range(3):
                acc[c] += cl[c][ty, tx] * w
        acc = acc / S if cl is None else acc * (r * r / S)
        out[:, a:e] = torch.where(_valid(z), acc, 0.0)
    return out


def _light(P, g):
    M, size = g["to_light"].astype(np.float64), g["map"].shape[0]
    L = [M[j, 0] * P[0] + M[j, 1] * P[1] + M[j, 2] * P[2] + M[j, 3] for j in range(3)]
    dr = -L[2]
    su, sv = 0.5 * size + L[0] / dr * g["light_focal"], 0.5 * size - L[1] / dr * g["light_focal"]
    return dr, su, sv, (dr > 0) & (su >= 0) & (su < size) & (sv >= 0) & (sv < size)


def _shadow(zl, i, focal, ys, xs, g, smp, hard):
    """PCSS visibility, or the one-sample shadow bit, at the texels (ys, xs) of a level."""
    H, W = zl.shape
    f, cx, cy = _camera(W, H, focal, i)
    sm, size, bias = g["map"].double(), g["map"].shape[0], _f32(SHADOW_BIAS)
    out = torch.zeros((1, ys.numel()), dtype=torch.float64, device=zl.device)
    for a, e in _blocks(ys.numel()):
        y, x = ys[a:e], xs[a:e]
        z = zl[y, x]
        dr, su, sv, inside = _light(_position(x, y, z, f, cx, cy), g)
        inside = inside & _valid(z)
        su, sv, dr = (torch.where(inside, t, 1.0) for t in (su, sv, dr))
        thr = dr - bias

        def tap(R, p):
            tx, ty = (su + R * p[0]).floor().clamp(0, size - 1).long(), (sv + R * p[1]).floor().clamp(0, size - 1).long()
            return sm[ty, tx]

        if hard:
            out[0, a:e] = inside & (tap(torch.zeros_like(su), (0.0, 0.0)) < thr)
            continue
        l = g["light_focal"] * 0.5 * LIGHT_SIZE
        Rs = l * (dr - LIGHT_NEAR) / (dr * LIGHT_NEAR)
        total, count = torch.zeros_like(z), torch.zeros_like(z)
        for p in smp["blocker"].tolist():
            s = tap(Rs, p)
            total, count = total + torch.where(s < thr, s, 0.0), count + (s < thr)
        some = inside & (count > 0)
        db = torch.where(some, total / count, 1.0)
        Rf = torch.where(some, l * (dr - db) / (db * dr), 0.0)
        lit = torch.zeros_like(z)
        for p in smp["pcf"].tolist():
            lit = lit + ~(tap(Rf, p) < thr)
        out[0, a:e] = torch.where(some, lit / smp["pcf"].shape[0], 1.0)
    return out


def _neighbours(H, W):
    """(own, other) slices of the four neighbour pairs."""
    a, b, f = slice(None, -1), slice(1, None), slice(None)
    return [((f, a), (f, b)), ((f, b), (f, a)), ((a, f), (b, f)), ((b, f), (a, f))]


def _edges(z, n, hard):
    H, W = z.shape
    ok = _valid(z)
    E = torch.zeros((H, W), dtype=torch.bool, device=z.device)
    for own, other in _neighbours(H, W):
        E[own] |= ~ok[other]
        E[own] |= sum(n[j][own] * n[j][other] for j in range(3)) < _f32(NORMAL_COS)
        if hard is not None:
            E[own] |= hard[own] != hard[other]
    t = _f32(DEPTH_RATIO)
    if W >= 3:
        E[:, 1:-1] |= (z[:, :-2] + z[:, 2:] - 2 * z[:, 1:-1]).abs() > t * z[:, 1:-1]
    if H >= 3:
        E[1:-1] |= (z[:-2] + z[2:] - 2 * z[1:-1]).abs() > t * z[1:-1]
    return E & ok


def _pool(E, s):
    H, W = E.shape
    return E.reshape(H // s, s, W // s, s).amax((1, 3)) if s > 1 else E


def _blurred(E, sigma2):
    s2 = _f32(sigma2)
    r = int(math.ceil(3.0 * math.sqrt(s2))) if s2 > 0 else 0
    g = [math.exp(-k * k / (2.0 * s2)) if s2 > 0 else 1.0 for k in range(-r, r + 1)]
    g = torch.tensor(g, dtype=torch.float64, device=E.device) / sum(g)
    x = torch.nn.functional.pad(E.double(), (r, r, r, r))
    H, W = E.shape
    h = sum(g[k] * x[:, k:k + W] for k in range(2 * r + 1))
    return sum(g[k] * h[k:k + H] for k in range(2 * r + 1))


def _taps(n_full, s, n):
    u = (np.arange(n_full) + 0.5) / s - 0.5
    lo = np.floor(u)
    return np.clip(lo, 0, n - 1).astype(np.int64), np.clip(lo + 1, 0, n - 1).astype(np.int64), u - lo


def _upsample(W, H, i, values, stencil):
    """Bilinear of [C][level] over the stencil's texels alone, renormalised, and the sum of their weights."""
    dev = values.device
    Hi, Wi = values.shape[-2:]
    x0, x1, fx = (torch.from_numpy(t).to(dev) for t in _taps(W, 1 << (i - 1), Wi))
    y0, y1, fy = (torch.from_numpy(t).to(dev) for t in _taps(H, 1 << (i - 1), Hi))
    num, den = 0.0, 0.0
    for ty, by in ((y0, 1.0 - fy), (y1, fy)):
        for tx, bx in ((x0, 1.0 - fx), (x1, fx)):
            at = (ty[:, None], tx[None, :])
            b = by[:, None] * bx[None, :]
            st = stencil[at]
            num = num + torch.where(st[None], b[None] * values[(slice(None),) + at], 0.0)
            den = den + torch.where(st, b, 0.0)
    return num, den


def _pyramid(case, z, n, hard, mp):
    levels = _levels(case)
    H, W = z.shape
    E = _edges(z, n, hard)
    if mp.fovea is not None:
        gx, gy, ri, ro = (_f32(v) for v in mp.fovea)
        d2 = ((torch.arange(W, device=z.device) + 0.5 - gx) ** 2)[None, :].double() + \
            ((torch.arange(H, device=z.device) + 0.5 - gy) ** 2)[:, None].double()
        E = (E & (d2 <= ro * ro)) | (d2 <= ri * ri)
    alpha, stencil = {}, {}
    for i in levels[:-1]:
        alpha[i] = _blurred(_pool(E, 1 << (i - 1)), mp.sigma2[i - 1])
        stencil[i] = alpha[i] > 0
    for a, b in zip(levels[:-2], levels[1:-1]):
        stencil[b] = stencil[b] | _pool(stencil[a], 1 << (b - a))
    stencil[levels[-1]] = torch.ones((H >> (levels[-1] - 1), W >> (levels[-1] - 1)), dtype=torch.bool, device=z.device)
    return alpha, stencil


def _bilateral(c, z, stencil):
    H, W = z.shape
    ok = stencil & _valid(z)
    pad = torch.nn.functional.pad
    zp, cp, kp = pad(z, (2, 2, 2, 2), value=1.0), pad(torch.where(ok, c, 0.0), (2, 2, 2, 2)), pad(ok, (2, 2, 2, 2))
    zc = torch.where(ok, z, 1.0)
    num, den = torch.zeros_like(c), torch.zeros_like(c)
    b = (1 / 16, 4 / 16, 6 / 16, 4 / 16, 1 / 16)
    for dy in range(5):
        for dx in range(5):
            zq, at = zp[dy:dy + H, dx:dx + W], (slice(dy, dy + H), slice(dx, dx + W))
            w = torch.where(kp[at], b[dy] * b[dx] * (1.0 - (zq - zc).abs() / (_f32(0.05) * zc)).clamp(min=0), 0.0)
            num, den = num + w * cp[at], den + w
    return torch.where(ok, num / den.clamp(min=1e-30), c)


def _exact_frame(case, g, smp):
    mp = _mask_params(case)
    z, n = g["depth"].double(), g["normal"].double()
    col = g["color"].double() if "color" in g else None
    H, W = z.shape
    C = 3 if case["effect"] == "ssgi" else 1
    levels = _levels(case)

    def texels(stencil):
        return torch.nonzero(stencil, as_tuple=True)

    def evaluate(i, ys, xs):
        if case["effect"] == "shadow":
            return _shadow(_at_level(z, i), i, g["focal"], ys, xs, g, smp, False)
        return _gather_effect(_at_level(z, i), _at_level(n, i), None if col is None else _at_level(col, i), i, g["focal"],
                              ys, xs, smp["kernel"], case["radius"])

    everywhere = torch.ones((H, W), dtype=torch.bool, device=z.device)
    if case["call"] == "naive":
        out = evaluate(1, *texels(everywhere)).reshape(C, H, W)
        return (out if C > 1 else out[0]), None
    hard = None
    if case["effect"] == "shadow":
        hard = _shadow(z, 1, g["focal"], *texels(everywhere), g, smp, True).reshape(H, W) > 0
    alpha, stencil = _pyramid(case, z, n, hard, mp)
    image = None
    for i in reversed(levels):
        st = stencil[i]
        ys, xs = texels(st)
        if case["call"] == "fullres":
            ys, xs = texels(everywhere)
            c = _gather_effect(z, n, None, 1, g["focal"], ys, xs, smp[i], case["radius"]).reshape(1, H, W)
        else:
            c = torch.zeros((C,) + st.shape, dtype=torch.float64, device=z.device)
            c[:, ys, xs] = evaluate(i, ys, xs)
            if case["call"] == "blur" and i > 1:
                c[0] = _bilateral(c[0], _at_level(z, i), st)
            num, den = _upsample(W, H, i, c, st)
            c = torch.where(den > 0, num / torch.where(den > 0, den, 1.0), 0.0)
        if image is None:
            image = c
            continue
        A, _ = _upsample(W, H, i, alpha[i][None], torch.ones_like(st))
        _, den = _upsample(W, H, i, alpha[i][None], st)
        al = torch.where(den > 0, (A[0] * _f32(mp.weight[i - 1])).clamp(max=1.0), 0.0)
        image = c * al + image * (1.0 - al)
    return (image if C > 1 else image[0]), alpha


def exact(case, seed):
    dev = torch.device("cuda")
    smp = _samples(case, seed, dev)
    got = [_exact_frame(case, _inputs(case, seed, k, dev), smp) for k in range(len(frame_sizes(case)))]
    if case["call"] == "batch":
        return [image for image, _ in got]
    if case["call"] == "steps":
        image, alpha = got[0]
        return {"image": image, "edge": None, "level_map": None, "count": None,
                "alpha": {str(i): t for i, t in alpha.items()}, "stencil": {str(i): None for i in alpha},
                "depth": {str(i): None for i in _levels(case) if i > 1}}
    return got[0][0]
