"""The splits and short cuts inside the kernels at the sizes where they can
go wrong, bit for bit against the oracle (a split that is right changes no
bit, so no tolerance is needed):

  * samples tested in groups with a remainder, with and without the depth
    test that lets a group skip its general form (noisy depth on both sides
    of the sampling radius, samples off the screen and behind the camera,
    samples longer than the radius), on dense and on strided level planes;
  * light gathered in groups of four samples, taps in groups of eight;
  * a_i taken from row tables or from the plane, for every blur radius, and
    the blur of heights that end inside a tile;
  * the edge image of widths not divisible by 4, from a single tile down to
    widths below 4, with full and half normals;
  * the shadow bits computed inside the edge tiles of a frame;
  * list building with and without the level map in its first launch."""
import math
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
import scenegen
from paper_1906_04576_amd import mr

pytestmark = pytest.mark.gpu

DEV = "cuda"
F32 = np.float32
COS25 = float(F32(math.cos(math.radians(25.0))))


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def noisy(W, H, seed, lo=0.2, hi=40.0, holes=0.03):
    """Depth noise (log-uniform, some background of every kind) and unit
    normals that face anywhere in the front half space."""
    rng = np.random.default_rng(seed)
    d = np.exp(rng.uniform(math.log(lo), math.log(hi), (H, W))).astype(F32)
    # most blocks are smooth, so that coarse levels keep texels
    by, bx = np.mgrid[0:H, 0:W] // 24
    smooth = rng.random((H // 24 + 1, W // 24 + 1))[by, bx] < 0.7
    base = np.exp(rng.uniform(math.log(lo), math.log(hi), (H // 24 + 1, W // 24 + 1)))[by, bx].astype(F32)
    d[smooth] = base[smooth]
    bad = rng.random((H, W)) < np.where(smooth, 0.0005, holes)
    d[bad] = rng.choice(np.array([np.inf, -np.inf, np.nan, 0.0, -2.0], F32), int(bad.sum()))
    n = rng.normal(size=(3, H, W))
    n[2] = -np.abs(n[2]) - 0.05
    n[:, smooth] = np.array([0.0, 0.0, -1.0])[:, None]
    n = (n / np.sqrt((n * n).sum(0))).astype(F32)
    return d, n


def rendered(W, H, seed, cam):
    sc = scenegen.make_scene(seed, 40, 12)
    return sc, scenegen.render_gbuffer(sc, scenegen.orbit_view(cam), W, H)


def mps(N, en=None, sigma2=None, radius=None):
    a = dict(num_levels=N, level_enable=(1 << N) - 1 if en is None else en,
             sigma2=(1.848,) * (N - 1) + (0.0,) if sigma2 is None else sigma2,
             weight=(50.0,) * (N - 1) + (1.0,), radius=(-1,) * N if radius is None else radius, normal_cos=COS25)
    return mr.MaskParams(**a), oracle.MaskParams(**a)


def same(got, ref, what):
    g = got.cpu().numpy() if isinstance(got, torch.Tensor) else got
    assert g.shape == ref.shape, what
    assert np.array_equal(g, ref, equal_nan=True), f"{what}: {int((g != ref).sum())} values differ"


# (samples, radius, kernel scale): group remainders 0..7 on both sides of one
# and of several groups; radii below, inside and above the depths
SAMPLES = [(1, 0.5, 1.0), (2, 3.0, 1.0), (3, 0.05, 1.0), (4, 1.0, 1.0), (7, 0.5, 3.0), (8, 1.0, 1.0), (9, 8.0, 1.0),
           (12, 0.1, 1.0), (15, 50.0, 1.0), (16, 0.5, 1.0), (17, 0.02, 1.0), (24, 2.0, 1.0), (31, 0.3, 8.0),
           (33, 1.0, 1.0), (50, 0.5, 1.0)]


@pytest.mark.parametrize("effect", ["ssao", "ssgi"])
@pytest.mark.parametrize("S,radius,scale", SAMPLES)
def test_sample_groups(effect, S, radius, scale):
    # (width and texel count end inside a wave and inside a block)
    W, H, f = 196, 84, F32(90.0)
    log(f"[gpu] {effect} groups: S={S} r={radius} scale={scale}")
    d, n = noisy(W, H, 40 + S)
    K = (scenegen.ssao_kernel(S, seed=70 + S) * F32(scale)).astype(F32)
    rng = np.random.default_rng(S)
    color = rng.random((3, H, W)).astype(F32)
    mp, omp = mps(3, sigma2=(0.1, 0.1, 0.0))
    dd, nn, kk, cc = dev(d), dev(n), dev(K), dev(color)
    op = (oracle.SSAOParams if effect == "ssao" else oracle.SSGIParams)(K, radius, 0.02)

    def run(masks):
        a = dict(mp=mp if masks is not None else None, masks=masks)
        if effect == "ssao":
            return mr.mr_eval_ssao(dd, nn, f, kk, radius, 0.02, **a)
        return mr.mr_eval_ssgi(dd, nn, cc, f, kk, radius, 0.02, **a)

    dense = mr.mr_build_masks(dd, nn, f, mp)
    strided = mr.mr_build_masks(dd, nn, f, mp, level_map=False, level_depth=False)
    outs = [run(dense), run(strided)]
    plain = run(None)
    torch.cuda.synchronize()
    pyr = oracle.build_pyramid(oracle.edge_image(d, n, omp.depth_ratio, omp.normal_cos), omp)

    def ref(i, st):
        z, m = oracle.level_sample(d, i), oracle.level_sample(n, i)
        if effect == "ssao":
            return oracle.ssao_level(z, m, f, i, op, st)
        return oracle.ssgi_level(z, m, oracle.level_sample(color, i), f, i, op, st)

    for i in pyr.levels:
        st = None if i == pyr.levels[-1] else pyr.stencil[i]
        r = ref(i, st)
        sel = np.ones(r.shape[-2:], bool) if st is None else st.astype(bool)
        assert sel.any(), f"level {i} evaluates nothing"
        for o, what in zip(outs, ("level depth", "strided depth")):
            same(o[i].cpu().numpy()[..., sel], r[..., sel], f"level {i}, {what}")
    same(plain[1], ref(1, None), "naive pass")


def test_fast_reciprocal_square_root_is_exact_over_its_range():
    """Every float of the range against the IEEE operations (a native program
    built with the library's flags)."""
    exe = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "_bin", "rsqrt_check")
    assert os.path.exists(exe), "tests/native programs are not built (run __graft_entry__.build())"
    log("[gpu] rsqrt_check (exhaustive)")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    log(r.stdout.strip())
    assert r.returncode == 0 and "mismatches 0" in r.stdout, r.stdout + r.stderr


# focal lengths on both sides of the exact quotients' range, radii on both
# sides of the fast light's, colours and normals of any size
@pytest.mark.parametrize("focal,radius,scale", [(90.0, 0.5, 1.0), (2.0 ** -13, 0.5, 1.0), (2.0 ** 24, 0.5, 1.0),
                                                (90.0, 1e-6, 1.0), (90.0, 5e-6, 1.0), (0.01, 2.0, 1.0),
                                                (90.0, 1.0, 1e-12), (90.0, 1.0, 1e-20), (90.0, 1.0, 1e12)])
def test_light_ranges(focal, radius, scale):
    W, H, f = 132, 50, F32(focal)
    log(f"[gpu] light ranges f={focal} r={radius} normals x {scale}")
    d, n = noisy(W, H, 77, lo=2.0, hi=2.5)
    if radius < 1e-3:
        d = (d * F32(radius)).astype(F32)
    m = n.copy()
    rng = np.random.default_rng(3)
    m[:, rng.random((H, W)) < 0.5] *= F32(scale)
    m[:, rng.random((H, W)) < 0.1] = 0.0
    color = (rng.random((3, H, W)) * 1e3).astype(F32)
    K = scenegen.ssao_kernel(15, seed=5)
    with np.errstate(all="ignore"):
        ref = oracle.ssgi_level(d, m, color, f, 1, oracle.SSGIParams(K, radius, 0.02), None)
    out = mr.mr_eval_ssgi(dev(d), dev(m), dev(color), f, dev(K), radius, 0.02)
    torch.cuda.synchronize()
    same(out[1], ref, "naive pass")


@pytest.mark.parametrize("nb,npcf,sm", [(1, 1, 1), (2, 7, 5), (7, 8, 64), (8, 9, 256), (9, 16, 3), (17, 33, 128)])
def test_tap_groups(nb, npcf, sm):
    W, H = 196, 84
    log(f"[gpu] taps {nb}/{npcf}, map {sm}")
    sc, gb = rendered(W, H, 5, 3)
    si = scenegen.render_shadow_inputs(sc, gb.view, max(sm, 2))
    smap = np.ascontiguousarray(si.shadow_map[:sm, :sm])
    bd, pd = scenegen.disk_samples(nb, 3), scenegen.disk_samples(npcf, 4)
    size = F32(float(si.light_size) * 4)
    op = oracle.ShadowParams(smap, si.view_to_light, si.light_focal, size, si.light_near, F32(0.05), bd, pd)
    sp = mr.shadow_params(dev(smap), si.view_to_light, si.light_focal, size, si.light_near, 0.05, dev(bd), dev(pd))
    d = dev(gb.depth)
    out = mr.mr_eval_shadow(d, gb.focal, sp)
    hard = mr.mr_shadow_hard(d, gb.focal, sp)
    torch.cuda.synchronize()
    same(out[1], oracle.pcss_level(gb.depth, gb.focal, 1, op, None), "soft shadow")
    same(hard, oracle.hard_shadow(gb.depth, gb.focal, 1, op), "hard shadow")


@pytest.mark.parametrize("R", list(range(0, 9)) + [12, 16])
def test_blur_radii(R):
    """Both frame paths and the step-by-step masks.  Heights end inside the
    blur's tile of 8 rows at every level."""
    log(f"[gpu] blur radius {R}")
    s2 = 0.0 if R == 0 else (R / 2.5) ** 2
    for W, H, N in ((256, 76, 3), (212, 44, 3), (50, 26, 2), (6, 2, 2)):
        rad = (R,) * (N - 1) + (0,)
        mp, omp = mps(N, sigma2=(s2,) * (N - 1) + (0.0,), radius=rad)
        _, gb = rendered(W, H, 9 + N, 2)
        K = scenegen.ssao_kernel(8)
        d, n = dev(gb.depth), dev(gb.normal)
        sp = mr.ssao_params(dev(K), 1.0, 0.02)
        masks = mr.mr_build_masks(d, n, gb.focal, mp)
        frame = mr.mr_frame("ssao", d, n, gb.focal, mp, sp)
        torch.cuda.synchronize()
        pyr = oracle.build_pyramid(oracle.edge_image(gb.depth, gb.normal, omp.depth_ratio, omp.normal_cos), omp)
        cnt = masks.count.cpu().numpy().view(np.uint32)
        for i in pyr.levels[:-1]:
            same(masks.alpha[i], pyr.alpha[i], f"{W}x{H} a_{i}")
            same(masks.stencil[i], pyr.stencil[i], f"{W}x{H} stencil {i}")
            assert cnt[i - 1] == len(pyr.worklist[i])
        ref = oracle.frame("ssao", gb.depth, gb.normal, gb.focal, omp, oracle.SSAOParams(K, 1.0, 0.02)).out
        same(frame, ref, f"{W}x{H} frame")


@pytest.mark.parametrize("N", [1, 2])
@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 62, 127, 129, 130, 131, 254, 257, 258, 259, 514])
def test_edges_of_ragged_widths(W, f16, N):
    """(An odd width has one level only.)  Rows of background and edges at
    the last columns, where the loads of a row's last lane are shifted."""
    if N == 2 and W % 2:
        N = 1
    for H in (2, 16, 22):
        log(f"[gpu] edges {W}x{H} N={N} f16={f16}")
        d, n = noisy(W, H, 300 + W + H, lo=4.0, hi=6.0, holes=0.1)
        nh = n.astype(np.float16) if f16 else n
        n32 = nh.astype(F32)
        mp, omp = mps(N)
        masks = mr.mr_build_masks(dev(d), dev(nh), F32(60.0), mp)
        torch.cuda.synchronize()
        E = oracle.edge_image(d, n32, omp.depth_ratio, omp.normal_cos)
        pyr = oracle.build_pyramid(E, omp)
        same(masks.edge, pyr.E, "edge image")
        same(masks.level_map, pyr.level_map, "level map")
        if N == 2:
            same(masks.alpha[1], pyr.alpha[1], "a_1")
            same(masks.level_depth[2], oracle.level_sample(d, 2), "level depth")


@pytest.mark.parametrize("W,H,N", [(128, 8, 2), (256, 36, 3), (384, 72, 4), (640, 200, 4)])
@pytest.mark.parametrize("f16", [False, True])
def test_shadow_bits_in_the_edge_tiles(W, H, N, f16):
    log(f"[gpu] soft-shadow frame {W}x{H} N={N} f16={f16}")
    sc, gb = rendered(W, H, 6, 4)
    depth = gb.depth.copy()
    rng = np.random.default_rng(W + H)
    bad = rng.random(depth.shape) < 0.05
    depth[bad] = rng.choice(np.array([np.inf, np.nan, 0.0, -1.0], F32), int(bad.sum()))
    si = scenegen.render_shadow_inputs(sc, gb.view, 96)
    bd, pd = scenegen.disk_samples(5, 1), scenegen.disk_samples(11, 2)
    nh = gb.normal.astype(np.float16) if f16 else gb.normal
    op = oracle.ShadowParams(si.shadow_map, si.view_to_light, si.light_focal, si.light_size, si.light_near,
                             F32(0.05), bd, pd)
    sp = mr.shadow_params(dev(si.shadow_map), si.view_to_light, si.light_focal, si.light_size, si.light_near, 0.05,
                          dev(bd), dev(pd))
    mp, omp = mps(N)
    out = mr.mr_frame("shadow", dev(depth), dev(nh), gb.focal, mp, sp)
    torch.cuda.synchronize()
    same(out, oracle.frame("shadow", depth, nh.astype(F32), gb.focal, omp, op).out, "frame")


@pytest.mark.parametrize("level_map", [True, False])
@pytest.mark.parametrize("W,H,N", [(5, 3, 1), (66, 34, 2), (180, 68, 3), (520, 264, 4), (1040, 528, 5)])
def test_lists_with_and_without_the_level_map(W, H, N, level_map):
    log(f"[gpu] lists {W}x{H} N={N} level_map={level_map}")
    d, n = noisy(W, H, W, holes=0.01)
    mp, omp = mps(N, sigma2=(0.1,) * (N - 1) + (0.0,))
    masks = mr.mr_build_masks(dev(d), dev(n), F32(60.0), mp, level_map=level_map)
    torch.cuda.synchronize()
    pyr = oracle.build_pyramid(oracle.edge_image(d, n, omp.depth_ratio, omp.normal_cos), omp)
    cnt = masks.count.cpu().numpy().view(np.uint32)
    for i in pyr.levels[:-1]:
        k = len(pyr.worklist[i])
        assert cnt[i - 1] == k, f"count {i}"
        same(masks.worklist[i][:k].cpu().numpy().view(np.uint32), pyr.worklist[i], f"list {i}")
    if level_map:
        same(masks.level_map, pyr.level_map, "level map")


@pytest.mark.parametrize("R", [1, 2])
@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("W,H,N,levels,rel", [(128, 8, 4, 0b1111, 0.05), (128, 40, 2, 0b0011, 0.5),
                                              (640, 72, 3, 0b0111, 3.0), (1152, 40, 4, 0b1110, 1e-3),
                                              (256, 64, 3, 0b0101, 1e-14), (256, 64, 3, 0b0111, 1e25)])
def test_bilateral_windows(W, H, N, levels, rel, f16, R):
    """Windows cut by every border, across stencil words and ranking tiles
    (1152 columns: 36 words), and tolerances outside the range of the
    quotient from one reciprocal."""
    log(f"[gpu] bilateral {W}x{H} N={N} levels={levels:04b} rel={rel} R={R} f16={f16}")
    d, n = noisy(W, H, W + H, lo=2.0, hi=6.0)
    K = scenegen.ssao_kernel(8)
    mp, omp = mps(N, sigma2=(0.1,) * (N - 1) + (0.0,))
    nh = n.astype(np.float16) if f16 else n
    out = mr.mr_frame("ssao", dev(d), dev(nh), F32(80.0), mp, mr.ssao_params(dev(K), 1.0, 0.02),
                      bilateral=mr.Bilateral(levels=levels, radius=R, depth_rel=rel),
                      level_dtype=torch.float16 if f16 else torch.float32)
    torch.cuda.synchronize()
    ref = oracle.frame("ssao", d, nh.astype(F32), F32(80.0), omp, oracle.SSAOParams(K, 1.0, 0.02),
                       level_dtype=np.float16 if f16 else None,
                       bilateral=oracle.BilateralParams(levels=levels, radius=R, depth_rel=rel))
    same(out, ref.out, "blurred frame")
