"""Sample sets and disks around the 1024 entries that are staged in LDS (the
larger ones, up to MR_MAX_SAMPLES, are read from global memory), bit for bit
against the oracle: naive passes, evaluation on mask buffers, compact frames,
batches; and SSGI's general form of the samples (depths on both sides of the
radius) with every remainder of its groups."""
import math
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


def scene(W, H, seed, lo=3.0, hi=6.0):
    """Smooth blocks of log-uniform depth, a few invalid texels, unit normals."""
    rng = np.random.default_rng(seed)
    by, bx = np.mgrid[0:H, 0:W] // 12
    shape = (H // 12 + 1, W // 12 + 1)
    d = np.exp(rng.uniform(math.log(lo), math.log(hi), shape))[by, bx]
    d = (d * rng.uniform(0.99, 1.01, (H, W))).astype(F32)
    bad = rng.random((H, W)) < 0.01
    d[bad] = rng.choice(np.array([np.inf, np.nan, 0.0, -1.0], F32), int(bad.sum()))
    n = rng.normal(size=(3,) + shape)[:, by, bx]
    n[2] = -np.abs(n[2]) - 0.3
    n = (n / np.sqrt((n * n).sum(0))).astype(F32)
    color = rng.random((3, H, W)).astype(F32)
    return d, n, color


def mps(N):
    a = dict(num_levels=N, level_enable=(1 << N) - 1, sigma2=(0.1,) * (N - 1) + (0.0,), weight=(50.0,) * (N - 1) + (1.0,),
             normal_cos=COS25)
    return mr.MaskParams(**a), oracle.MaskParams(**a)


def same(got, ref, what):
    g = got.cpu().numpy()
    assert g.shape == ref.shape, what
    assert np.array_equal(g, ref, equal_nan=True), f"{what}: {int((g != ref).sum())} values differ"


@pytest.mark.parametrize("effect", ["ssao", "ssgi"])
# (samples, radius): around the staged sets, a larger one; radii below and
# among the depths
@pytest.mark.parametrize("S,radius", [(1023, 0.5), (1024, 1.0), (1025, 0.5), (1025, 4.0), (1027, 8.0), (2050, 1.0)])
def test_around_the_staged_samples(effect, S, radius):
    W, H, f = 128, 40, F32(70.0)
    log(f"[gpu] {effect} S={S} r={radius}")
    d, n, color = scene(W, H, S)
    K = scenegen.ssao_kernel(S, seed=S)
    mp, omp = mps(2)
    op = (oracle.SSAOParams if effect == "ssao" else oracle.SSGIParams)(K, radius, 0.02)
    col = color if effect == "ssgi" else None
    dd, nn, cc, kk = dev(d), dev(n), dev(color) if effect == "ssgi" else None, dev(K)
    sp = mr.ssao_params(kk, radius, 0.02)
    frame = mr.mr_frame(effect, dd, nn, f, mp, sp, color=cc)
    naive = mr.mr_frame(effect, dd, nn, f, mp, sp, multires=False, color=cc)
    batch = mr.Batch(effect, [dict(depth=dd, normal=nn, focal=f, color=cc)] * 2, mp, sp)()
    masks = mr.mr_build_masks(dd, nn, f, mp)
    if effect == "ssao":
        dense = mr.mr_eval_ssao(dd, nn, f, kk, radius, 0.02, mp, masks)
    else:
        dense = mr.mr_eval_ssgi(dd, nn, cc, f, kk, radius, 0.02, mp, masks)
    torch.cuda.synchronize()
    kw = dict(color=col) if effect == "ssgi" else {}
    multi = oracle.frame(effect, d, n, f, omp, op, **kw)
    full = oracle.frame(effect, d, n, f, omp, op, multires=False, **kw).out
    assert full.max() > 0.0
    same(naive, full, "naive pass")
    same(frame, multi.out, "compact frame")
    for o in batch:
        same(o, multi.out, "batch")
    same(dense[2], (oracle.ssao_level(oracle.level_sample(d, 2), oracle.level_sample(n, 2), f, 2, op, None)
                    if effect == "ssao" else
                    oracle.ssgi_level(oracle.level_sample(d, 2), oracle.level_sample(n, 2),
                                      oracle.level_sample(color, 2), f, 2, op, None)), "coarsest level on mask buffers")


@pytest.mark.parametrize("nb,npcf", [(1024, 1025), (1025, 3), (3, 1025), (1024, 1024), (1031, 1039)])
def test_around_the_staged_disks(nb, npcf):
    W, H = 128, 40
    log(f"[gpu] disks {nb}/{npcf}")
    sc = scenegen.make_scene(5, 40, 12)
    gb = scenegen.render_gbuffer(sc, scenegen.orbit_view(3), W, H)
    si = scenegen.render_shadow_inputs(sc, gb.view, 64)
    bd, pd = scenegen.disk_samples(nb, 3), scenegen.disk_samples(npcf, 4)
    size = F32(float(si.light_size) * 4)
    op = oracle.ShadowParams(si.shadow_map, si.view_to_light, si.light_focal, size, si.light_near, F32(0.05), bd, pd)
    sp = mr.shadow_params(dev(si.shadow_map), si.view_to_light, si.light_focal, size, si.light_near, 0.05, dev(bd),
                          dev(pd))
    mp, omp = mps(2)
    d, n = dev(gb.depth), dev(gb.normal)
    naive = mr.mr_frame("shadow", d, n, gb.focal, mp, sp, multires=False)
    frame = mr.mr_frame("shadow", d, n, gb.focal, mp, sp)
    torch.cuda.synchronize()
    ref = oracle.frame("shadow", gb.depth, gb.normal, gb.focal, omp, op, multires=False).out
    assert ref.min() < 1.0
    same(naive, ref, "naive pass")
    same(frame, oracle.frame("shadow", gb.depth, gb.normal, gb.focal, omp, op).out, "frame")


@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 7, 9])
@pytest.mark.parametrize("radius", [2.0, 5.0, 30.0])
def test_light_of_near_texels(S, radius):
    """Depths of 3 to 6 with radii on both sides: waves of the general form."""
    W, H, f = 128, 48, F32(70.0)
    log(f"[gpu] near texels S={S} r={radius}")
    d, n, color = scene(W, H, 90 + S)
    K = scenegen.ssao_kernel(S, seed=S)
    mp, omp = mps(2)
    op = oracle.SSGIParams(K, radius, 0.02)
    sp = mr.ssao_params(dev(K), radius, 0.02)
    dd, nn, cc = dev(d), dev(n), dev(color)
    naive = mr.mr_frame("ssgi", dd, nn, f, mp, sp, multires=False, color=cc)
    frame = mr.mr_frame("ssgi", dd, nn, f, mp, sp, color=cc)
    torch.cuda.synchronize()
    same(naive, oracle.frame("ssgi", d, n, f, omp, op, multires=False, color=color).out, "naive pass")
    same(frame, oracle.frame("ssgi", d, n, f, omp, op, color=color).out, "frame")
