"""Naive passes on either grid (resident for few samples or taps, a block per
256 texels from there on), and taps left over after the groups of eight: every
count around the rules, on images below and above one chunk per resident
block, bit for bit the oracle's values."""
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


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def scenes():
    out = {}
    for W, H in ((130, 37), (1500, 700)):  # 19 chunks; 4102 chunks, more than are resident
        sc = scenegen.make_scene(5, 40, 12)
        gb = scenegen.render_gbuffer(sc, scenegen.orbit_view(3), W, H)
        out[W] = (sc, gb, scenegen.lambert_color(sc, gb))
    return out


@pytest.mark.parametrize("W", [130, 1500])
@pytest.mark.parametrize("S", [1, 2, 5, 7, 8, 9])
def test_samples_on_either_grid(scenes, W, S):
    sc, gb, col = scenes[W]
    log(f"[gpu] naive grids W={W} S={S}")
    K = scenegen.ssao_kernel(S, seed=S)
    d, n, c, k = dev(gb.depth), dev(gb.normal), dev(col), dev(K)
    ao = mr.mr_eval_ssao(d, n, gb.focal, k, 1.0, 0.02)[1]
    gi = mr.mr_eval_ssgi(d, n, c, gb.focal, k, 2.0, 0.02)[1]
    torch.cuda.synchronize()
    ref = oracle.ssao_level(gb.depth, gb.normal, gb.focal, 1, oracle.SSAOParams(K, 1.0, 0.02), None)
    assert np.array_equal(ao.cpu().numpy(), ref)
    ref = oracle.ssgi_level(gb.depth, gb.normal, col.astype(F32), gb.focal, 1, oracle.SSGIParams(K, 2.0, 0.02), None)
    assert np.array_equal(gi.cpu().numpy(), ref)


@pytest.mark.parametrize("W", [130, 1500])
@pytest.mark.parametrize("nb,npcf", [(1, 1), (1, 2), (2, 2), (3, 4), (5, 6), (7, 12), (13, 15)])
def test_taps_on_either_grid(scenes, W, nb, npcf):
    sc, gb, _ = scenes[W]
    log(f"[gpu] naive grids W={W} taps {nb}/{npcf}")
    si = scenegen.render_shadow_inputs(sc, gb.view, 96)
    bd, pd = scenegen.disk_samples(nb, 3), scenegen.disk_samples(npcf, 4)
    size = F32(float(si.light_size) * 4)
    sp = mr.shadow_params(dev(si.shadow_map), si.view_to_light, si.light_focal, size, si.light_near, 0.05, dev(bd),
                          dev(pd))
    out = mr.mr_eval_shadow(dev(gb.depth), gb.focal, sp)[1]
    torch.cuda.synchronize()
    op = oracle.ShadowParams(si.shadow_map, si.view_to_light, si.light_focal, size, si.light_near, F32(0.05), bd, pd)
    assert np.array_equal(out.cpu().numpy(), oracle.pcss_level(gb.depth, gb.focal, 1, op, None))
