"""The SSAO launches with depth tiles test their samples in groups of 4 and
keep a_i's row tables in the tile's LDS: sample counts around whole groups,
and images whose blocks go from list chunks on to tiles (more chunks than
blocks), bit for bit the frame that gathers from the depth plane."""
import math
import sys

import numpy as np
import pytest
import torch

import scenegen
from paper_1906_04576_amd import mr

pytestmark = pytest.mark.gpu

DEV = "cuda"


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def noisy_frame(W, H, seed, noise):
    """Smooth blocks with a share of noisy ones: long lists and a dense level."""
    rng = np.random.default_rng(seed)
    by, bx = np.mgrid[0:H, 0:W] // 32
    base = rng.uniform(4.0, 8.0, (H // 32 + 1, W // 32 + 1)).astype(np.float32)
    d = base[by, bx].copy()
    loud = rng.random((H // 32 + 1, W // 32 + 1))[by, bx] < noise
    d[loud] *= rng.uniform(0.8, 1.2, int(loud.sum())).astype(np.float32)
    n = np.zeros((3, H, W), np.float32)
    n[0], n[2] = 0.28, -0.96
    return torch.from_numpy(d).to(DEV), torch.from_numpy(n).to(DEV)


def params(N):
    return mr.MaskParams(num_levels=N, level_enable=(1 << N) - 1, sigma2=(1.848,) * (N - 1) + (0.0,),
                         weight=(50.0,) * (N - 1) + (1.0,), normal_cos=float(np.float32(math.cos(math.radians(25.0)))))


@pytest.mark.parametrize("W,H,N,noise", [(256, 96, 3, 0.3), (2048, 1536, 2, 0.5), (3072, 1024, 2, 0.9)])
@pytest.mark.parametrize("S", [1, 3, 4, 5, 7, 8, 11, 12, 13, 256])
def test_groups_and_row_tables_in_the_tile(W, H, N, noise, S):
    log(f"[gpu] depth tiles {W}x{H} N={N} S={S}")
    d, n = noisy_frame(W, H, W + S, noise)
    sp = mr.ssao_params(torch.from_numpy(scenegen.ssao_kernel(S, seed=S)).to(DEV), 1.0, 0.02)
    mp = params(N)
    ref = mr.mr_frame("ssao", d, n, np.float32(300.0), mp, sp)
    got = {h: mr.mr_frame("ssao", d, n, np.float32(300.0), mp, sp, eval_halo=h) for h in (8, 16, 24)}
    torch.cuda.synchronize()
    assert float(ref.max()) > 0.0
    for h, out in got.items():
        assert torch.equal(out, ref), h
