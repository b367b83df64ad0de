"""a_i and the stencil of levels large enough for blur tiles of 32 rows (2048
of them fill the chip; smaller levels take tiles of 8), bit for bit the
oracle's: sizes on both sides of the rule, heights that end inside a tile,
widths that end inside a tile and inside a word, every kind of radius."""
import math
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_1906_04576_amd import mr

pytestmark = pytest.mark.gpu

DEV = "cuda"


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("W,H,R", [(4096, 4096, 6), (4096, 4064, 6), (4096, 4066, 3), (4102, 3890, 0), (4102, 3890, 1),
                                   (4102, 3890, 8), (4102, 3890, 9), (4102, 3890, 16)])
def test_tall_blur_tiles(W, H, R):
    log(f"[gpu] blur tiles {W}x{H} R={R}")
    g = torch.Generator(device=DEV).manual_seed(W + H + R)
    d = torch.full((H, W), 5.0, device=DEV)
    spikes = torch.rand((H, W), generator=g, device=DEV) < 3e-4
    spikes[0, 0] = spikes[-1, -1] = spikes[H // 2, W // 2] = True
    d[spikes] = 9.0
    n = torch.zeros((3, H, W), device=DEV)
    n[2] = -1.0
    a = dict(num_levels=2, level_enable=3, sigma2=(0.0 if R == 0 else (R / 2.5) ** 2, 0.0), weight=(50.0, 1.0),
             radius=(R, 0), normal_cos=float(np.float32(math.cos(math.radians(25.0)))))
    mp = mr.MaskParams(**a)
    m = mr.mr_build_masks(d, n, np.float32(100.0), mp, masks=mr.alloc_masks(W, H, np.float32(100.0), mp, DEV,
                                                                            level_map=False, level_depth=False))
    torch.cuda.synchronize()
    ref = oracle.build_pyramid(m.edge.cpu().numpy(), oracle.MaskParams(**a))
    assert ref.E.sum() > 1000
    assert np.array_equal(m.alpha[1].cpu().numpy(), ref.alpha[1])
    assert np.array_equal(m.stencil[1].cpu().numpy(), ref.stencil[1])
    assert int(m.count[0].item()) == int(ref.stencil[1].sum())
