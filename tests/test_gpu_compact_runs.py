"""Work lists of levels whose chunks are summed in runs (above 4096 chunks of
4096 texels), against the stencils' nonzero positions: sizes on both sides of
one chunk per run, ragged ends, full and nearly empty stencils."""
import math
import sys

import pytest
import torch

from paper_1906_04576_amd import mr

pytestmark = pytest.mark.gpu

DEV = "cuda"


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("level_map", [True, False])
@pytest.mark.parametrize("W,H,N,share", [(4096, 4096, 3, 2e-4), (4096, 4098, 2, 2e-4), (4102, 4100, 2, 2e-4),
                                         (8192, 6152, 4, 1e-5), (8192, 6152, 2, 0.5), (16384, 8200, 3, 1e-6),
                                         (5000, 10002, 2, 0.0)])
def test_lists_in_runs_of_chunks(W, H, N, share, level_map):
    log(f"[gpu] lists {W}x{H} N={N} share={share} level_map={level_map}")
    g = torch.Generator(device=DEV).manual_seed(W + H)
    d = torch.full((H, W), 5.0, device=DEV)
    spikes = torch.rand((H, W), generator=g, device=DEV) < share
    spikes[-1, -1] = True  # the last texel is listed at every level
    d[spikes] = 9.0
    n = torch.zeros((3, H, W), dtype=torch.float16, device=DEV)
    n[2] = -1.0
    mp = mr.MaskParams(num_levels=N, level_enable=(1 << N) - 1, sigma2=(0.1,) * (N - 1) + (0.0,),
                       weight=(50.0,) * (N - 1) + (1.0,), normal_cos=math.cos(math.radians(25.0)))
    m = mr.mr_build_masks(d, n, 100.0, mp, masks=mr.alloc_masks(W, H, 100.0, mp, DEV, level_map=level_map,
                                                                level_depth=False))
    torch.cuda.synchronize()
    for i in range(1, N):
        want = torch.nonzero(m.stencil[i].reshape(-1)).reshape(-1).to(torch.int32)
        k = int(m.count[i - 1].item())
        assert k == want.numel() and k > 0, (i, k, want.numel())
        assert torch.equal(m.worklist[i].reshape(-1)[:k].view(torch.int32), want), i
    assert int(m.count[N - 1].item()) == 0
    if level_map:
        owner = torch.full((H, W), N, dtype=torch.uint8, device=DEV)
        for i in range(N - 1, 0, -1):
            s = 1 << (i - 1)
            covered = m.stencil[i].bool().repeat_interleave(s, 0).repeat_interleave(s, 1)
            owner[covered] = i
        assert torch.equal(m.level_map, owner)
