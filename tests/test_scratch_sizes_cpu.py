"""Scratch of a compact soft-shadow frame: a_i and values of the list levels
by rank and the coarsest level's values, each on a 256-byte boundary, and
nothing else (its shadow bits live in the edge tiles only)."""
import pytest

from paper_1906_04576_amd import mr


def up(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("W,H,N,en", [(3840, 2160, 4, 0b1111), (384, 256, 4, 0b1101), (128, 6, 2, 0b11)])
def test_soft_shadow_scratch_holds_no_shadow_bits(W, H, N, en):
    mp = mr.MaskParams(num_levels=N, level_enable=en, sigma2=(0.924,) * (N - 1) + (0.0,),
                       weight=(100.0,) * (N - 1) + (1.0,))
    _, scratch = mr.mr_pyramid_bytes(W, H, 100.0, mp, mr.MR_EFFECT_SHADOW)
    n = {i: (W >> (i - 1)) * (H >> (i - 1)) for i in range(1, N + 1) if (en >> (i - 1)) & 1}
    assert scratch == sum(2 * up(4 * n[i]) for i in n if i < N) + up(4 * n[N])
