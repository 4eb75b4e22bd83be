"""Decoding a small call (a head per wave) gives the rows of a large one (32 points per
wave), to the bit, and a large one those of the oracle (other tests): one to 24,577
points, the last size of the one and the first of the other on 256 compute units,
with blocks whose logits leave the range of the unshifted softmax.
"""
import numpy as np
import pytest

from gpu_helpers import banner, to_device
from ts3_synth import make_weights, round_bf16

pytestmark = pytest.mark.gpu

BIG = 40_000


@pytest.mark.parametrize("C,H,M", [(128, 8, 64), (128, 8, 32), (64, 4, 32)])
def test_small_calls_give_the_rows_of_a_large_one(C, H, M):
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    banner(f"decoding in small calls: C={C} H={H} M={M}")
    rng = np.random.default_rng(12)
    x64 = rng.standard_normal((BIG, C))
    # Rows whose logits leave the range take their block of 32 rows to the shifted softmax,
    # whose bf16 weights are rounded after the division instead of before: to compare to
    # the bit, no such row in a block that one of the calls below cuts short.
    far = rng.integers(0, BIG, 300)
    far = far[~np.isin(far // 32, [0, 1, 255, 256, 768])]
    x64[np.append(far, 24_575)] *= 400.0
    x = to_device(round_bf16(x64), "bf16")
    lw = LayerWeights(make_weights(C, H, M, C // H, seed=3, bias_seed=4))
    with PhysicsAttention(C, H, M, C // H, 0.5, "bf16", group_span=4096, max_points=BIG) as layer:
        whole = layer.forward(lw, x, tile=4096, chunk=BIG).clone()
        for n in (1, 31, 33, 8_191, 8_193, 24_576, 24_577):
            out = torch.full((n + 1, C), 7.0, dtype=x.dtype, device=x.device)
            layer.deslice(lw, x[:n], out[:n])
            assert bool((out[n] == 7.0).all()), n
            assert torch.equal(out[:n], whole[:n]), n


def test_wide_rows_do_not_depend_on_the_calls_size():
    """C = 256: up to 64 points per compute unit run in blocks of 64, more in blocks of 128.
    Rows that need the shifted softmax take their tile of 16 there in either, so calls
    that start on a multiple of 16 agree to the bit, such rows included."""
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    C, H, M = 256, 8, 64
    banner("decoding wide rows in small and large calls")
    rng = np.random.default_rng(12)
    x64 = rng.standard_normal((BIG, C))
    x64[rng.integers(0, BIG, 300)] *= 400.0
    x = to_device(round_bf16(x64), "bf16")
    lw = LayerWeights(make_weights(C, H, M, C // H, seed=3, bias_seed=4))
    with PhysicsAttention(C, H, M, C // H, 0.5, "bf16", group_span=4096, max_points=BIG) as layer:
        whole = layer.forward(lw, x, tile=4096, chunk=BIG).clone()
        for a, b in ((0, 4_096), (16, 8_000), (20_000, 36_384), (39_984, BIG), (0, 16_384), (0, 16_400)):
            assert torch.equal(layer.deslice(lw, x[a:b]), whole[a:b]), (a, b)
