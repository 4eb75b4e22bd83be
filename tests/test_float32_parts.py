"""Float32 operands keep all their bits: no part of the three-part operands, and no product
of the parts that matter, is lost in any contraction of the float32 kernels.

A lost part costs 2^-18 of what it touches, which for most contractions is no more than the
error of float32 sums, so the bars of the parity tests pass it.  Here the error against
float64 is compared with the pattern that each mistake would give (three_part.py): its
share of the pattern is one with the mistake, and measured within 0.11 without; the bar is
0.25.  The CPU tests plant every mistake in the emulation and see the bar exceeded.
"""
import numpy as np
import pytest

import oracle
import three_part as T
from gpu_helpers import banner, state_of, to_device, to_host
from oracle import backward as BW

SHARE = 0.25
# (C, H, M, N): every tile count and both widths of the tuned kernels, several blocks of points;
# then runtime shapes (forward only): half a K step, five slice tiles and more
TUNED = [(64, 4, 16, 150), (64, 2, 32, 150), (128, 8, 16, 129), (128, 2, 32, 200), (128, 8, 64, 130)]
RUNTIME = [(48, 3, 48, 129), (256, 8, 64, 64), (512, 8, 16, 70), (160, 10, 144, 65)]


def mistakes(shape):
    names = T.FORWARD + (T.BACKWARD if shape in TUNED else ())
    return [(n, k) for n in names for k in T.KINDS]


@pytest.mark.parametrize("C,H,M,N", [TUNED[0], TUNED[2], RUNTIME[0], RUNTIME[2]])
def test_a_planted_mistake_shows_beside_rounding_of_its_size(C, H, M, N):
    """Rounding noise of 1e-6 of each output, as large as any float32 kernel here shows."""
    shape = (C, H, M, N)
    x, g, W = T.case(*shape)
    ref = T.run(x, g, W, H, M, 2.0, backward=shape in TUNED)
    # without a mistake the emulation is the oracle
    want = BW.layer_backward(x, W, g, H, M, 2.0)
    want["out"] = oracle.layer_forward_fast(x, W, H, M, 2.0)
    for k in set(want) & set(ref):
        assert np.abs(ref[k] - want[k]).max() <= 1e-11 * np.abs(want[k]).max(), k
    rng = np.random.default_rng(1)
    for m in mistakes(shape):
        planted = T.run(x, g, W, H, M, 2.0, plant=m, backward=shape in TUNED)
        name, pat = T.pattern(ref, planted, list(ref))
        noise = rng.standard_normal(pat.shape) * 1e-6 * np.sqrt((ref[name] ** 2).mean())
        assert abs(T.share(noise, pat)) <= SHARE, (m, name)
        assert T.share(noise + planted[name] - ref[name], pat) >= 3 * SHARE, (m, name)


@pytest.mark.gpu
@pytest.mark.parametrize("C,H,M,N", TUNED + RUNTIME)
def test_no_part_is_lost(C, H, M, N):
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    shape = (C, H, M, N)
    banner(f"three-part operands: C={C} H={H} M={M} N={N} fp32")
    x, g, W = T.case(*shape)
    backward = shape in TUNED
    lw, xd = LayerWeights(W), to_device(x, "fp32")
    with PhysicsAttention(C, H, M, C // H, 0.5, "fp32", group_span=4096, max_points=N) as layer:
        got = {"out": to_host(layer.forward(lw, xd, tile=4096))}
        st = state_of(layer)
        got.update(s_raw=st["s_raw"], d=st["d"])
        if backward:
            dx, grads = layer.backward(lw, xd, to_device(g, "fp32"), tile=4096)
            got.update(dx=to_host(dx), **{k: v.cpu().numpy().astype(np.float64) for k, v in grads.items()})
        torch.cuda.synchronize()
    ref = T.run(x, g, W, H, M, 2.0, backward=backward)
    for m in mistakes(shape):
        name, pat = T.pattern(ref, T.run(x, g, W, H, M, 2.0, plant=m, backward=backward), list(got))
        s = T.share(got[name] - ref[name], pat)
        print(f"{m[0]} {m[1]}: share {s:+.3f} in {name}", flush=True)
        assert abs(s) <= SHARE, (m, name, s)


@pytest.mark.gpu
def test_runtime_shapes_keep_the_slice_weights_in_bf16_storage():
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    C, H, M, N = 48, 3, 48, 129
    banner("three-part slice weights: C=48 H=3 M=48 bf16")
    x, g, W = T.case(C, H, M, N, bf16_storage=True)
    with PhysicsAttention(C, H, M, C // H, 0.5, "bf16", group_span=4096, max_points=N) as layer:
        layer.forward(LayerWeights(W), to_device(x, "bf16"), tile=4096)
        st = state_of(layer)
    ref = T.run(x, g, W, H, M, 2.0, backward=False, stored_bf16=True)
    planted = T.run(x, g, W, H, M, 2.0, plant=("P1.sum", "a"), backward=False, stored_bf16=True)
    for name in ("s_raw", "d"):
        s = T.share(st[name] - ref[name], planted[name] - ref[name])
        print(f"share {s:+.3f} in {name}", flush=True)
        assert abs(s) <= SHARE, (name, s)
