"""Float32 storage at the edges of its kernels: one point, one more and one less than a
block, one head and several, every tile count, and both block sizes of pass 2.

Operands enter the matrix cores as three bfloat16 parts with float32 sums: the bars are a
small multiple of the errors measured (gpu_helpers.FP32_BARS).  Whether a part of an
operand is lost, which costs less than these bars, is test_float32_parts.py's question.
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_bf16_close, banner, fp32_bar, normwise, state_of, to_device, to_host
from oracle import backward as BW
from ts3_synth import make_weights, round_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,M,N,Q", [
    (64, 4, 16, 1, 64),
    (64, 2, 32, 65, 1000),     # one point past a 64-point block
    (64, 16, 32, 127, 64),     # head width 4
    (128, 8, 16, 129, 128),    # one point past a 128-point block
    (128, 2, 32, 700, 300),
    (128, 8, 64, 2_000, 2_000),
    (128, 8, 64, 9_000, 9_000),  # parts of many blocks
])
def test_forward_and_backward_against_the_oracle(C, H, M, N, Q):
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    banner(f"float32 kernels: C={C} H={H} M={M} N={N} Q={Q}")
    rng = np.random.default_rng(N)
    x64 = rng.standard_normal((N, C)).astype(np.float32).astype(np.float64)
    g64 = rng.standard_normal((N, C)).astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=2, bias_seed=3)
    W64 = {k: v.astype(np.float64) for k, v in W.items()}
    lw = LayerWeights(W)
    x, g = to_device(x64, "fp32"), to_device(g64, "fp32")
    ref = oracle.build_state(x64, W, H, M, 2.0)
    bref = BW.layer_backward(x64, W64, g64, H, M, 2.0)
    with PhysicsAttention(C, H, M, C // H, 0.5, "fp32", group_span=Q, max_points=N) as layer:
        out = layer.forward(lw, x, tile=Q)
        st = state_of(layer)
        dx, grads = layer.backward(lw, x, g, tile=Q)
        torch.cuda.synchronize()
    pairs = {"out": (to_host(out), oracle.deslice(x64, W["W2"], W["b2"], ref["Z"], W["b3"], H, M, 2.0)),
             "s_raw": (st["s_raw"], ref["s_raw"]), "d": (st["d"], ref["d"]), "dx": (to_host(dx), bref["dx"])}
    # one point: all slice tokens coincide, so the logits and q and k get no gradient, only rounding
    pairs.update({n: (to_host(v), bref[n]) for n, v in grads.items()
                  if N > 1 or n not in ("dW2", "db2", "dWq", "dWk")})
    for n, (got, want) in pairs.items():
        e = normwise(got, want)
        print(f"{n}: normwise {e:.2e}", flush=True)
        assert e <= fp32_bar(n), (n, e)


def test_both_block_sizes_of_pass_2_decode_a_point_the_same():
    """Up to 128 points per compute unit run in blocks of 128, more in blocks of 256."""
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    C, H, M, N = 128, 8, 64, 70_001
    banner("float32 pass 2: blocks of 128 and 256 points")
    x = torch.randn((N, C), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    lw = LayerWeights(make_weights(C, H, M, C // H, seed=2, bias_seed=3))
    with PhysicsAttention(C, H, M, C // H, 0.5, "fp32", group_span=4096, max_points=N) as layer:
        whole = layer.forward(lw, x, tile=4096).clone()
        parts = torch.cat([layer.deslice(lw, x[a:a + 9_999]) for a in range(0, N, 9_999)])
        torch.cuda.synchronize()
    assert torch.equal(whole, parts)


def test_logits_far_apart_and_an_unreachable_slice():
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    C, H, M, N = 64, 4, 32, 600
    x64 = np.random.default_rng(3).standard_normal((N, C)).astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=5)
    W["b2"] = np.where(np.arange(H * M) % M < 8, -1e4, W["b2"]).astype(np.float32)
    tau = 2.0 ** -6
    ref = oracle.build_state(x64, W, H, M, 1 / tau)
    with PhysicsAttention(C, H, M, C // H, tau, "fp32", group_span=256, max_points=N) as layer:
        out = to_host(layer.forward(LayerWeights(W), to_device(x64, "fp32"), tile=256))
        st = state_of(layer)
    assert np.isfinite(out).all()
    assert (st["d"][:, :8] == 0).all() and (st["s_raw"][:, :8] == 0).all()
    assert normwise(st["d"], ref["d"]) <= 1e-4


@pytest.mark.parametrize("C,H,M,dtype", [
    (64, 4, 32, "fp32"), (128, 8, 64, "fp32"), (256, 8, 64, "fp32"), (48, 3, 32, "bf16"),
    (64, 4, 16, "bf16"), (64, 4, 32, "bf16"), (128, 8, 64, "bf16"), (256, 8, 64, "bf16"),
])
def test_minus_infinity_in_b2_closes_a_slice(C, H, M, dtype):
    """A closed slice has no weight, no sums and no gradient; the others are the oracle's."""
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    banner(f"closed slices: C={C} H={H} M={M} {dtype}")
    N, closed = 600, np.arange(H * M) % M % 5 == 1
    rng = np.random.default_rng(4)
    x64 = rng.standard_normal((N, C))
    x64 = round_bf16(x64) if dtype == "bf16" else x64.astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=5, bias_seed=6)
    W["b2"] = np.where(closed, -np.inf, W["b2"]).astype(np.float32)
    W64 = {k: v.astype(np.float64) for k, v in W.items()}
    lw, x = LayerWeights(W), to_device(x64, dtype)
    ref = oracle.build_state(x64, W64, H, M, 2.0)
    want = oracle.deslice(x64, W["W2"], W["b2"], ref["Z"], W["b3"], H, M, 2.0)
    with PhysicsAttention(C, H, M, C // H, 0.5, dtype, group_span=256, max_points=N) as layer:
        out = to_host(layer.forward(lw, x, tile=256))
        st = state_of(layer)
        if dtype == "fp32" and C <= 128:
            g64 = rng.standard_normal((N, C)).astype(np.float32).astype(np.float64)
            dx, grads = layer.backward(lw, x, to_device(g64, "fp32"), tile=256)
            bref = BW.layer_backward(x64, W64, g64, H, M, 2.0)
            assert normwise(to_host(dx), bref["dx"]) <= fp32_bar("dx")
            for n, v in grads.items():
                assert normwise(to_host(v), bref[n]) <= fp32_bar(n), n
            assert bool((grads["dW2"][:, torch.from_numpy(closed)] == 0).all())
    assert (st["d"].reshape(-1)[closed] == 0).all()
    if dtype == "fp32":
        assert normwise(out, want) <= fp32_bar("out")
    else:
        assert_bf16_close(out, want, "out")
