"""The slice-domain kernels (last fold level, Linear1, token attention, Linear3)
at the edges of what they accept, against the oracle: head widths that do not
divide a workgroup, one wide head, a working set past 64 KiB of
LDS, one and several runs of part sums, both fold precisions, and no biases.

All sums are float32 (or float64 in the fold) of well-scaled terms: the bars are a small
multiple of the errors measured (gpu_helpers.FP32_BARS).
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import banner, fp32_bar, normwise, state_of, to_device, to_host
from ts3_synth import make_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,M", [
    (128, 1, 16),   # one head of width 128: its backward leaves Linear1 and Linear3 in memory
    (128, 2, 32),   # 150 KB of LDS with them
    (64, 16, 16),   # heads of width 4
])
def test_token_backward(C, H, M):
    import torch
    from oracle import backward as BW
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    N = 700
    banner(f"token backward: C={C} H={H} M={M}")
    rng = np.random.default_rng(9)
    x64, g64 = (rng.standard_normal((N, C)).astype(np.float32).astype(np.float64) for _ in range(2))
    W = make_weights(C, H, M, C // H, seed=6, bias_seed=7)
    ref = BW.layer_backward(x64, {k: np.asarray(v, np.float64) for k, v in W.items()}, g64, H, M, 2.0)
    lw, x, g = LayerWeights(W), to_device(x64, "fp32"), to_device(g64, "fp32")
    with PhysicsAttention(C, H, M, C // H, 0.5, "fp32", group_span=256, max_points=N) as layer:
        layer.forward(lw, x, tile=256)
        dx, grads = layer.backward(lw, x, g, tile=256)
        torch.cuda.synchronize()
    got = dict(dx=to_host(dx), **{k: v.cpu().numpy().astype(np.float64) for k, v in grads.items()})
    for k in ("dx", "dW2", "db2", "dW1", "db1", "dWq", "dWk", "dWv", "dW3", "db3"):
        e = normwise(got[k], ref[k])
        print(f"{k}: normwise {e:.2e}", flush=True)
        assert e <= fp32_bar(k), (k, e)


@pytest.mark.parametrize("C,H,M,N,Q,accum,biases", [
    (96, 32, 16, 700, 64, "fp32", True),      # head width 3: 85 groups of threads, one thread idle
    (240, 1, 16, 300, 300, "fp64", True),     # head width 240: one group of threads
    (224, 2, 64, 500, 128, "fp32", False),    # head width 112, 104 KiB of LDS
    (48, 3, 144, 400, 100, "fp64", True),     # 144 slices: 9 columns per lane of the softmax
    (64, 4, 32, 9000, 100, "fp32", True),     # 90 spans: two runs
    (64, 4, 32, 9000, 100, "fp64", False),
])
def test_slice_tokens_and_attention(C, H, M, N, Q, accum, biases):
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    banner(f"token side: C={C} H={H} M={M} N={N} Q={Q} {accum}")
    x64 = np.random.default_rng(5).standard_normal((N, C)).astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=6, bias_seed=7)
    if not biases:
        for b in ("b1", "b2", "b3"):
            W[b] = np.zeros_like(W[b])
    ref = oracle.build_state(x64, W, H, M, 2.0)
    out_ref = oracle.deslice(x64, W["W2"], W["b2"], ref["Z"], W["b3"], H, M, 2.0)
    lw = LayerWeights({k: v for k, v in W.items() if biases or not k.startswith("b")})
    x = to_device(x64, "fp32")
    with PhysicsAttention(C, H, M, C // H, 0.5, "fp32", group_span=Q, max_points=N, accum=accum) as layer:
        out = layer.forward(lw, x, tile=Q)
        st = state_of(layer)
    for k in ("s_raw", "d", "s", "s1", "Z"):
        e = normwise(st[k], ref[k])
        print(f"{k}: normwise {e:.2e}", flush=True)
        assert e <= fp32_bar(k), (k, e)
    assert normwise(to_host(out), out_ref) <= fp32_bar("out")
