"""The runtime-shape kernels (any C and M that are multiples of 16) at the edges of
their tiles, against the oracle: a channel count with half a K32 step, one to
sixteen slice tiles, head groups with padding and a last group of fewer heads,
channels in several chunks, blocks of 32 and 64 points, and ragged point counts.

Float32 storage computes on exact three-part operands with float32 sums: the bars are a
small multiple of the errors measured (gpu_helpers.FP32_BARS).  bf16 storage rounds x, W2' and Z as stored.
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_bf16_close, assert_state_close, banner, fp32_bar, normwise, rel_l2, state_of, to_device, to_host
from ts3_synth import make_weights, round_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,M,N", [
    (16, 1, 16, 1),       # half a K step, one slice tile, one point
    (48, 3, 48, 129),     # half a K step; a last group of one head; one point past two blocks
    (80, 5, 80, 65),      # five slice tiles, five channel tiles
    (160, 10, 144, 300),  # nine slice tiles; a group of one head with 16 padding slots
    (64, 16, 192, 77),    # twelve slice tiles
    (256, 16, 128, 130),  # eight slice tiles
    (512, 8, 16, 200),    # four channel tiles per wave
    (512, 8, 32, 127),
    (512, 16, 96, 63),    # channels in chunks
    (256, 8, 64, 1000),
])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_runtime_shapes_at_tile_edges(C, H, M, N, dtype):
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    if dtype == "bf16" and (C, M) == (256, 64):
        pytest.skip("a tuned shape")
    banner(f"runtime shape C={C} H={H} M={M} N={N} {dtype}")
    x64 = np.random.default_rng(N).standard_normal((N, C))
    x64 = round_bf16(x64) if dtype == "bf16" else x64.astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=8, bias_seed=9)
    ref = oracle.build_state(x64, W, H, M, 2.0)
    out_ref = oracle.deslice(x64, W["W2"], W["b2"], ref["Z"], W["b3"], H, M, 2.0)
    lw = LayerWeights(W)
    x = to_device(x64, dtype)
    with PhysicsAttention(C, H, M, C // H, 0.5, dtype, group_span=192, max_points=N) as layer:
        out = layer.forward(lw, x, tile=192, chunk=100)
        st = state_of(layer)
        # an injected state whose rows differ strongly
        rng = np.random.default_rng(2)
        Z, b3 = rng.standard_normal((H, M, C)), rng.standard_normal(C)
        layer.set_state(lw, Z, b3)
        inj = layer.deslice(lw, x)
    inj_ref = oracle.deslice(x64, W["W2"], W["b2"], Z.astype(np.float32), b3.astype(np.float32), H, M, 2.0)
    if dtype == "bf16":
        assert_bf16_close(to_host(out), out_ref, "out")
        assert_state_close(st, ref, "state")
        assert rel_l2(to_host(inj), inj_ref) <= 2e-2
    else:
        for what, got, want in (("out", to_host(out), out_ref), ("s_raw", st["s_raw"], ref["s_raw"]),
                                ("d", st["d"], ref["d"]), ("injected", to_host(inj), inj_ref)):
            e = normwise(got, want)
            print(f"{what}: normwise {e:.2e}", flush=True)
            assert e <= fp32_bar("out" if what == "injected" else what), (what, e)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_runtime_shape_with_logits_far_apart(dtype):
    """Logits spread over thousands of exp2 units: one-hot weights, and slices that no point reaches."""
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    C, H, M, N = 96, 3, 48, 700
    x64 = np.random.default_rng(3).standard_normal((N, C))
    x64 = round_bf16(x64) if dtype == "bf16" else x64.astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=5)
    W["W2"] = (round_bf16(W["W2"].astype(np.float64)) if dtype == "bf16" else W["W2"]).astype(np.float32)
    W["b2"] = W["b2"].reshape(H, M).copy()
    W["b2"][:, :16] = -1e4  # slices that no point reaches
    W["b2"] = W["b2"].reshape(-1)
    tau = 2.0 ** -6
    ref = oracle.build_state(x64, W, H, M, 1 / tau)
    lw = LayerWeights(W)
    with PhysicsAttention(C, H, M, C // H, tau, dtype, group_span=256, max_points=N) as layer:
        out = to_host(layer.forward(lw, to_device(x64, dtype), tile=256))
        st = state_of(layer)
    assert np.isfinite(out).all()
    assert (st["d"][:, :16] == 0).all() and (st["s_raw"][:, :16] == 0).all()
    if dtype == "fp32":
        assert normwise(st["d"], ref["d"]) <= 1e-4
