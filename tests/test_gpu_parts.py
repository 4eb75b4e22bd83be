"""Spans cut into parts (a mesh of few spans): every pass-1 kernel against the
oracle, and the guarantees that must not depend on the cut.

9,001 points in spans of 4,096 give parts of 64 to 192 points, the last span
and its last part ragged.  A part's sum and the fold are float32 sums as before, so
the bars are those of the other tests.
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import (assert_bf16_close, assert_state_close, banner, fp32_bar, match_sums, normwise, rel_l2, state_of,
                         sums_key, to_device, to_host)
from ts3_synth import make_weights, round_bf16

pytestmark = pytest.mark.gpu

N, Q = 9_001, 4_096
SHAPES = [(128, 8, 64, "bf16"),   # projected sums, three block streams
          (128, 2, 64, "bf16"),   # two heads per workgroup, raw sums
          (256, 8, 64, "bf16"),   # wide rows
          (64, 4, 16, "bf16"),    # one head per workgroup
          (128, 8, 64, "fp32"),
          (48, 1, 80, "fp32")]    # runtime shape


@pytest.mark.parametrize("C,H,M,dtype", SHAPES)
def test_parts_match_the_oracle_and_do_not_depend_on_the_tiling(C, H, M, dtype):
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    from paper_2602_04940_amd.layer import layer_forward_noalloc
    banner(f"parts: C={C} H={H} M={M} {dtype}, {N} points in spans of {Q}")
    x64 = np.random.default_rng(8).standard_normal((N, C))
    x64 = round_bf16(x64) if dtype == "bf16" else x64.astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=3, bias_seed=4)
    lw = LayerWeights(W)
    x = to_device(x64, dtype)
    ref = oracle.build_state(x64, W, H, M, 2.0)
    ref_out = oracle.deslice(x64, W["W2"], W["b2"], ref["Z"], W["b3"], H, M, 2.0)
    with PhysicsAttention(C, H, M, C // H, 0.5, dtype, group_span=Q, max_points=N) as layer:
        out = layer.forward(lw, x, tile=2 * Q, chunk=1000).clone()
        st = state_of(layer)
        spans = layer.get_spans(0, 3)
        # tile by tile, last tile first
        layer.reset()
        for t0 in (2 * Q, Q, 0):
            layer.accumulate(lw, x[t0:t0 + Q], t0)
        layer.finalize(lw)
        layer.attention(lw)
        assert torch.equal(layer.deslice(lw, x), out)
        # a mesh whose first span never arrives: its parts count as zero
        layer.reset()
        layer.accumulate(lw, x[Q:2 * Q], Q)
        layer.accumulate(lw, x[2 * Q:], 2 * Q)
        layer.finalize(lw)
        layer.attention(lw)
        late = state_of(layer)
        # fewer points than max_points
        few = layer.forward(lw, x[:Q + 77].contiguous(), tile=Q, chunk=4096).clone()
    noalloc = torch.empty_like(x)
    layer_forward_noalloc(C, H, M, lw, x, Q, 4096, noalloc, dtype=dtype, group_span=Q)
    torch.cuda.synchronize()
    assert torch.equal(noalloc, out)

    late_ref = match_sums(late, oracle.build_state(x64[Q:], W, H, M, 2.0), x64[Q:], W, H, M, 2.0)
    few_ref = oracle.layer_forward_fast(x64[:Q + 77], W, H, M, 2.0)
    match_sums(st, ref, x64, W, H, M, 2.0)
    key = sums_key(st)
    if dtype == "bf16":
        assert_bf16_close(to_host(out), ref_out, "out")
        assert_state_close(st, ref, "state")
        assert_state_close(late, late_ref, "state without the first span")
        assert_bf16_close(to_host(few), few_ref, "out of fewer points")
    else:
        for what, bar, got, want in (("out", "out", to_host(out), ref_out), (key, key, st[key], ref[key]),
                                     ("d", "d", st["d"], ref["d"]), ("late sums", key, late[key], late_ref[key]),
                                     ("few", "out", to_host(few), few_ref)):
            e = normwise(got, want)
            print(f"{what}: normwise {e:.2e}", flush=True)
            assert e <= fp32_bar(bar), (what, e)
    # the spans that get_spans reports add up to the state (float32 sums of three terms)
    total = spans.astype(np.float64).sum(axis=0)
    assert np.abs(total[..., :-1] - st[key]).max() <= 1e-5 * np.abs(st[key]).max()
    assert np.abs(total[..., -1] - st["d"]).max() <= 1e-5 * st["d"].max()


@pytest.mark.parametrize("N", [2_000, 9_001])
def test_spans_of_a_mesh_much_shorter_than_group_span(N):
    """One span of up to 2^30 points whose mesh has a few thousand: get_spans needs room for
    the parts that exist, not for those of a whole span."""
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    C, H, M = 128, 8, 64
    banner(f"parts of one span of 2^30 points, {N} points")
    x64 = np.random.default_rng(8).standard_normal((N, C)).astype(np.float32).astype(np.float64)
    W = make_weights(C, H, M, C // H, seed=3, bias_seed=4)
    with PhysicsAttention(C, H, M, C // H, 0.5, "fp32", group_span=1 << 30, max_points=N) as layer:
        layer.forward(LayerWeights(W), to_device(x64, "fp32"), tile=1 << 30)
        span = layer.get_spans(0, 1)[0]
        st = state_of(layer)
    # float32 sums of at most 64 parts in order, both of them
    assert np.abs(span[..., :-1] - st["s_raw"]).max() <= 1e-5 * np.abs(st["s_raw"]).max()
    assert np.abs(span[..., -1] - st["d"]).max() <= 1e-5 * st["d"].max()


@pytest.mark.parametrize("C,H,M,dtype", [(64, 4, 16, "fp32"), (64, 8, 16, "bf16")])
def test_spans_of_one_point_and_more_workgroups_than_a_launch_holds(C, H, M, dtype):
    """2.2M spans of one point are 8.8M and 17.6M workgroups: more than 2^32 threads in one
    launch, though each tile of 65,536 points holds far fewer."""
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    N, tile = 2_200_000, 65_536
    banner(f"{N} spans of one point: C={C} H={H} M={M} {dtype}")
    x = torch.randn((N, C), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    x = x.to(torch.bfloat16) if dtype == "bf16" else x
    lw = LayerWeights(make_weights(C, H, M, C // H, seed=3, bias_seed=4))
    outs, states = [], []
    for Q in (1, 4096):
        with PhysicsAttention(C, H, M, C // H, 0.5, dtype, group_span=Q, max_points=N, accum="fp64") as layer:
            outs.append(to_host(layer.forward(lw, x, tile=tile, chunk=tile)[-5000:]))
            states.append(state_of(layer))
    # The same terms in other groups.  Sums of 4,096 positive-weighted terms in float32 against
    # terms added in float64: within 4,096 half ulps at the worst, a few at random (measured
    # 9e-8); the bar is 16 half ulps.
    for k in ("s_raw", "d"):
        e = normwise(states[0][k], states[1][k])
        print(f"{k}: normwise {e:.2e}", flush=True)
        assert e <= 2.0 ** -20, (k, e)
    assert rel_l2(outs[0], outs[1]) <= (1e-2 if dtype == "bf16" else 2.0 ** -20)
