"""Decoding more points than one block per workgroup, for every bf16 kernel of pass 2:
rows of late blocks and of the ragged last one against the oracle, through deslice, forward
with small and large chunks and the entry that allocates nothing, which must all give
the same bits, and the same twice.

65,537 points are one more than one block per workgroup of the 256-point kernels on 256
compute units; 600,001 points give a workgroup up to ten blocks.
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_bf16_close, banner, to_host
from ts3_synth import make_weights

pytestmark = pytest.mark.gpu

SIZES = (65_537, 100_003, 600_001)
TILE = 65_536


@pytest.mark.parametrize("C,H,M", [
    (64, 4, 16), (64, 2, 32), (128, 8, 16), (128, 4, 64),  # a head's Z at a time
    (64, 4, 32), (128, 8, 32), (128, 8, 64),               # slice-state form
    (256, 8, 64),                                          # wide rows
])
def test_late_blocks_match_the_oracle_by_every_route(C, H, M):
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    from paper_2602_04940_amd import _lib as L
    from paper_2602_04940_amd.layer import layer_forward_noalloc
    rng = np.random.default_rng(C + M)
    big = max(SIZES)
    xs = torch.randn((big, C), generator=torch.Generator("cuda").manual_seed(M), device="cuda").to(torch.bfloat16)
    W = make_weights(C, H, M, C // H, seed=3, bias_seed=4)
    lw = LayerWeights(W)
    for n in SIZES:
        banner(f"late blocks: C={C} H={H} M={M} bf16, {n} points")
        x = xs[:n].contiguous()
        noalloc = torch.empty_like(x)
        layer_forward_noalloc(C, H, M, lw, x, TILE, TILE, noalloc, group_span=8192)
        with PhysicsAttention(C, H, M, C // H, 0.5, "bf16", group_span=8192, max_points=n) as layer:
            out = layer.forward(lw, x, tile=TILE, chunk=TILE).clone()
            Z = layer.get(L.TS3_ZP).astype(np.float64)
            whole = layer.deslice(lw, x)
            again = layer.deslice(lw, x)
            large = layer.forward(lw, x, tile=TILE, chunk=1_000_000)
        torch.cuda.synchronize()
        for what, got in (("deslice", whole), ("second deslice", again), ("chunks of 1M", large), ("no-alloc", noalloc)):
            assert torch.equal(got, out), (n, what)
        # the first and last rows of each 65,536, some between, and the ragged end
        rows = np.unique(np.concatenate(
            [np.arange(a, min(a + 16, n)) for a in range(0, n, 65_536)] + [np.arange(n - 300, n)] +
            [rng.integers(a, min(a + 65_536, n), 64) for a in range(0, n, 65_536)]))
        xr = to_host(x[torch.from_numpy(rows).cuda()])
        assert_bf16_close(to_host(out[torch.from_numpy(rows).cuda()]),
                          oracle.deslice(xr, W["W2"], W["b2"], Z, W["b3"], H, M, 2.0), f"{n} points", block=16)


@pytest.mark.parametrize("C,H,M", [(64, 4, 32), (128, 8, 32), (128, 8, 64), (128, 4, 64), (256, 8, 64)])
@pytest.mark.parametrize("n", [30_001, 65_537 + 224])
def test_last_row_outside_the_unshifted_softmax(C, H, M, n):
    """A last row whose logits leave the unshifted softmax's range, in a block with up to
    seven waves past the end (which work on that row as well), alone and with 40 rows
    before it.  The temperature makes W2' = W2, which is bfloat16, so the logits are exact
    to float32 and one-hot weights are as sharp here as in the oracle."""
    import torch
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    from paper_2602_04940_amd import _lib as L
    from ts3_synth import round_bf16
    banner(f"last row outside the window: C={C} H={H} M={M} bf16, {n} points")
    tau = float(np.float32(1.4426950408889634))
    W = make_weights(C, H, M, C // H, seed=3, bias_seed=4)
    W["W2"] = round_bf16(W["W2"].astype(np.float64)).astype(np.float32)
    lw = LayerWeights(W)
    rng = np.random.default_rng(n)
    Z, b3 = rng.standard_normal((H, M, C)), rng.standard_normal(C)
    xs = torch.randn((n, C), generator=torch.Generator("cuda").manual_seed(M), device="cuda")
    for far in (1, 41):
        x = xs.clone()
        x[-far:] *= 400.0
        x = x.to(torch.bfloat16)
        with PhysicsAttention(C, H, M, C // H, tau, "bf16", group_span=8192, max_points=n) as layer:
            layer.forward(lw, x, tile=65_536)
            cached = [layer.deslice(lw, x) for _ in range(2)]
            state = layer.get(L.TS3_ZP).astype(np.float64)
            layer.set_state(lw, Z, b3)
            injected = [layer.deslice(lw, x) for _ in range(2)]
        torch.cuda.synchronize()
        xr = to_host(x[-300:])
        for what, (a, b), zz, bb in (("cached", cached, state, W["b3"]),
                                     ("injected", injected, Z.astype(np.float32), b3.astype(np.float32))):
            assert torch.equal(a, b), (far, what)
            assert_bf16_close(to_host(a[-300:]), oracle.deslice(xr, W["W2"], W["b2"], zz, bb, H, M, 1 / tau),
                              f"{far} far rows, {what}", block=16)
