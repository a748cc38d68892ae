"""The whole-grid launches (many tiles per launch, blocks read in place) against the per-tile calls of the same
grid, which test_gpu_parity.py checks against the oracle: ragged blocks, grouped heads, strided inputs, every
kind of grid."""
import math

import pytest
import torch

from helpers import assert_close, np64

pytestmark = pytest.mark.gpu
BF = torch.bfloat16

# heads, kv_heads, rows per block, grid, H, causal, layout, packed
CASES = [
    (3, 3, 37, 5, 128, True, "cyclic", False),        # blocks of less than a wavefront's rows
    (4, 2, 130, 4, 96, True, "contiguous", False),    # triangle of tiles, grouped heads
    (2, 1, 200, 3, 80, False, "contiguous", True),    # all tiles, packed inputs
    (8, 2, 65, 7, 64, True, "cyclic", True),
    (5, 5, 300, 1, 128, True, "contiguous", False),   # a grid of one tile
    (64, 64, 2048, 2, 64, False, "cyclic", False),    # long rows, many heads
    (2, 2, 700, 2, 128, True, "contiguous", False),   # few tiles
    (8, 1, 90, 4, 96, True, "cyclic", False),         # ... the heads of a group
    (30, 30, 300, 3, 128, True, "contiguous", False),
    (60, 30, 270, 2, 80, True, "cyclic", True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dq%dkv_%dx%d_H%d_%s_%s" % (c[0], c[1], c[2], c[3], c[4], "causal" if c[5] else "full", c[6]))
def test_batched_grid_equals_the_per_tile_calls(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d, grid as g2d
    heads, kvh, rows, side, H, causal, layout, packed = case
    n, scale = rows * side, 1.0 / math.sqrt(H)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(19)

    def make(h):
        if packed:
            return torch.randn(n, h, H, generator=gen, device="cuda").to(BF).permute(1, 0, 2)
        return torch.randn(h, n, H, generator=gen, device="cuda").to(BF)
    Q, K, V, dO = make(heads), make(kvh), make(kvh), make(heads)
    print("grid case", case, flush=True)
    assert a2d._ext().grid_forward(Q, K, V, side, causal, layout == "cyclic", scale) is not None
    O, lse = g2d.forward(Q, K, V, side, causal, layout, scale)
    Or, lr = g2d.forward(Q, K, V, side, causal, layout, scale, merge="ring")      # tile by tile
    assert_close(O, np64(Or), BF, "O")
    assert_close(lse, np64(lr), torch.float32, "lse", rel=False)
    assert a2d._ext().grid_backward(Q, K, V, Or, dO, lr, side, causal, layout == "cyclic", scale) is not None
    got = g2d.backward(Q, K, V, Or, dO, lr, side, causal, layout, scale)
    again = g2d.backward(Q, K, V, Or, dO, lr, side, causal, layout, scale)
    ref = g2d.backward(Q, K, V, Or, dO, lr, side, causal, layout, scale, ds_handover=False)      # tile by tile
    for name, x, y, z in zip(("dQ", "dK", "dV"), got, again, ref):
        assert torch.equal(x, y), name + " differs from call to call"
        err = (x.float() - z.float()).norm() / z.float().norm()
        assert err < 4e-3, "%s: relative error %.2e" % (name, err)    # both round their sums to bf16 once
