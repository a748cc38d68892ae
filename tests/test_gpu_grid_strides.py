"""The whole-grid calls return tensors with the strides of the inputs they belong to (a model that keeps packed
activations views O and the gradients as it views Q, K and V), with the values of the calls on plain copies."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16

# heads, kv_heads, rows per block, grid, H, causal, layout, which of Q, K and V, dO are packed
CASES = [
    (4, 4, 70, 2, 128, True, "cyclic", "q kv g"),
    (6, 2, 33, 3, 80, True, "contiguous", "q kv g"),
    (4, 2, 64, 2, 96, False, "contiguous", "q"),
    (2, 2, 45, 4, 64, True, "cyclic", "kv"),
    (1, 1, 50, 2, 64, True, "contiguous", "q kv g"),         # one head: packed and plain are the same
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dq%dkv_%dx%d_H%d_%s_%s" % (*c[:5], c[6], c[7].replace(" ", "_")))
def test_outputs_keep_the_strides(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d, grid as g2d
    heads, kvh, rows, side, H, causal, layout, packed = case
    n, scale = rows * side, 1.0 / math.sqrt(H)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(23)
    print("grid strides case", case, flush=True)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(BF)
    token_major = lambda h: normal(n, h, H).permute(1, 0, 2)
    Q = token_major(heads) if "q" in packed.split() else normal(heads, n, H)
    dO = token_major(heads) if "g" in packed.split() else normal(heads, n, H)
    if "kv" in packed.split():                               # one [tokens][2][heads][H] projection
        kv = normal(n, 2, kvh, H)
        K, V = kv[:, 0].permute(1, 0, 2), kv[:, 1].permute(1, 0, 2)
    else:
        K, V = normal(kvh, n, H), normal(kvh, n, H)
    assert a2d._ext().grid_forward(Q, K, V, side, causal, layout == "cyclic", scale) is not None
    O, lse = g2d.forward(Q, K, V, side, causal, layout, scale)
    grads = g2d.backward(Q, K, V, O, dO, lse, side, causal, layout, scale)
    plain = [x.contiguous() for x in (Q, K, V)]
    Op, lp = g2d.forward(*plain, side, causal, layout, scale)
    gp = g2d.backward(*plain, Op, dO.contiguous(), lp, side, causal, layout, scale)
    assert lse.is_contiguous() and torch.equal(lse, lp)
    for name, like, x, y in zip(("O", "dQ", "dK", "dV"), (Q, Q, K, V), (O, *grads), (Op, *gp)):
        assert x.stride() == torch.empty_like(like).stride(), name
        assert torch.equal(x, y), name
    if "q" in packed.split():
        assert O.permute(1, 0, 2).view(n, heads * H).data_ptr() == O.data_ptr()
