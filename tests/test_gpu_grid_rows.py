"""The whole-grid launches, which walk all tiles of a grid row (O, dQ) or column (dK, dV) at once, against full attention in
fp64 on the GPU: edges of the blocks and workgroups in layouts of every kind, one-row blocks, split walks, every
workgroup shape."""
import math

import pytest
import torch

from test_gpu_split_walks import _rel

pytestmark = pytest.mark.gpu

# heads, kv_heads, rows per block, grid, H
CASES = [
    (1, 1, 1, 2, 64),
    (3, 1, 1, 32, 128),            # one row of every column
    (2, 2, 63, 2, 128),
    (2, 1, 64, 3, 80),
    (4, 4, 65, 8, 96),             # more columns than the parts of a split walk step over
    (1, 1, 129, 5, 128),
    (40, 40, 257, 2, 64),
    (48, 24, 255, 4, 128),
    (16, 8, 513, 3, 96),
    (2, 2, 2000, 1, 128),          # a grid of one tile
    # every workgroup shape of both kernels, whole walks and shared ones, in each layout and head size (tests/test_host_routes.py)
    (8, 1, 17, 3, 80),
    (8, 1, 132, 7, 64),
    (88, 11, 16, 3, 96),
    (1, 1, 641, 5, 96),
    (1, 1, 16, 1, 128),
    (1, 1, 131, 7, 80),
    (27, 27, 278, 2, 80),
    (61, 61, 140, 4, 64),
    (1, 1, 205, 5, 80),
    (16, 2, 144, 5, 96),
    (272, 34, 16, 1, 128),
    (52, 26, 150, 3, 128),
    (3, 3, 678, 5, 64),
    (1, 1, 585, 5, 128),
    (80, 80, 212, 4, 80),
    (66, 33, 35, 2, 128),
    (3, 3, 1953, 4, 64),
    (40, 5, 140, 4, 96),
    (64, 8, 802, 4, 128),
    (32, 32, 139, 6, 128),
    (1, 1, 583, 9, 80),
    (54, 27, 205, 6, 96),
    (1, 1, 560, 9, 64),
    (4, 2, 1634, 3, 80),
    (27, 27, 139, 7, 80),
    (27, 27, 142, 7, 64),
]
# walks whose forward keeps a SIMD's wavefronts in opposite phases: both workgroup shapes under the mask in each layout, unmasked ones
# whole and shared (tests/test_host_routes.py)
PHASED = [
    (48, 48, 242, 7, 128),
    (40, 8, 212, 8, 128),
    (10, 5, 388, 8, 128),
    (12, 12, 323, 8, 128),
    (16, 8, 258, 7, 128),
    (10, 5, 242, 7, 128),
    (6, 6, 449, 6, 128),
    (4, 2, 388, 8, 128),
]


@pytest.mark.parametrize("layout", ["cyclic", "contiguous"])
@pytest.mark.parametrize("causal", [True, False], ids=["causal", "full"])
@pytest.mark.parametrize("case", CASES + PHASED, ids=lambda c: "%dq%dkv_%dx%d_H%d" % c)
def test_grid_rows(case, causal, layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d, grid as g2d
    heads, kvh, rows, side, H = case
    n, scale, gen = rows * side, 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(29)
    print("grid rows case", case, causal, layout, flush=True)
    make = lambda h: torch.randn(h, n, H, generator=gen, device="cuda").to(torch.bfloat16)
    Q, K, V = make(heads), make(kvh), make(kvh)
    q = Q.double()
    k, v = (x.double().repeat_interleave(heads // kvh, 0) for x in (K, V))
    S = torch.bmm(q, k.transpose(1, 2).contiguous()) * scale
    if causal:
        S = S.masked_fill(torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1), -math.inf)
    lse = torch.logsumexp(S, 2)
    O = torch.bmm(torch.exp(S - lse[..., None]), v)
    assert a2d._ext().grid_forward(Q, K, V, side, causal, layout == "cyclic", scale) is not None
    got, got_lse = g2d.forward(Q, K, V, side, causal, layout, scale)
    # P and O rounded to bf16 once each: 2^-9 a term at most, 3e-3 of the norm and less
    assert _rel(got, O) < 5e-3, "O: %.2e" % _rel(got, O)
    assert (got_lse.double() - lse).abs().max() < 1e-4
    again, again_lse = g2d.forward(Q, K, V, side, causal, layout, scale)
    assert torch.equal(got, again) and torch.equal(got_lse, again_lse)

    dO, Os = make(heads), O.to(torch.bfloat16)
    P = torch.exp(S - lse[..., None])
    w = dO.double()
    dS = P * (torch.bmm(w, v.transpose(1, 2).contiguous()) - (w * Os.double()).sum(2)[..., None])
    fold = lambda x: x.view(kvh, heads // kvh, n, H).sum(1)
    ref = (torch.bmm(dS, k) * scale, fold(torch.bmm(dS.transpose(1, 2).contiguous(), q)) * scale,
           fold(torch.bmm(P.transpose(1, 2).contiguous(), w)))
    args = (Q, K, V, Os, dO, lse.float())
    assert a2d._ext().grid_backward(*args, side, causal, layout == "cyclic", scale) is not None
    grads = g2d.backward(*args, side, causal, layout, scale)
    again = g2d.backward(*args, side, causal, layout, scale)
    for name, x, y, z in zip(("dQ", "dK", "dV"), grads, ref, again):
        assert torch.equal(x, z), name
        # P, dS and the results rounded to bf16 (a sequence of one or two tokens has a dQ and dK of almost nothing)
        assert _rel(x, y) < 1e-2 or (x.double() - y).abs().max() < 2e-2, "%s: %.2e" % (name, _rel(x, y))


@pytest.mark.parametrize("layout", ["cyclic", "contiguous"])
@pytest.mark.parametrize("causal", [True, False], ids=["causal", "full"])
def test_long_blocks(causal, layout):
    """Blocks of 46400 rows, whose tiles have more than 2^31 scores (dS of one would be more than 4 GiB): some rows and some
    keys, at the edges of the blocks and inside, against fp64."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d, grid as g2d
    T, side, H = 46400, 2, 64
    n, scale, gen = T * side, 0.125, torch.Generator(device="cuda")
    gen.manual_seed(37)
    print("long blocks", causal, layout, flush=True)
    Q, K, V, dO = (torch.randn(1, n, H, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    assert a2d._ext().grid_forward(Q, K, V, side, causal, layout == "cyclic", scale) is not None
    O, lse = g2d.forward(Q, K, V, side, causal, layout, scale)
    args = (Q, K, V, O, dO, lse, side, causal, layout == "cyclic", scale)
    assert a2d._ext().grid_backward(*args) is not None
    dQ, dK, dV = (x[0] for x in g2d.backward(Q, K, V, O, dO, lse, side, causal, layout, scale))
    q, k, v, g, o = (x[0].double() for x in (Q, K, V, dO, O))
    at = torch.tensor([0, 1, 31, 255, 256, 46339, 46340, 46341, T - 1, T, T + 1, 60001, n - 257, n - 2, n - 1], device="cuda")
    token = torch.arange(n, device="cuda")
    delta, ls = (g * o).sum(1), lse[0].double()
    S = q[at] @ k.t().contiguous() * scale                       # rows `at`
    if causal:
        S.masked_fill_(token[None, :] > at[:, None], -math.inf)
    assert (torch.logsumexp(S, 1) - ls[at]).abs().max() < 1e-4
    P = torch.exp(S - ls[at, None])
    assert _rel(O[0, at], P @ v) < 5e-3
    dS = P * (g[at] @ v.t().contiguous() - delta[at, None])
    # (the first row sees itself alone: its dQ is rounding noise)
    first = 1 if causal else 0
    assert _rel(dQ[at][first:], ((dS @ k) * scale)[first:]) < 1e-2
    S = k[at] @ q.t().contiguous() * scale                       # keys `at`
    if causal:
        S.masked_fill_(token[None, :] < at[:, None], -math.inf)
    P = torch.exp(S - ls[None, :])
    assert _rel(dV[at], P @ g) < 1e-2
    dS = P * (v[at] @ g.t().contiguous() - delta[None, :])
    assert _rel(dK[at], (dS @ q) * scale) < 1e-2
