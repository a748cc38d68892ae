"""Causal tiles of many heads, whose workgroups go out by size in chunks of heads: chunks of four, equal larger ones,
heads left over from eight XCDs and from a chunk - every block of every head is written once, against fp64 on the GPU."""
import math

import pytest
import torch

from test_gpu_split_walks import _rel

pytestmark = pytest.mark.gpu

# heads, kv_heads, nq, nkv, H: many query blocks (forward, dQ) or many key blocks (dK / dV)
CASES = [
    (256, 256, 1600, 40, 64),      # 32 heads an XCD, seven turns: chunks of four
    (259, 259, 40, 1600, 64),      # 32 heads an XCD: two equal chunks of key blocks, three heads left over
    (296, 148, 1450, 33, 80),      # grouped heads: 18 units an XCD, two equal chunks
    (227, 227, 1793, 24, 128),     # 28 heads an XCD, a ragged eighth block, three heads left over
    (136, 136, 1300, 70, 96),      # 17 heads an XCD: 9 and 8
    (168, 168, 70, 1300, 128),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dq%dkv_%dx%dH%d" % c)
def test_every_block_once(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, kvh, nq, nkv, H = case
    scale, gen = 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(3)
    print("order case", case, flush=True)
    make = lambda h, n: torch.randn(h, n, H, generator=gen, device="cuda").to(torch.bfloat16)
    Q, dO, K, V = make(heads, nq), make(heads, nq), make(kvh, nkv), make(kvh, nkv)
    q, g = Q.double(), dO.double()
    k, v = (x.double().repeat_interleave(heads // kvh, 0) for x in (K, V))
    prod = lambda x, y: torch.bmm(x, y.transpose(1, 2).contiguous())
    hidden = torch.arange(nkv, device="cuda")[None, :] > torch.arange(nq, device="cuda")[:, None]
    S = (prod(q, k) * scale).masked_fill(hidden, -math.inf)
    lse = torch.logsumexp(S, 2)
    P = torch.exp(S - lse[..., None])
    O = torch.bmm(P, v)
    Os = O.to(torch.bfloat16)
    dS = P * (prod(g, v) - (g * Os.double()).sum(2)[..., None])
    fold = lambda x: x.view(kvh, heads // kvh, nkv, H).sum(1)
    ref = (torch.bmm(dS, k) * scale, fold(torch.bmm(dS.transpose(1, 2).contiguous(), q)) * scale,
           fold(torch.bmm(P.transpose(1, 2).contiguous(), g)))
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    N, m, l = a2d.partial_fwd(Q, K, V, 0, 0, True, scale, out=(nan(heads, nq, H), nan(heads, nq), nan(heads, nq)))
    assert _rel(N / l[..., None], O) < 1e-2 and _rel(m + torch.log(l), lse) < 1e-3
    for keep in (False, True):
        out = (nan(heads, nq, H), nan(kvh, nkv, H), nan(kvh, nkv, H))
        got = a2d.partial_bwd(Q, K, V, Os, dO, lse.float(), 0, 0, True, scale, out=out, ds_handover=keep)
        for name, x, y in zip(("dQ", "dK", "dV"), got, ref):
            assert _rel(x, y) < 1e-2, "%s: %.2e (keep %d)" % (name, _rel(x, y), keep)
