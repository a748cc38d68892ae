"""dK/dV in workgroups of 256 keys, which calls with many key blocks take: ragged last blocks (a wavefront with one
key, wavefronts with none), grouped heads, sub-blocks, rows and keys that see nothing, one query row, both dQ paths,
against fp64 on the GPU."""
import math

import pytest
import torch

from test_gpu_split_walks import _rel

pytestmark = pytest.mark.gpu

# heads, kv_heads, nq, nkv, H, causal, q_off, segments (kv_off, rows)
# 256 keys a workgroup, in one launch with dQ ...
CASES = [
    (150, 150, 100, 300, 128, False, 0, [(0, 300)]),
    (120, 120, 333, 257, 96, True, 0, [(0, 257)]),
    (340, 170, 65, 289, 80, True, 200, [(0, 64), (100, 225)]),
    (120, 120, 1, 301, 64, False, 0, [(0, 301)]),
    (176, 88, 70, 512, 64, True, 450, [(30, 512)]),           # the last keys are seen by no row
    (45, 45, 90, 641, 128, True, 300, [(300, 128), (0, 513)]),  # first rows see nothing of the first sub-block
    # ... and in a launch of their own, at H = 128 with dS kept too
    (600, 600, 100, 300, 128, False, 0, [(0, 300)]),
    (600, 600, 1, 301, 128, False, 0, [(0, 301)]),
    (400, 400, 333, 257, 96, True, 0, [(0, 257)]),
    (500, 250, 65, 289, 80, True, 200, [(0, 64), (100, 225)]),
    (600, 600, 1, 301, 64, False, 0, [(0, 301)]),
    (500, 250, 90, 321, 128, True, 150, [(200, 128), (0, 193)]),
]
# 128 keys a workgroup
NARROW = [
    (90, 90, 100, 300, 128, False, 0, [(0, 300)]),
    (90, 90, 333, 257, 96, True, 0, [(0, 257)]),
    (180, 90, 65, 289, 80, True, 200, [(0, 64), (100, 225)]),
    (90, 90, 1, 301, 64, False, 0, [(0, 301)]),
]


@pytest.mark.parametrize("case", CASES + NARROW, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_wide_key_blocks(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, kvh, nq, nkv, H, causal, q_off, segs = case
    scale, gen = 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(11)
    print("wide case", case, flush=True)
    make = lambda h, n: torch.randn(h, n, H, generator=gen, device="cuda").to(torch.bfloat16)
    Q, dO, K, V = make(heads, nq), make(heads, nq), make(kvh, nkv), make(kvh, nkv)
    q, g = Q.double(), dO.double()
    k, v = (x.double().repeat_interleave(heads // kvh, 0) for x in (K, V))
    pos = torch.cat([torch.arange(r, device="cuda") + o for o, r in segs])
    prod = lambda x, y: torch.bmm(x, y.transpose(1, 2).contiguous())
    S = prod(q, k) * scale
    if causal:
        S.masked_fill_(pos[None, None, :] > torch.arange(nq, device="cuda")[None, :, None] + q_off, -math.inf)
    lse = torch.logsumexp(S, 2)
    seen = lse > -math.inf
    P = torch.exp(S - torch.where(seen, lse, torch.zeros_like(lse))[..., None]) * seen[..., None]
    O = torch.bmm(P, v)
    Os = O.to(torch.bfloat16)
    dS = P * (prod(g, v) - (g * Os.double()).sum(2)[..., None])
    fold = lambda x: x.view(kvh, heads // kvh, nkv, H).sum(1)
    ref = (torch.bmm(dS, k) * scale, fold(torch.bmm(dS.transpose(1, 2).contiguous(), q)) * scale,
           fold(torch.bmm(P.transpose(1, 2).contiguous(), g)))
    out = {}
    for keep in (False, True):
        out[keep] = a2d.partial_bwd(Q, K, V, Os, dO, lse.float(), q_off, 0, causal, scale, segments=segs, ds_handover=keep)
        for name, x, y in zip(("dQ", "dK", "dV"), out[keep], ref):
            assert _rel(x, y) < 1e-2, "%s: %.2e (keep %d)" % (name, _rel(x, y), keep)
    assert torch.equal(out[False][1], out[True][1]) and torch.equal(out[False][2], out[True][2])
