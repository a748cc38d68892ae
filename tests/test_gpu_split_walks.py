"""Few row blocks against a long walk: calls whose walks are shared by several workgroups and merged (through scratch
memory the torch layer offers), and head counts whose blocks are spread over the XCDs, against fp64 on the GPU.
Every call form, ragged sizes, sub-blocks, rows and whole blocks that see no key, empty shares."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

# dtype, heads, kv_heads, nq, nkv, H, causal, q_off, segments (kv_off, rows)
CASES = [
    ("bf16", 1, 1, 130, 5000, 128, False, 0, [(0, 5000)]),
    ("bf16", 3, 1, 65, 3333, 96, True, 3200, [(0, 1000), (1100, 2333)]),      # parts cross the sub-blocks
    ("bf16", 2, 2, 400, 2900, 64, True, 40, [(0, 64), (300, 2836)]),          # most parts see nothing
    ("bf16", 9, 3, 33, 1400, 80, True, 0, [(0, 700), (700, 700)]),
    ("bf16", 5, 5, 4200, 140, 128, True, 0, [(100, 140)]),                    # long walk of dK / dV; first rows see no key
    ("bf16", 8, 1, 600, 90, 64, False, 0, [(0, 90)]),                         # ... over the heads of a group
    ("f32", 1, 1, 50, 1500, 128, True, 1450, [(0, 700), (700, 800)]),
    ("f32", 3, 3, 900, 70, 80, True, 0, [(0, 70)]),
    ("f32", 6, 2, 40, 333, 96, False, 0, [(0, 333)]),
]


def _rel(x, y):
    return float((x.double() - y).norm() / y.norm().clamp_min(1e-30))


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_%dq%dkv_%dx%dH%d_%s" % (c[0], *c[1:6], "causal" if c[6] else "full"))
def test_split_walks(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    dtype, heads, kvh, nq, nkv, H, causal, q_off, segs = case
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tol = 1e-2 if dtype == "bf16" else 2e-5
    scale, gen = 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(5)
    print("split case", case, flush=True)
    make = lambda h, n: torch.randn(h, n, H, generator=gen, device="cuda").to(dt)
    Q, dO, K, V = make(heads, nq), make(heads, nq), make(kvh, nkv), make(kvh, nkv)
    q, g = Q.double(), dO.double()
    k, v = (x.double().repeat_interleave(heads // kvh, 0) for x in (K, V))
    pos = torch.cat([torch.arange(r, device="cuda") + o for o, r in segs])
    S = torch.stack([torch.mm(q[h], k[h].t().contiguous()) for h in range(heads)]) * scale
    if causal:
        S.masked_fill_(pos[None, None, :] > torch.arange(nq, device="cuda")[None, :, None] + q_off, -math.inf)
    m = S.amax(2)
    seen = m > -math.inf
    P = torch.exp(S - m.nan_to_num(neginf=0.0)[..., None])
    l, N = P.sum(2), torch.bmm(P, v)
    # forward: plain, normalised, accumulated onto itself (N and l double)
    N1, m1, l1 = a2d.partial_fwd(Q, K, V, q_off, 0, causal, scale, segments=segs)
    for _ in range(2):
        assert all(torch.equal(x, y) for x, y in zip((N1, m1, l1), a2d.partial_fwd(Q, K, V, q_off, 0, causal, scale, segments=segs)))
    assert torch.equal(m1 > -math.inf, seen) and bool((l1[~seen] == 0).all()) and bool((N1[~seen] == 0).all())
    assert _rel(N1, N) < tol and _rel(l1, l) < tol and _rel(m1[seen], m[seen]) < tol
    On, ln = a2d.partial_fwd_norm(Q, K, V, q_off, 0, causal, scale, segments=segs)
    O, lse = N / l.clamp_min(1e-300)[..., None], m + torch.log(l)
    assert _rel(On, O) < tol and _rel(ln[seen], lse[seen]) < tol and bool((ln[~seen] == -math.inf).all())
    out = tuple(x.clone() for x in (N1, m1, l1))
    a2d.partial_fwd(Q, K, V, q_off, 0, causal, scale, out=out, segments=segs, accumulate=True)
    assert _rel(out[0], 2 * N) < tol and _rel(out[2], 2 * l) < tol
    # backward from the saved O and lse, both dQ paths, and dQ accumulated
    Os, ls = O.to(dt), lse.float()
    D = (g * Os.double()).sum(2)
    W = torch.exp(S - torch.where(seen, ls.double(), torch.zeros_like(lse))[..., None]) * seen[..., None]
    dS = W * (torch.stack([torch.mm(g[h], v[h].t().contiguous()) for h in range(heads)]) - D[..., None])
    fold = lambda x: x.view(kvh, heads // kvh, nkv, H).sum(1)
    ref = (torch.bmm(dS, k) * scale, fold(torch.stack([torch.mm(dS[h].t().contiguous(), q[h]) for h in range(heads)])) * scale,
           fold(torch.stack([torch.mm(W[h].t().contiguous(), g[h]) for h in range(heads)])))
    aligned = all(sum(r for _, r in segs[:i]) % 64 == 0 for i in range(len(segs)))
    for keep in ((False, True) if dtype == "bf16" and aligned else (False,)):
        for split in ((False, True) if kvh != heads else (False,)):
            got = a2d.partial_bwd(Q, K, V, Os, dO, ls, q_off, 0, causal, scale, segments=segs, ds_handover=keep, split_groups=split)
            for name, x, y in zip(("dQ", "dK", "dV"), got, ref):
                assert _rel(x, y) < tol, "%s: %.2e (keep %d split %d)" % (name, _rel(x, y), keep, split)
    acc = tuple(x.clone() for x in got)
    a2d.partial_bwd(Q, K, V, Os, dO, ls, q_off, 0, causal, scale, segments=segs, out=acc, accumulate=True)
    assert _rel(acc[0], 2 * ref[0]) < tol and _rel(acc[1], ref[1]) < tol
