"""Scores that overflow where the mask hides them: q.k of a hidden pair is infinite (every input finite), inside a
32 x 32 block that other rows see, and between the last row - which the kernels re-read in place of rows past the end -
and a key no row sees.  Such pairs have no part in the result, whichever form of the dK/dV kernel a call takes."""
import math

import pytest
import torch

from test_gpu_split_walks import _rel

pytestmark = pytest.mark.gpu

# dtype, heads, H: tiles of 100 x 300, which take, from few heads to many, 32 keys per workgroup, 128 and 256 in one launch with
# dQ, 128 in a launch of their own, 256 in one (at H = 128 with dS kept where allowed)
CASES = [("bf16", 4, 128), ("bf16", 90, 128), ("bf16", 90, 80), ("f32", 4, 64),
         ("bf16", 150, 128), ("bf16", 150, 96), ("bf16", 150, 80), ("bf16", 150, 64), ("bf16", 170, 64),
         ("bf16", 600, 128), ("bf16", 600, 96), ("bf16", 600, 80), ("bf16", 600, 64)]
NQ, NKV, OFF = 100, 300, 192                       # row i sees the keys up to i + OFF
BIG = 1e20


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_%dheads_H%d" % c)
def test_hidden_overflow(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    dtype, heads, H = case
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tol = 1e-2 if dtype == "bf16" else 2e-5
    scale, gen = 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(7)
    print("hidden case", case, flush=True)
    make = lambda n: torch.randn(heads, n, H, generator=gen, device="cuda").to(dt)
    Q, dO, K, V = make(NQ), make(NQ), make(NKV), make(NKV)
    Q[..., :2] = 0                                 # (the two columns meet in hidden pairs only)
    K[..., :2] = 0
    Q[:, 32:48, 0] = BIG                           # these rows see all of their diagonal block but its last key
    K[:, OFF + 63, 0] = BIG
    Q[:, -1, 1] = BIG
    K[:, NQ + OFF + 3, 1] = BIG                    # behind the last key that any row sees
    q, k, v, g = Q.double(), K.double(), V.double(), dO.double()
    prod = lambda x, y: torch.bmm(x, y.transpose(1, 2).contiguous())
    hidden = torch.arange(NKV, device="cuda")[None, :] > torch.arange(NQ, device="cuda")[:, None] + OFF
    S = (prod(q, k) * scale).masked_fill(hidden, -math.inf)
    assert float((prod(q, k) * hidden).abs().max()) > 3.5e38 and float(S.max()) < 100
    lse = torch.logsumexp(S, 2)
    P = torch.exp(S - lse[..., None])
    O = torch.bmm(P, v)
    Os = O.to(dt)
    dS = P * (prod(g, v) - (g * Os.double()).sum(2)[..., None])
    ref = (torch.bmm(dS, k) * scale, torch.bmm(dS.transpose(1, 2).contiguous(), q) * scale,
           torch.bmm(P.transpose(1, 2).contiguous(), g))
    N, m, l = a2d.partial_fwd(Q, K, V, OFF, 0, True, scale)
    assert _rel(N / l[..., None], O) < tol and _rel(m + torch.log(l), lse) < tol
    for keep in ((False, True) if dtype == "bf16" else (False,)):
        got = a2d.partial_bwd(Q, K, V, Os, dO, lse.float(), OFF, 0, True, scale, ds_handover=keep)
        for name, x, y in zip(("dQ", "dK", "dV"), got, ref):
            assert bool(torch.isfinite(x).all()), "%s is not finite (keep %d)" % (name, keep)
            assert _rel(x[..., 2:], y[..., 2:]) < tol, "%s: %.2e (keep %d)" % (name, _rel(x[..., 2:], y[..., 2:]), keep)
