"""The merges at the edges of what a workgroup and a thread own: shares that end inside a row, a wavefront or the workgroup, every number
of groups a thread has, and the larger launches' form against the smaller ones'."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_close, np64

pytestmark = pytest.mark.gpu
DT = {"bf16": torch.bfloat16, "f32": torch.float32}


@pytest.fixture(scope="module")
def a2d():
    from paper_2503_15758_amd import binding
    binding.lib()
    return binding


def triples(k, rows, H, seed):
    g = torch.Generator().manual_seed(seed)
    N = [torch.randn(rows, H, generator=g) for _ in range(k)]
    m = [torch.randn(rows, generator=g) * 5 for _ in range(k)]
    l = [torch.rand(rows, generator=g) * 9 + 1 for _ in range(k)]
    m[-1][rows // 2] = -float("inf"); l[-1][rows // 2] = 0.0; N[-1][rows // 2] = 0.0
    return N, m, l


# (H, rows): 4-column groups a row 1, 16, 17, 20, 32, 256; shares are of 256, 512 and 1024 groups
@pytest.mark.parametrize("H,rows", [(4, 255), (4, 1025), (64, 16), (64, 33), (68, 61), (80, 13), (80, 103), (128, 1), (128, 97), (1024, 5)])
@pytest.mark.parametrize("k,out", [(2, "bf16"), (3, "f32"), (4, "bf16"), (6, "bf16"), (8, "f32"), (16, "bf16"), (20, "f32")])
def test_shares(a2d, H, rows, k, out):
    N, m, l = triples(k, rows, H, 41 * k + rows)
    dN, dm, dl = ([x.cuda() for x in t] for t in (N, m, l))
    O, lse = a2d.fix(dN, dm, dl, DT[out])
    Or, lr = oracle.fix([np64(x) for x in N], [np64(x) for x in m], [np64(x) for x in l])
    assert_close(O, Or, DT[out], "fix O")
    assert_close(lse, lr, torch.float32, "fix lse", rel=False)
    s = a2d.fix_bwd([(x / k ** 0.5) for x in dN], torch.float32)
    assert_close(s, sum(np64(x) for x in N) / k ** 0.5, torch.float32, "sum")
    n, lw = a2d.fix_norm([x.to(DT[out]) for x in dN], dm, torch.float32)
    nr, nl = oracle.fix_norm([np64(x.to(DT[out])) for x in N], [np64(x) for x in m])
    assert_close(n, nr, torch.float32, "fix_norm O")
    assert_close(lw, nl, torch.float32, "fix_norm lse", rel=False)


@pytest.mark.parametrize("k", [8, 16])
def test_large_launches_as_small_ones(a2d, k):
    """From 2^21 column groups on a thread has another number of them; the sums are the same, in the same order."""
    rows, H, cut = 65536 + 77, 128, 40000
    g = torch.Generator(device="cuda").manual_seed(k)
    N = [torch.randn(rows, H, generator=g, device="cuda") for _ in range(k)]
    m = [torch.randn(rows, generator=g, device="cuda") * 5 for _ in range(k)]
    l = [torch.rand(rows, generator=g, device="cuda") + 1 for _ in range(k)]
    cuts = lambda t: ([x[:cut].contiguous() for x in t], [x[cut:].contiguous() for x in t])
    (Na, Nb), (ma, mb), (la, lb) = cuts(N), cuts(m), cuts(l)
    for whole, a, b in ((a2d.fix(N, m, l), a2d.fix(Na, ma, la), a2d.fix(Nb, mb, lb)),
                        (a2d.attnfix(N, m, l), a2d.attnfix(Na, ma, la), a2d.attnfix(Nb, mb, lb)),
                        ((a2d.fix_bwd(N),), (a2d.fix_bwd(Na),), (a2d.fix_bwd(Nb),))):
        for w, x, y in zip(whole, a, b):
            assert torch.equal(w, torch.cat([x, y]))
