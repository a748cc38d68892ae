"""The backward's routes - one launch for dQ and dK / dV; dQ, then dK / dV; dK / dV leaving dS, then dQ - at the edges of
their blocks, against fp64 on the GPU.  A call of at most six turns of the chip (256-row and 256-key blocks over 256 compute
units) goes out in one launch, one of more in launches of its own, at H = 128 with dS kept where that is allowed."""
import math

import pytest
import torch

from test_gpu_split_walks import _rel

pytestmark = pytest.mark.gpu
BF = torch.bfloat16

# heads, kv_heads, nq, nkv, H, causal, q_off, sub-blocks (None: one), packed
ONE = [
    (1, 1, 1, 1, 64, False, 0, None, False),
    (3, 3, 31, 65, 80, True, 40, None, False),
    (2, 1, 33, 129, 96, True, 100, None, True),              # grouped heads, O and dO of different strides
    (5, 5, 129, 127, 128, False, 0, None, True),
    (6, 2, 257, 255, 128, True, 0, None, False),
    (4, 2, 300, 513, 64, True, 250, [(30, 200), (300, 313)], True),
    (90, 90, 256, 700, 128, True, 444, None, False),         # 256 keys a workgroup, delta by a launch of its own
    (70, 35, 520, 300, 96, False, 0, None, True),
    (2, 2, 90, 3000, 80, True, 2910, None, False),           # dQ in parts, its workgroups first
    (2, 2, 3000, 90, 80, True, 0, None, False),              # dK / dV in parts
]
MANY = [
    (800, 800, 33, 129, 128, True, 96, None, False),
    (800, 400, 256, 256, 128, True, 0, None, True),
    (420, 420, 257, 300, 128, True, 60, [(0, 128), (200, 172)], False),
    (790, 790, 100, 60, 128, False, 0, None, False),         # few keys: 128 a workgroup
    (800, 800, 65, 70, 80, True, 5, None, False),
]


def _check(case, keep):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, kvh, nq, nkv, H, causal, q_off, segs, packed = case
    scale, gen = 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(31)
    print("route case", case, keep, flush=True)

    def make(h, n):
        if packed:
            return torch.randn(n, h, H, generator=gen, device="cuda").to(BF).permute(1, 0, 2)
        return torch.randn(h, n, H, generator=gen, device="cuda").to(BF)
    Q, dO, K, V = make(heads, nq), make(heads, nq), make(kvh, nkv), make(kvh, nkv)
    q, g = Q.double(), dO.double()
    k, v = (x.double().repeat_interleave(heads // kvh, 0) for x in (K, V))
    pos = torch.cat([torch.arange(r, device="cuda") + o for o, r in segs or [(0, nkv)]])
    prod = lambda x, y: torch.bmm(x.contiguous(), y.transpose(1, 2).contiguous())
    S = prod(q, k) * scale
    if causal:
        S.masked_fill_(pos[None, None, :] > torch.arange(nq, device="cuda")[None, :, None] + q_off, -math.inf)
    lse = torch.logsumexp(S, 2)
    seen = lse > -math.inf
    P = torch.exp(S - torch.where(seen, lse, torch.zeros_like(lse))[..., None]) * seen[..., None]
    O = torch.bmm(P, v.contiguous())
    Os = O.to(BF)                                            # (plain also where dO is packed)
    dS = P * (prod(g, v) - (g * Os.double()).sum(2)[..., None])
    fold = lambda x: x.view(kvh, heads // kvh, nkv, H).sum(1)
    ref = (torch.bmm(dS, k.contiguous()) * scale, fold(torch.bmm(dS.transpose(1, 2).contiguous(), q.contiguous())) * scale,
           fold(torch.bmm(P.transpose(1, 2).contiguous(), g.contiguous())))
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    out = (nan(heads, nq, H), nan(kvh, nkv, H), nan(kvh, nkv, H))
    args = (Q, K, V, Os, dO, lse.float(), q_off, 0, causal, scale)
    got = a2d.partial_bwd(*args, out=out, segments=segs, ds_handover=keep)
    for name, x, y in zip(("dQ", "dK", "dV"), got, ref):
        # P and dS rounded to bf16: 2^-9 a term (one key: dQ and dK are rounding noise beside dO, V of size 1)
        assert _rel(x, y) < 1e-2 or (x.double() - y).abs().max() < 2e-2, "%s: %.2e" % (name, _rel(x, y))
    again = a2d.partial_bwd(*args, segments=segs, ds_handover=keep)
    assert all(torch.equal(x, y) for x, y in zip(got, again))
    base = torch.randn(heads, nq, H, generator=gen, device="cuda")
    acc = a2d.partial_bwd(*args, out=(base.clone(), *(torch.empty_like(x) for x in got[1:])), segments=segs, accumulate=True,
                          ds_handover=keep)
    assert torch.equal(acc[1], got[1]) and torch.equal(acc[2], got[2])
    assert (acc[0] - base - got[0]).abs().max() < 1e-5 * (1 + got[0].abs().max())
    return got


@pytest.mark.parametrize("case", ONE + MANY, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_routes(case):
    recomputed, kept = _check(case, False), _check(case, True)
    assert torch.equal(recomputed[1], kept[1]) and torch.equal(recomputed[2], kept[2])
    assert _rel(kept[0], recomputed[0].double()) < 1e-2 or (kept[0] - recomputed[0]).abs().max() < 2e-2


# heads, nq, nkv: few rows; in one launch of 128 and of 256 keys a workgroup; dQ, then dK / dV, or with dS kept
DELTA = [(8, 40, 33), (6, 300, 500), (60, 700, 129), (90, 256, 700), (800, 33, 129)]


@pytest.mark.parametrize("H", [64, 80, 96, 128])
@pytest.mark.parametrize("case", DELTA, ids=lambda c: "%dx%dx%d" % c)
def test_one_delta_for_all_gradients(case, H):
    """dQ and dK use the same bits of delta = rowsum(dO o O), shown by products that cancel, so that its value is that of the
    order of its sums.  Row 0 sees key 0 alone, with probability 1 (q.k scale = lse = 4, a power of two: no rounding); the other
    rows' probabilities and V are zero, so that in 64 columns dQ of row 0 and dK of key 0 are both -scale bf16(delta)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, nq, nkv = case
    scale, gen, some = 2.0 ** -4, torch.Generator(device="cuda"), 0
    print("delta case", case, H, flush=True)
    make = lambda n: torch.randn(heads, n, H, generator=gen, device="cuda")
    Q, K = torch.ones(heads, nq, H, device="cuda", dtype=BF), torch.ones(heads, nkv, H, device="cuda", dtype=BF)
    Q[..., 64:] = 0
    V = torch.zeros_like(K)
    lse = torch.full((heads, nq), 1e30, device="cuda")
    lse[:, 0] = 64 * scale
    for seed in range(4):
        gen.manual_seed(seed)
        dO, O = make(nq).to(BF), (make(nq) * 2.0 ** torch.randint(-20, 20, (heads, nq, H), generator=gen, device="cuda")).to(BF)
        O[..., H // 2:] = -O[..., :H // 2]                       # exact sum: zero
        dO[..., H // 2:] = dO[..., :H // 2]
        order = torch.randperm(H, generator=gen, device="cuda")
        O, dO = O[..., order].contiguous(), dO[..., order].contiguous()
        for keep in (False, True):
            dQ, dK, _ = a2d.partial_bwd(Q, K, V, O, dO, lse, 0, 0, True, scale, ds_handover=keep)
            some += int((dQ[:, 0, 0] != 0).sum())
            assert not dQ[:, 1:].any()
            assert torch.equal(dQ[:, 0, :64], dK[:, 0, :64]), "dQ %s, dK %s" % (dQ[:4, 0, 0], dK[:4, 0, 0])
    assert some > 0


@pytest.mark.parametrize("H", [64, 80, 96, 128])
def test_no_memory_for_a_ds_that_is_not_kept(H):
    """ds_handover without a workspace: memory for dS (64 MiB here) is taken where it may be kept, at H = 128."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, n = 8, 2048
    make = lambda: torch.randn(heads, n, H, device="cuda").to(BF)
    Q, K, V, O, dO = (make() for _ in range(5))
    lse = torch.full((heads, n), 8.0, device="cuda")
    took = {}
    for keep in (False, True):
        a2d.partial_bwd(Q, K, V, O, dO, lse, ds_handover=keep)
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        a2d.partial_bwd(Q, K, V, O, dO, lse, ds_handover=keep)
        took[keep] = torch.cuda.max_memory_allocated() - before
    assert (took[True] - took[False] >= 2 * heads * n * n) == (H == 128) and (H == 128 or took[True] == took[False]), took


@pytest.mark.parametrize("H", [64, 80, 96, 128])
def test_delta_against_64_bits(H):
    """delta of whole rows as delta_kernel leaves it in the workspace, from products of bf16 pairs: against 64 bits, and against
    unpacked fp32 multiply-adds in the same order."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, nq, nkv = 90, 256, 700
    assert a2d.tile_route(heads, nq, nkv, H, causal=True, q_off=444, backward=True)["kernels"][0] == "delta_kernel"
    gen = torch.Generator(device="cuda")
    gen.manual_seed(41)
    make = lambda n: torch.randn(heads, n, H, generator=gen, device="cuda").to(BF)
    Q, K, V, O, dO = make(nq), make(nkv), make(nkv), make(nq), make(nq)
    lse = torch.full((heads, nq), 7.0, device="cuda")
    ws = torch.empty(a2d.workspace_bytes(a2d.tile_desc(Q, K, 444, 0, True, None), a2d.OP_PARTIAL_BWD), dtype=torch.uint8,
                     device="cuda")
    a2d.partial_bwd(Q, K, V, O, dO, lse, 444, 0, True, workspace=ws)
    got = ws[:4 * heads * nq].view(torch.float32).view(heads, nq).double()
    prod = O.double() * dO.double()                              # (exact; in fp32 too: 16 bits of mantissa)
    exact, size = prod.sum(2), prod.abs().sum(2)
    chunks = prod.float().view(heads, nq, H // 8, 8)
    t = torch.zeros(heads, nq, 16, device="cuda")
    for e in range(8):
        t[..., :H // 8] += chunks[..., e]
    for o in (1, 2, 4, 8):
        t = t + t[..., torch.arange(16, device="cuda") ^ o]
    plain = t[..., 0].double()
    off, plain_off = ((x - exact).abs() / size for x in (got, plain))
    print("H %d: mean error of the magnitudes' sum %.2e, unpacked %.2e" % (H, off.mean(), plain_off.mean()), flush=True)
    # eight products and four exchanges: at most twelve roundings of a partial sum
    assert off.max() < 12 * 2.0 ** -24 and off.mean() <= 1.05 * plain_off.mean()
