"""Forward tiles of few rows: 32 (64) query rows a workgroup, whose eight (four) key lanes share the walk by slabs of 32 keys and
merge their (N, m, l) inside the kernel.  At the edges of rows, slabs and sub-blocks, against fp64 on the GPU; the three forms of
the call: plain, accumulating, normalised."""
import math

import pytest
import torch

from test_gpu_split_walks import _rel

pytestmark = pytest.mark.gpu
BF = torch.bfloat16

# heads, kv_heads, nq, nkv, H, causal, q_off, sub-blocks (None: one), packed, sigma
# 32 rows a workgroup
ROWS32 = [
    (1, 1, 1, 1, 128, False, 0, None, False, 1),
    (3, 3, 31, 33, 64, False, 0, None, True, 1),             # two of the eight wavefronts have keys
    (2, 1, 32, 255, 80, True, 230, None, False, 1),
    (4, 2, 33, 256, 96, True, 250, None, True, 4),           # one slab each; a row beyond the block
    (5, 5, 65, 257, 128, True, 200, None, False, 6),         # one key beyond the first round
    (2, 2, 100, 300, 64, True, -40, None, False, 1),         # rows that see nothing
    (8, 2, 90, 700, 128, True, 640, [(3, 31), (64, 1), (65, 300), (600, 368)], True, 3),
    (3, 1, 64, 513, 80, True, 500, [(0, 33), (400, 480)], False, 1),
    (17, 17, 480, 545, 128, False, 0, None, False, 8),
    (30, 10, 250, 1030, 96, True, 780, None, True, 1),
    (1, 1, 40, 9000, 128, False, 0, None, False, 2),         # a walk worth sharing between workgroups too
]
# 64 rows
ROWS64 = [
    (40, 40, 300, 300, 128, False, 0, None, False, 2),
    (40, 20, 290, 333, 80, True, 60, None, True, 1),
    (20, 10, 610, 129, 64, True, -30, None, False, 3),       # rows that see nothing; one key in the second round
    (24, 6, 610, 129, 80, True, -30, None, True, 1),
    (44, 11, 250, 500, 96, True, 300, [(0, 31), (40, 1), (90, 300), (420, 168)], True, 1),
    (44, 11, 305, 82, 128, True, -101, None, False, 2),      # a block whose rows all see nothing; lanes without keys
    (9, 9, 1375, 83, 64, True, -288, None, True, 1),
    (50, 50, 284, 80, 64, False, 0, None, False, 1),         # a lane without keys, one with half a slab
    (8, 2, 1192, 93, 128, False, 0, None, True, 4),
    (148, 74, 36, 96, 96, False, 0, None, False, 1),         # rows in the second of the two row groups: four
]
# fewer keys than two rounds: 128 rows, in pairs of workgroups
PAIRS = [
    (26, 13, 610, 129, 64, True, -30, None, False, 3),
    (70, 70, 225, 31, 128, False, 0, None, True, 1),
]
CASES = ROWS32 + ROWS64 + PAIRS


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_small_rows(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding as a2d
    heads, kvh, nq, nkv, H, causal, q_off, segs, packed, sigma = case
    scale, gen = 1.0 / math.sqrt(H), torch.Generator(device="cuda")
    gen.manual_seed(17)
    print("small case", case, flush=True)

    def make(h, n, s=1.0):
        shape = (n, h, H) if packed else (h, n, H)
        x = (torch.randn(shape, generator=gen, device="cuda") * s).to(BF)
        return x.permute(1, 0, 2) if packed else x
    Q, K, V = make(heads, nq, sigma), make(kvh, nkv), make(kvh, nkv)
    K2, V2 = make(kvh, 70), make(kvh, 70)
    pos = torch.cat([torch.arange(r, device="cuda") + o for o, r in segs or [(0, nkv)]])
    pos2 = torch.arange(70, device="cuda") + q_off

    def reference(K, V, pos):
        k, v = (x.double().repeat_interleave(heads // kvh, 0).contiguous() for x in (K, V))
        S = torch.bmm(Q.double().contiguous(), k.transpose(1, 2).contiguous()) * scale
        if causal:
            S.masked_fill_(pos[None, None, :] > torch.arange(nq, device="cuda")[None, :, None] + q_off, -math.inf)
        m = S.max(2).values
        P = torch.exp(S - torch.where(m > -math.inf, m, torch.zeros_like(m))[..., None])
        return torch.bmm(P, v), m, P.sum(2)

    def check(got, ref):
        N, m, l = ref
        seen = m > -math.inf
        assert torch.equal(got[1] == -math.inf, ~seen) and (got[1].double() - m)[seen].abs().max() < 1e-4 * sigma * sigma
        # l: fp32 sums; N: P rounded to bf16, 2^-9 a term
        assert _rel(got[2], l) < 1e-4 * sigma * sigma and _rel(got[0], N) < 5e-3
        assert not got[0][~seen].any() and not got[2][~seen].any()

    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    first = reference(K, V, pos)
    got = a2d.partial_fwd(Q, K, V, q_off, 0, causal, scale, out=(nan(heads, nq, H), nan(heads, nq), nan(heads, nq)), segments=segs)
    check(got, first)
    assert all(torch.equal(x, y) for x, y in zip(got, a2d.partial_fwd(Q, K, V, q_off, 0, causal, scale, segments=segs)))

    norm = a2d.partial_fwd_norm(Q, K, V, q_off, 0, causal, scale, segments=segs)
    seen = first[1] > -math.inf
    O = torch.where(seen[..., None], first[0] / first[2].clamp_min(1e-300)[..., None], torch.zeros_like(first[0]))
    assert _rel(norm[0], O) < 8e-3 and torch.equal(norm[1] == -math.inf, ~seen)
    assert (norm[1].double() - (first[1] + torch.log(first[2])))[seen].abs().max() < 2e-4 * sigma * sigma

    second = reference(K2, V2, pos2)                         # one block more, onto the first
    m = torch.maximum(first[1], second[1])
    w = [torch.where(p[1] > -math.inf, torch.exp(p[1] - torch.where(m > -math.inf, m, torch.zeros_like(m))), torch.zeros_like(m))
         for p in (first, second)]
    both = (first[0] * w[0][..., None] + second[0] * w[1][..., None], m, first[2] * w[0] + second[2] * w[1])
    check(a2d.partial_fwd(Q, K2, V2, q_off, q_off, causal, scale, out=got, accumulate=True), both)
