"""The 16 x 16 tiles inside a wavefront's 32 rows and keys, at their edges: sizes one off multiples of 16, diagonals at every
offset within a tile, against fp64 on the GPU."""
import math

import pytest
import torch

import test_gpu_f32_kernels as f32
import test_gpu_small_rows as forward
from test_gpu_bwd_routes import _check

pytestmark = pytest.mark.gpu

# heads, kv_heads, nq, nkv, H, causal, q_off, sub-blocks, packed; dK/dV in 256 keys a workgroup, dS kept where H = 128
BACKWARD = [(600, 600, nq, nkv, H, causal, q_off, None, False)
            for nq, nkv, H, causal, q_off in [
                (15, 257, 128, False, 0), (17, 271, 128, True, 240), (33, 273, 128, True, 243), (47, 289, 128, True, 257),
                (49, 303, 96, True, 271), (16, 272, 80, True, 259), (31, 305, 80, False, 0), (65, 287, 64, True, 239)]]


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("case", BACKWARD, ids=lambda c: "%dx%dH%d_%d" % (c[2], c[3], c[4], c[6]))
def test_backward_tile_edges(case, keep):
    from paper_2503_15758_amd import binding as a2d
    heads, kvh, nq, nkv, H, causal, q_off = case[:7]
    route = a2d.tile_route(heads, nq, nkv, H, causal=causal, q_off=q_off, backward=True, ds_handover=keep)
    assert route["keys"] == 256, route
    assert ("bwd_dq_ds_kernel" in route["kernels"]) == (keep and H == 128), route
    _check(case, keep)


# the same with the rows of a workgroup that the route has to have
FORWARD = [(rows, (heads, heads, nq, nkv, H, causal, q_off, None, False, 2))
           for rows, heads, nq, nkv, H, causal, q_off in [
               (32, 2, 15, 17, 64, True, 2), (32, 3, 17, 47, 80, True, 30), (32, 2, 47, 271, 96, True, 223), (32, 1, 49, 303, 128, True, 257),
               (64, 150, 47, 129, 64, True, 81), (64, 40, 271, 303, 80, True, 33), (64, 40, 273, 287, 96, True, 15), (64, 40, 289, 305, 128, True, 16),
               (128, 40, 783, 801, 64, True, 17), (128, 80, 783, 801, 96, True, 15), (128, 80, 1009, 1041, 128, True, 31),
               (256, 64, 783, 801, 80, True, 33), (256, 64, 1009, 1041, 128, True, 17)]]


@pytest.mark.parametrize("rows,case", FORWARD, ids=lambda c: "%dx%dH%d_%d" % (c[2], c[3], c[4], c[6]) if isinstance(c, tuple) else c)
def test_forward_tile_edges(rows, case):
    from paper_2503_15758_amd import binding as a2d
    heads, _, nq, nkv, H, causal, q_off = case[:7]
    assert a2d.tile_route(heads, nq, nkv, H, causal=causal, q_off=q_off)["rows"] == rows
    forward.test_small_rows(case)


# walks of 64-key steps: from one step on, and (H = 128, from 14 steps of a key lane on) those whose wavefronts go through them in
# opposite phases; key lanes with unlike numbers of steps, sub-blocks that rows or all of a block see nothing of, in front, in between and behind
WALKS = [(form, (heads, heads, nq, nkv, H, causal, q_off, segs, packed, 2))
         for form, heads, nq, nkv, H, causal, q_off, segs, packed in [
             ((256, 1), 250, 250, 1, 128, False, 0, None, False), ((256, 1), 250, 250, 65, 80, True, -100, None, True),
             ((256, 1), 250, 250, 264, 96, True, 20, [(300, 64), (0, 130), (90, 70)], True),
             ((128, 2), 120, 256, 385, 128, False, 0, None, False), ((128, 1), 250, 128, 700, 64, True, -60, None, False),
             # opposite phases
             ((256, 1), 200, 250, 897, 128, False, 0, None, False), ((256, 1), 200, 250, 961, 128, True, 900, None, True),
             ((256, 1), 200, 250, 1218, 128, True, 1000, [(0, 65), (2000, 70), (90, 1018), (1100, 65)], False),
             ((256, 1), 200, 250, 1100, 128, True, 960, [(1300, 64), (0, 965), (990, 71)], False),
             ((128, 2), 120, 256, 1857, 128, False, 0, None, False), ((128, 2), 120, 256, 1921, 128, True, 1730, None, True),
             ((128, 2), 120, 256, 2000, 128, True, 1900, [(2200, 64), (0, 1800), (1850, 71), (3000, 65)], False)]]


@pytest.mark.parametrize("form,case", WALKS, ids=lambda c: "%dx%dH%d_%d" % (c[2], c[3], c[4], c[6]) if len(c) > 2 else "%dx%d" % c)
def test_forward_walks(form, case):
    from paper_2503_15758_amd import binding as a2d
    heads, _, nq, nkv, H, causal, q_off, segs = case[:8]
    route = a2d.tile_route(heads, nq, nkv, H, causal=causal, q_off=q_off, segments=segs)
    assert (route["rows"], route["lanes"], route["parts_q"]) == (*form, 1), route
    assert route["phased"] == (nkv >= (1857 if form[1] == 2 else 897)), route
    forward.test_small_rows(case)


@pytest.mark.parametrize("form,heads,nq,nkv,q_off", [((256, 1), 200, 250, 961, 900), ((128, 2), 120, 256, 1921, 1730)])
def test_phased_walk_continues_a_partial(form, heads, nq, nkv, q_off):
    """An accumulating call whose wavefronts are in opposite phases: it starts from the (N, m, l) of 70 keys, some rows' of none."""
    from paper_2503_15758_amd import binding as a2d
    H, scale = 128, 128 ** -0.5
    route = a2d.tile_route(heads, nq, nkv, H, causal=True, q_off=q_off)
    assert (route["rows"], route["lanes"], route["parts_q"], route["phased"]) == (*form, 1, True), route
    gen = torch.Generator(device="cuda").manual_seed(nkv)
    make = lambda n: torch.randn(heads, n, H, generator=gen, device="cuda").bfloat16()
    Q, K1, V1, K2, V2 = make(nq), make(70), make(70), make(nkv), make(nkv)
    at = torch.cat([torch.arange(70, device="cuda") + q_off + 100, torch.arange(nkv, device="cuda")])   # (the first rows see none of the 70)
    out = a2d.partial_fwd(Q, K1, V1, q_off, q_off + 100, True, scale)
    N, m, l = a2d.partial_fwd(Q, K2, V2, q_off, 0, True, scale, out=out, accumulate=True)
    k, v = torch.cat([K1, K2], 1).double(), torch.cat([V1, V2], 1).double()
    S = torch.bmm(Q.double(), k.transpose(1, 2).contiguous()) * scale
    S.masked_fill_(at[None, None, :] > torch.arange(nq, device="cuda")[None, :, None] + q_off, -math.inf)
    lse = torch.logsumexp(S, 2)
    O = torch.bmm(torch.exp(S - lse[..., None]), v)
    # (fp32 sums; P rounded to bf16, 2^-9 a term)
    assert (m.double() + l.double().log() - lse).abs().max() < 1e-4
    assert ((N / l[..., None]).double() - O).norm() / O.norm() < 5e-3


# fp32 backward: steps of 16 rows and keys, four key lanes; delta by a launch in front (the last four) and by the tiles themselves
F32 = [(1, 1, 1, 1, 64, False, 0, [(0, 1)]), (2, 2, 15, 17, 80, True, 2, [(0, 17)]), (3, 3, 17, 63, 96, True, 46, [(0, 63)]),
       (2, 1, 65, 129, 128, True, 64, [(0, 129)]), (4, 2, 33, 79, 64, True, 46, [(0, 30), (40, 49)]), (5, 5, 79, 65, 96, False, 0, [(0, 65)]),
       (60, 30, 513, 545, 64, True, 415, [(0, 545)]), (36, 36, 511, 767, 80, True, 255, [(0, 767)]),
       (34, 34, 497, 769, 96, True, 271, [(0, 769)]), (16, 8, 529, 639, 128, False, 0, [(0, 639)])]


@pytest.mark.parametrize("case", F32, ids=lambda c: "%dx%dH%d" % (c[2], c[3], c[4]))
def test_f32_tile_edges(case):
    from paper_2503_15758_amd import binding as a2d
    heads, kvh, nq, nkv, H, causal, q_off, segs = case
    route = a2d.tile_route(heads, nq, nkv, H, dtype=torch.float32, kv_heads=kvh, causal=causal, q_off=q_off, segments=segs, backward=True)
    assert ("delta_kernel" in route["kernels"]) == (nq > 400), route
    f32.test_f32_tiles_at_every_launch_shape(a2d, case)
