"""fp32 tile kernels at each launch shape, against the fp64 oracle: 16-row and (forward) 32-row workgroups, each of
four key lanes, at ragged sizes, for every head size, with masks and grouped heads.
(The small cases of test_gpu_parity.py all take 16 rows.)"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2503_15758_amd import synth
from helpers import assert_close, np64

pytestmark = pytest.mark.gpu
F32 = torch.float32


@pytest.fixture(scope="module")
def a2d():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding
    binding.lib()
    return binding


# heads, kv_heads, nq, nkv, H, causal, q_off, segments (kv_off, rows)
CASES = [
    (9, 9, 479, 131, 64, False, 0, [(0, 131)]),                    # 30 row blocks per head, the last one ragged
    (6, 2, 700, 77, 80, True, 30, [(0, 77)]),                      # grouped; keys the first rows do not see
    (67, 67, 497, 50, 96, True, 20, [(0, 17), (40, 33)]),          # 16 blocks of 32 rows per head: 32-row workgroups
    (64, 8, 513, 19, 128, True, 0, [(0, 3), (1, 16)]),             # 32-row workgroups, the last with one row; fewer key blocks than lanes
    (34, 34, 961, 33, 80, False, 0, [(0, 33)]),
    (2, 1, 17, 1000, 96, True, 990, [(5, 999), (0, 1)]),           # few row blocks, many key blocks: the walks are shared
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dq%dkv_%dx%dxH%d" % c[:5])
def test_f32_tiles_at_every_launch_shape(a2d, case):
    heads, kvh, nq, nkv, H, causal, q_off, segs = case
    grp, scale = heads // kvh, 1.0 / math.sqrt(H)
    Q, dO = (synth.normal((heads, nq, H), 71, s, 1.0, "f32") for s in (0, 1))
    K, V = (synth.normal((kvh, nkv, H), 71, s, 1.0, "f32") for s in (2, 3))
    hs = [h for k in sorted({0, kvh // 2, kvh - 1}) for h in range(k * grp, (k + 1) * grp)]
    ks = sorted({h // grp for h in hs})
    kh = [h // grp for h in hs]
    pos = oracle.segment_positions(segs)
    Qh, dOh, Kh, Vh = np64(Q[hs]), np64(dO[hs]), np64(K[kh]), np64(V[kh])
    Nr, mr, lr = oracle.partial_fwd_pos(Qh, Kh, Vh, q_off, pos, causal, scale)
    Qd, Kd, Vd, dOd = (t.cuda() for t in (Q, K, V, dO))
    print("f32 case", case, flush=True)
    N, m, l = (np64(t[hs]) for t in a2d.partial_fwd(Qd, Kd, Vd, q_off, 0, causal, scale, segments=segs))
    ok = ~np.isinf(mr)
    assert np.array_equal(np.isneginf(m), ~ok) and np.all(N[~ok] == 0) and np.all(l[~ok] == 0)
    assert_close(m[ok], mr[ok], F32, "m", rel=False)
    assert_close(N[ok] / l[ok][:, None], Nr[ok] / lr[ok][:, None], F32, "N/l")
    assert_close(m[ok] + np.log(l[ok]), mr[ok] + np.log(lr[ok]), F32, "m + ln l", rel=False)
    # gradients, from the tile's own O and lse (rows that see nothing: lse = -inf)
    O, lse = a2d.fix(*([t] for t in a2d.partial_fwd(Qd, Kd, Vd, q_off, 0, causal, scale, segments=segs)), F32)
    Oh, lh = np64(O[hs]), np64(lse[hs])
    rq, rk, rv = oracle.partial_bwd_pos(Qh, Kh, Vh, Oh, dOh, lh, q_off, pos, causal, scale)
    got = a2d.partial_bwd(Qd, Kd, Vd, O, dOd, lse, q_off, 0, causal, scale, segments=segs)
    again = a2d.partial_bwd(Qd, Kd, Vd, O, dOd, lse, q_off, 0, causal, scale, segments=segs)
    for x, y in zip(got, again):
        assert torch.equal(x, y)
    fold = lambda x: x.reshape(len(ks), grp, nkv, H).sum(1)
    assert_close(np64(got[0][hs]), rq, F32, "dQ")
    assert_close(np64(got[1][ks]), fold(rk), F32, "dK")
    assert_close(np64(got[2][ks]), fold(rv), F32, "dV")
