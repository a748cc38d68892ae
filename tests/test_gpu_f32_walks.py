"""The fp32 forward's walk: K through LDS one block ahead, V in registers one block ahead, both requested again past the walk's end.
Walks of no, one and several blocks for some or all of the key lanes, ragged last blocks, sub-blocks that are skipped."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2503_15758_amd import synth
from helpers import assert_close, np64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def a2d():
    from paper_2503_15758_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("H", [64, 80, 96, 128])
@pytest.mark.parametrize("heads", [2, 64])                     # 16- and 32-row workgroups (64 heads x 16 blocks of 32 rows)
@pytest.mark.parametrize("rows", [[1], [15], [16], [17], [64], [65], [129], [1, 16, 3], [70, 20, 33]])
@pytest.mark.parametrize("q_off", [None, 40, 0])               # no mask; sub-blocks seen in part, or not at all
def test_walks(a2d, H, heads, rows, q_off):
    nq, nkv, causal, scale = 33 if heads == 2 else 497, sum(rows), q_off is not None, 1.0 / math.sqrt(H)
    segs, at = [], 0
    for r in rows:
        segs.append((at, r))
        at += r + 25
    Q = synth.normal((heads, nq, H), 91, 0, 1.0, "f32")
    K, V = (synth.normal((heads, nkv, H), 91, s, 1.0, "f32") for s in (1, 2))
    hs = [0, heads - 1]
    Nr, mr, lr = oracle.partial_fwd_pos(np64(Q[hs]), np64(K[hs]), np64(V[hs]), q_off or 0, oracle.segment_positions(segs), causal, scale)
    N, m, l = (np64(t[hs]) for t in a2d.partial_fwd(Q.cuda(), K.cuda(), V.cuda(), q_off or 0, 0, causal, scale, segments=segs))
    ok = ~np.isinf(mr)
    assert np.array_equal(np.isneginf(m), ~ok) and np.all(N[~ok] == 0) and np.all(l[~ok] == 0)
    assert_close(m[ok], mr[ok], torch.float32, "m", rel=False)
    assert_close(N[ok] / l[ok][:, None], Nr[ok] / lr[ok][:, None], torch.float32, "N/l")
    assert_close(m[ok] + np.log(l[ok]), mr[ok] + np.log(lr[ok]), torch.float32, "m + ln l", rel=False)
