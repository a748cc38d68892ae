"""Backward of few rows and keys: 32 of them a workgroup, whose eight wavefronts share the walk by slabs of 32 and add up
their sums inside the kernel.  At the edges of rows, slabs, rounds of eight slabs and sub-blocks, against fp64 on the GPU."""
import pytest

from test_gpu_bwd_routes import _check

pytestmark = pytest.mark.gpu

# heads, kv_heads, nq, nkv, H, causal, q_off, sub-blocks (None: one), packed
CASES = [
    (2, 2, 32, 96, 128, False, 0, None, False),
    (2, 2, 64, 64, 128, True, 0, None, False),
    (1, 1, 33, 31, 64, True, 0, None, True),
    (6, 2, 255, 65, 80, True, -20, None, True),              # rows that see nothing, grouped heads
    (2, 2, 257, 256, 96, False, 0, None, False),             # one row beyond the first round
    (4, 2, 300, 289, 128, True, 30, None, True),
    (2, 1, 70, 600, 64, True, 560, [(2, 31), (40, 1), (60, 200), (300, 368)], False),
    (3, 3, 513, 95, 128, True, 0, [(0, 33), (400, 62)], True),   # keys that no row sees
    (8, 8, 500, 530, 80, False, 0, None, True),
    (5, 5, 40, 1100, 96, True, 1061, None, False),
]
# one block of keys: the paired workgroups
PAIRS = [
    (2, 2, 32, 32, 128, False, 0, None, False),
    (3, 1, 255, 33, 80, True, -20, None, True),
]
# more workgroups than compute units: dK and dV in one (heads x blocks of 32 queries + 2 x kv_heads x blocks of 32 keys > 256)
BOTH = [
    (40, 40, 65, 64, 128, False, 0, None, True),
    (24, 24, 130, 130, 80, True, 5, None, False),
    (14, 14, 330, 330, 64, True, -10, None, True),
    (60, 12, 70, 200, 128, True, 140, [(0, 33), (60, 167)], False),
    (34, 34, 64, 95, 96, False, 0, None, False),
]


@pytest.mark.parametrize("case", CASES + PAIRS + BOTH, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_small_bwd(case):
    _check(case, False)
