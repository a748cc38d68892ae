"""Merges of more column groups than HIP launches threads: they go out in slices, whose seams lie inside the tensors."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def a2d():
    from paper_2503_15758_amd import binding
    binding.lib()
    return binding


def test_more_groups_than_threads(a2d):
    """2^32 and some groups of normalised bf16 partials, three times the same: the same rows, and lse + ln 3."""
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 64 GiB of partials and results")
    rows, H, piece = (1 << 24) + 3, 1024, 1 << 20
    x = torch.empty(rows, H, dtype=torch.bfloat16, device="cuda")
    base = torch.randn(257, H, device="cuda").bfloat16()       # (257 rows in turn, with a column that numbers the pieces)
    for at in range(0, rows, piece):
        n = min(piece, rows - at)
        x[at:at + n] = base[torch.arange(at, at + n, device="cuda") % 257]
        x[at:at + n, 5] = at // piece + 1
    lse = torch.arange(rows, device="cuda", dtype=torch.float32) % 31
    O, L = a2d.fix_norm([x, x, x], [lse, lse, lse], torch.bfloat16)
    assert torch.all((L - lse - math.log(3.0)).abs() < 1e-5)
    for at in range(0, rows, piece):
        # a third of three times a row is that row in fp32 but for an ulp, which bf16 does not hold
        assert torch.equal(O[at:at + piece], x[at:at + piece]), at
    del x, O
    torch.cuda.empty_cache()
