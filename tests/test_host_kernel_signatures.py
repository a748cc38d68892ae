"""What the kernels' signatures and inline assembly promise the compiler (read from the sources: a broken promise shows only where a
compiler makes use of it)."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_15758_amd", "csrc")


@pytest.mark.parametrize("source, kernel", [("a2d_fwd_mfma.hip", "fwd_mfma_kernel"), ("a2d_f32_mfma.hip", "fwd_f32_kernel")])
def test_forward_outputs_may_alias_the_running_partial(source, kernel):
    """An accumulating forward call reads the triple it writes (`in` and the outputs are the same buffers), so the
    outputs must not be declared __restrict__."""
    text = open(os.path.join(CSRC, source)).read()
    parameters = re.search(r"\b%s\(\s*a2d_tile_desc(.*?)\)\s*\{" % kernel, text, re.S).group(1)
    assert "FwdInput in" in parameters
    for name in ("O_part", "m_out", "l_out"):
        (declared,) = [p for p in parameters.split(",") if re.search(r"\b%s$" % name, p.strip())]
        assert "__restrict__" not in declared, "%s: %s" % (kernel, declared.strip())
    # (what it only reads stays promised: the tile loads depend on it)
    assert all("__restrict__" in p for p in parameters.split(",") if re.search(r"\bconst \w+\*", p))


def test_assembly_that_uses_m0_says_so():
    """A direct load into LDS takes its address from m0, which the compiler may hold a value of its own in (an indexed
    register access, a message): the assembly names it as an input, and none writes it unnamed."""
    users = []
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read().replace("\\\n", "\n")        # (of macros too)
        for at in re.finditer(r"\basm\b", text):
            depth, end = 0, text.index("(", at.start())
            while True:                                                          # (its parentheses)
                depth += {"(": 1, ")": -1}.get(text[end], 0)
                end += 1
                if depth == 0:
                    break
            statement = text[at.start():end]
            code = statement.split("::")[0]
            assert not re.search(r"\bm0\s*,", code) or '"m0"' in statement, "%s: %s" % (name, statement)
            if "global_load_lds" in code:
                users.append(name)
                assert '"{m0}"' in statement, "%s: %s" % (name, statement)
    assert users == ["a2d_mfma.hpp"]
