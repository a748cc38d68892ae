"""The merges' loads in the compiled kernels: a thread requests all that it reads of the partials before it waits for the first of them,
and up to four partials their addresses come in together, but for sums of three and four."""
import os
import re
import subprocess

from paper_2503_15758_amd import build as lib_build
from test_host_registers import _code_objects

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(lib_build.HIPCC)), "llvm", "bin", "llvm-objdump")


def _listings(tmp_path, most=16):
    """name -> instructions of the merges' kernels of up to `most` partials"""
    found = {}
    for i, elf in enumerate(_code_objects(open(lib_build.LIB, "rb").read())):
        if b"sum_kernel" not in elf:
            continue
        path = tmp_path / ("%d.elf" % i)
        path.write_bytes(elf)
        text = subprocess.run([OBJDUMP, "--disassemble", "--no-show-raw-insn", "--no-leading-addr", str(path)], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n(?=\S*<_Z)", text):
            m = re.match(r"\S*<(_Z\w*?(sum|fix|fix_norm)_kernelI\w*?Li(\d+)ELi(\d+)E\w*)>:", block)
            if m and int(m[3]) <= most:
                found[m[1]] = (m[2], int(m[3]), int(m[4]), [l.split("//")[0].strip() for l in block.splitlines()[1:]])
    return found


def test_no_wait_between_a_threads_loads(tmp_path):
    kernels = _listings(tmp_path)
    assert len(kernels) > 40
    for name, (kind, kmax, cpt, code) in kernels.items():
        half = kind == "fix_norm" and "kernelIDF16b" in name
        wide = [i for i, l in enumerate(code) if l.startswith("buffer_load_dwordx2" if half else "buffer_load_dwordx4")]
        assert len(wide) == kmax * cpt, (name, len(wide))
        between = code[wide[0]:wide[-1]]
        assert not [l for l in between if l.startswith("s_waitcnt") and "vmcnt" in l], name
        if kmax <= 4 and not (kind == "sum" and kmax > 2):     # (sums of three and four spread their requests)
            assert not [l for l in between if l.startswith(("s_waitcnt", "s_cbranch", "s_branch"))], name


def test_merge_alone_ends_with_its_wide_store(tmp_path):
    """AttnFix without the division: a wait behind the store of N is a wait for that store."""
    kernels = {n: code for n, (kind, _, cpt, code) in _listings(tmp_path, 32).items() if kind == "fix" and cpt == 1 and "ELb1EE" in n}
    assert len(kernels) == 8
    for name, code in kernels.items():
        at = max(i for i, l in enumerate(code) if l.startswith("buffer_store_dwordx4"))
        assert not [l for l in code[at:] if l.startswith("s_waitcnt") and "vmcnt" in l], name
