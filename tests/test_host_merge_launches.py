"""The launches of a merge, counted by stand-ins for HIP's launch functions (no GPU): whatever the call takes, each has less than the
2^32 threads that HIP can launch, and together they cover the groups of four columns once."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# the kernels take (partials, k, first group, ...)
STUB = """#include <stdio.h>
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
static long long n, seen[4096][3];
long long launches(void) { return n; }
void forget(void) { n = 0; }
long long field(long long i, int f) { return seen[i][f]; }
int hipGetLastError(void) { return 0; }
static dim3 grid, block;
static size_t shared;
static void* queue;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* stream) {
  grid = g; block = b; shared = lds; queue = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** stream) {
  *g = grid; *b = block; *lds = shared; *stream = queue;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* stream) {
  if (n < 4096) {
    seen[n][0] = *(long long*)args[2];
    seen[n][1] = (long long)g.x * g.y * g.z;
    seen[n][2] = (long long)b.x * b.y * b.z;
  }
  ++n;
  return 0;
}
"""
CHILD = """
import ctypes, json, sys
stub, lib, cases = sys.argv[1], sys.argv[2], json.loads(sys.argv[3])
S = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
S.launches.restype = S.field.restype = ctypes.c_longlong
S.field.argtypes = [ctypes.c_longlong, ctypes.c_int]
L = ctypes.CDLL(lib)
at = lambda i: ctypes.c_void_p(1 << 20 | i << 8)           # (never read)
for op, k, groups, half in cases:
    S.forget()
    parts = lambda b: (ctypes.c_void_p * k)(*[at(b + i).value for i in range(k)])
    rows, n = ctypes.c_longlong(groups), ctypes.c_longlong(4 * groups)
    if op == "fix": st = L.a2d_fix(k, rows, 4, 1, parts(1), parts(40), parts(80), at(200), at(201), None)
    elif op == "attnfix": st = L.a2d_attnfix(k, rows, 4, parts(1), parts(40), parts(80), at(200), at(201), at(202), None)
    elif op == "fix_norm": st = L.a2d_fix_norm(k, rows, 4, half, 1, parts(1), parts(40), at(200), at(201), None)
    else: st = L.a2d_fix_bwd(k, n, 1, parts(1), at(200), None)
    print(json.dumps([st, [[S.field(i, f) for f in range(3)] for i in range(S.launches())]]))
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    from paper_2503_15758_amd import build as lib_build
    d = tmp_path_factory.mktemp("stub")
    src, stub = d / "stub.c", d / "stub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", str(stub)], check=True)

    def run(cases):
        out = subprocess.run([sys.executable, "-c", CHILD, str(stub), lib_build.LIB, json.dumps(cases)], cwd=ROOT, check=True,
                             capture_output=True, text=True).stdout
        return [json.loads(l) for l in out.splitlines()]
    return run


CASES = [(op, k, groups, half) for op in ("fix", "attnfix", "fix_norm", "fix_bwd") for k in (1, 2, 3, 4, 5, 6, 8, 16, 32)
         for groups in (1, 255, 257, (1 << 19) - 1, 1 << 19, (1 << 21) + 77, (1 << 31) - 1, (1 << 32) - 256, (1 << 32) - 255, (1 << 34) + 5, 1 << 39)
         for half in ((0, 1) if op == "fix_norm" else (0,))]


def test_launches_fit_and_cover(launches):
    for case, (status, made) in zip(CASES, launches(CASES)):
        groups, at = case[2], 0
        assert status == 0 and 1 <= len(made) <= 256, case
        for i, (first, blocks, threads) in enumerate(made):
            assert first == at and blocks * threads < 1 << 32, (case, i, first, blocks)
            # groups a block: as many as the next launch starts behind, and in the last one 1, 2 or 4 a thread
            share = (made[i + 1][0] - first) // blocks if i + 1 < len(made) else None
            if share is None:
                share = next((c * threads for c in (1, 2, 4) if (blocks - 1) * c * threads < groups - at <= blocks * c * threads), 0)
            assert share in (threads, 2 * threads, 4 * threads), (case, i, share)
            at += blocks * share
        assert at >= groups, case
        # below 2^31 groups: one launch, as callers that capture it count on
        assert len(made) == 1 or groups > (1 << 31), case


def test_large_cases_have_their_groups_a_thread(launches):
    """The cases of test_gpu_merge_shares.py take the forms that they are there for, and those are all that there are."""
    import test_gpu_merge_shares as t
    cases = [(op, k, rows * H // 4, int(op == "fix_norm")) for op, k, H, rows, _ in t.LARGE]
    seen = set()
    for (op, k, groups, _), case, (_, made) in zip(cases, t.LARGE, launches(cases)):
        assert made[0][1] == -(-groups // (256 * case[4])), case
        seen.add((op, k, case[4]))
    ops = ("fix", "fix_bwd", "fix_norm")
    every = [(op, k, 1 << i, int(op == "fix_norm")) for op in ops for k in (1, 2, 3, 4, 6, 8, 16) for i in range(14, 24)]
    for (op, k, groups, _), (_, made) in zip(every, launches(every)):
        cpt = groups // (256 * made[0][1])
        assert cpt == 1 or (op, k, cpt) in seen or (op, k) == ("fix_norm", 4), (op, k, groups, cpt)
