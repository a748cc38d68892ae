"""Builds liba2d.so (the C-ABI library) from csrc/ with hipcc for gfx950, and _native.so (its calls on
torch tensors, host code only) with g++.

Usage: python -m paper_2503_15758_amd.build [--force]
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "liba2d.so")
EXT = os.path.join(PKG, "_native.so")
SOURCES = ["a2d_api.hip", "a2d_device.hip", "a2d_fix.hip", "a2d_generic.hip", "a2d_f32_mfma.hip",
           "a2d_fwd_mfma.hip", "a2d_fwd_small.hip", "a2d_bwd_mfma.hip", "a2d_bwd_wide.hip", "a2d_bwd_one.hip", "a2d_bwd_small.hip", "a2d_grid.hip", "a2d_static.hip",
           "a2d_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC,
         # packed-fp32 VALU forms are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    if out.strip():
        print(out)


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _ext_command():
    import torch
    t = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
            "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", os.path.join(t, "include"),
            "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
            "-isystem", os.environ.get("ROCM_PATH", "/opt/rocm") + "/include", "-I", sysconfig.get_paths()["include"],
            os.path.join(CSRC, "a2d_torch.cpp"), "-o", EXT, "-L", PKG, "-l:liba2d.so", "-L", os.path.join(t, "lib"),
            "-lc10", "-lc10_hip", "-ltorch", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]


def build(force=False, verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    headers = [os.path.join(CSRC, "a2d_common.hpp"), os.path.join(CSRC, "a2d_mfma.hpp"),
               os.path.join(CSRC, "a2d_bwd.hpp"), os.path.join(CSRC, "a2d_bwd_dq.hpp"),
               os.path.join(CSRC, "a2d_bwd_pairs.hpp"), os.path.join(CSRC, "a2d_bwd_wide.hpp"),
               os.path.join(CSRC, "a2d_grid.hpp"), os.path.join(ROOT, "include", "a2d.h")]
    jobs, objs = [], []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, src.replace(".hip", ".o"))
        objs.append(o)
        if force or _stale(o, [s] + headers):
            jobs.append([HIPCC] + FLAGS + ["-c", s, "-o", o])
    with ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as ex:
        list(ex.map(_run, jobs))
    if force or jobs or _stale(LIB, objs):
        _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    if force or _stale(EXT, [os.path.join(CSRC, "a2d_torch.cpp"), os.path.join(CSRC, "a2d_grid.hpp"),
                             os.path.join(ROOT, "include", "a2d.h")]):
        _run(_ext_command())
    if verbose:
        print("built", LIB, "(%d objects recompiled)" % len(jobs))
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv)
