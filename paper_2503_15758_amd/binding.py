"""Binding of liba2d.so: the calls of include/a2d.h on torch tensors.

Argument marshalling only: every step of the path runs in the library's HIP
kernels.  torch supplies device memory and the current stream.  The compute calls
are marshalled by the extension module _native (csrc/a2d_torch.cpp), the queries,
diagnostics and raw exports through ctypes.  If the library or the extension has
not been built (python -m paper_2503_15758_amd.build) every call raises.

Memory: a tile call whose row blocks are too few for the chip shares their walks
among several workgroups and takes up to 32 MiB for each result it shares (forward;
dQ; dK and dV) from torch's allocator while it runs, also where `out` and `workspace`
are given.  Under torch.cuda.graph that is the graph's own pool.  On a stream that the
program captures by other means, no memory is taken and no walk is shared: the same
results up to the order of fp32 sums.  The same where there is no memory, with a
RuntimeWarning.
"""
import ctypes
import math
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "liba2d.so")

A2D_F32, A2D_BF16 = 0, 1
OP_PARTIAL_FWD, OP_FIX, OP_PARTIAL_BWD, OP_FIX_BWD, OP_PARTIAL_BWD_DS, OP_PARTIAL_BWD_SPLIT = 0, 1, 2, 3, 4, 5
MAX_PARTS = 32

EXPORTS = ("a2d_workspace_bytes", "a2d_partial_fwd", "a2d_fix", "a2d_attnfix", "a2d_partial_bwd", "a2d_fix_bwd",
           "a2d_partial_bwd_static",
           "a2d_partial_fwd_seg", "a2d_partial_bwd_seg", "a2d_partial_fwd_acc", "a2d_partial_bwd_acc",
           "a2d_partial_fwd_norm", "a2d_fix_norm", "a2d_partial_fwd_gqa", "a2d_partial_bwd_gqa",
           "a2d_fix_strided", "a2d_fix_bwd_strided", "a2d_fix_norm_strided",
           "a2d_mfma_ceiling_scratch_bytes", "a2d_mfma_ceiling", "a2d_forward_mix_ceiling", "a2d_backward_mix_ceiling", "a2d_lds_read_ceiling", "a2d_debug_force_generic",
           "a2d_debug_trace", "a2d_debug_trace_count", "a2d_copy_probe",
           "a2d_status_str", "a2d_last_error", "a2d_version")


class Layout(ctypes.Structure):
    """a2d_layout: element strides of a [heads][rows][H] tensor; (0, 0) = plain."""
    _fields_ = [("head", ctypes.c_int64), ("row", ctypes.c_int64)]


class TileDesc(ctypes.Structure):
    _fields_ = [("heads", ctypes.c_int32), ("nq", ctypes.c_int32), ("nkv", ctypes.c_int32),
                ("hdim", ctypes.c_int32), ("q_off", ctypes.c_int64), ("kv_off", ctypes.c_int64),
                ("causal", ctypes.c_int32), ("scale", ctypes.c_float), ("dtype", ctypes.c_int32),
                ("flags", ctypes.c_int32), ("lq", Layout), ("lk", Layout), ("lv", Layout), ("lo", Layout),
                ("ldo", Layout)]


class KvSegment(ctypes.Structure):
    _fields_ = [("kv_off", ctypes.c_int64), ("rows", ctypes.c_int32), ("pad", ctypes.c_int32)]


MAX_SEGMENTS = 32
TILE_ACCUMULATE, TILE_NORMALISED, TILE_SPLIT_GROUPS = 1, 2, 4
DESC_KEEP_DS = 1


class A2DError(RuntimeError):
    def __init__(self, status, detail):
        super().__init__("a2d status %d: %s" % (status, detail))
        self.status = status


_lib = None


def lib():
    """The loaded C-ABI library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError("liba2d.so is missing at %s: build it with "
                               "`python -m paper_2503_15758_amd.build`" % LIB_PATH)
        L = ctypes.CDLL(LIB_PATH)
        vp, fp = ctypes.c_void_p, ctypes.c_void_p
        L.a2d_workspace_bytes.restype = ctypes.c_size_t
        L.a2d_workspace_bytes.argtypes = [ctypes.POINTER(TileDesc), ctypes.c_int, ctypes.c_int]
        L.a2d_partial_fwd.restype = ctypes.c_int
        L.a2d_partial_fwd.argtypes = [ctypes.POINTER(TileDesc), vp, vp, vp, fp, fp, fp, vp,
                                      ctypes.c_size_t, vp]
        L.a2d_partial_fwd_seg.restype = ctypes.c_int
        L.a2d_partial_fwd_seg.argtypes = [ctypes.POINTER(TileDesc), ctypes.c_int, ctypes.POINTER(KvSegment),
                                          vp, vp, vp, fp, fp, fp, vp, ctypes.c_size_t, vp]
        L.a2d_partial_bwd_seg.restype = ctypes.c_int
        L.a2d_partial_bwd_seg.argtypes = [ctypes.POINTER(TileDesc), ctypes.c_int, ctypes.POINTER(KvSegment),
                                          vp, vp, vp, vp, vp, fp, fp, fp, fp, vp, ctypes.c_size_t, vp]
        L.a2d_partial_fwd_acc.restype = ctypes.c_int
        L.a2d_partial_fwd_acc.argtypes = L.a2d_partial_fwd_seg.argtypes
        L.a2d_partial_bwd_acc.restype = ctypes.c_int
        L.a2d_partial_bwd_acc.argtypes = L.a2d_partial_bwd_seg.argtypes
        L.a2d_partial_fwd_norm.restype = ctypes.c_int
        L.a2d_partial_fwd_norm.argtypes = [ctypes.POINTER(TileDesc), ctypes.c_int, ctypes.POINTER(KvSegment),
                                           vp, vp, vp, vp, fp, vp, ctypes.c_size_t, vp]
        # (every argument is typed: an untyped Python int travels as a 32-bit C int, and one that lands
        # on the stack - these calls have more arguments than registers - reaches a size_t parameter
        # with undefined upper bits)
        L.a2d_partial_fwd_gqa.restype = ctypes.c_int
        L.a2d_partial_fwd_gqa.argtypes = [ctypes.POINTER(TileDesc), ctypes.c_int32, ctypes.c_int,
                                          ctypes.POINTER(KvSegment), ctypes.c_int, vp, vp, vp, vp, fp, fp, vp,
                                          ctypes.c_size_t, vp]
        L.a2d_partial_bwd_gqa.restype = ctypes.c_int
        L.a2d_partial_bwd_gqa.argtypes = [ctypes.POINTER(TileDesc), ctypes.c_int32, ctypes.c_int,
                                          ctypes.POINTER(KvSegment), ctypes.c_int, vp, vp, vp, vp, vp, fp,
                                          fp, fp, fp, vp, ctypes.c_size_t, vp]
        L.a2d_fix_norm.restype = ctypes.c_int
        L.a2d_fix_norm.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                   ctypes.POINTER(vp), ctypes.POINTER(vp), vp, fp, vp]
        L.a2d_fix.restype = ctypes.c_int
        L.a2d_fix.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32,
                              ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(vp), vp, fp, vp]
        L.a2d_attnfix.restype = ctypes.c_int
        L.a2d_attnfix.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int32,
                                  ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(vp), fp, fp, fp, vp]
        L.a2d_partial_bwd.restype = ctypes.c_int
        L.a2d_partial_bwd.argtypes = [ctypes.POINTER(TileDesc), vp, vp, vp, vp, vp, fp, fp, fp, fp,
                                      vp, ctypes.c_size_t, vp]
        L.a2d_partial_bwd_static.restype = ctypes.c_int
        L.a2d_partial_bwd_static.argtypes = [ctypes.POINTER(TileDesc), vp, vp, vp, vp, vp, fp, fp, fp, fp, vp]
        L.a2d_fix_bwd.restype = ctypes.c_int
        L.a2d_fix_bwd.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int32, ctypes.POINTER(vp),
                                  vp, vp]
        L.a2d_fix_strided.restype = ctypes.c_int
        L.a2d_fix_strided.argtypes = [ctypes.c_int, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                      ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(vp), vp,
                                      ctypes.POINTER(Layout), vp, vp]
        L.a2d_fix_norm_strided.restype = ctypes.c_int
        L.a2d_fix_norm_strided.argtypes = [ctypes.c_int, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                           ctypes.c_int32, ctypes.POINTER(vp), ctypes.POINTER(vp), vp,
                                           ctypes.POINTER(Layout), vp, vp]
        L.a2d_fix_bwd_strided.restype = ctypes.c_int
        L.a2d_fix_bwd_strided.argtypes = [ctypes.c_int, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                          ctypes.POINTER(vp), vp, ctypes.POINTER(Layout), vp]
        L.a2d_mfma_ceiling_scratch_bytes.restype = ctypes.c_size_t
        L.a2d_mfma_ceiling_scratch_bytes.argtypes = []
        L.a2d_mfma_ceiling.restype = ctypes.c_int
        L.a2d_mfma_ceiling.argtypes = [ctypes.c_int, ctypes.c_int, vp, ctypes.c_size_t,
                                       ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_double)]
        L.a2d_backward_mix_ceiling.restype = ctypes.c_int
        L.a2d_backward_mix_ceiling.argtypes = [ctypes.c_int, ctypes.c_int, vp, ctypes.c_size_t,
                                               ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_double)]
        L.a2d_lds_read_ceiling.restype = ctypes.c_int
        L.a2d_lds_read_ceiling.argtypes = [ctypes.c_int, ctypes.c_int, vp, ctypes.c_size_t,
                                           ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_double)]
        L.a2d_forward_mix_ceiling.restype = ctypes.c_int
        L.a2d_forward_mix_ceiling.argtypes = [ctypes.c_int, vp, ctypes.c_size_t,
                                              ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_double)]
        L.a2d_debug_force_generic.restype = None
        L.a2d_debug_force_generic.argtypes = [ctypes.c_int]
        L.a2d_debug_trace.restype = None
        L.a2d_debug_trace.argtypes = [ctypes.POINTER(vp), ctypes.c_int]
        L.a2d_debug_trace_count.restype = ctypes.c_int
        L.a2d_debug_trace_count.argtypes = []
        L.a2d_copy_probe.restype = ctypes.c_int
        L.a2d_copy_probe.argtypes = [vp, vp, ctypes.c_size_t, vp]
        L.a2d_status_str.restype = ctypes.c_char_p
        L.a2d_status_str.argtypes = [ctypes.c_int]
        L.a2d_last_error.restype = ctypes.c_char_p
        L.a2d_last_error.argtypes = []
        L.a2d_version.restype = ctypes.c_char_p
        L.a2d_version.argtypes = []
        _lib = L
    return _lib


_native = None


def _ext():
    """The extension module that marshals the compute calls; raises if it has not been built."""
    global _native
    if _native is None:
        lib()
        try:
            from . import _native as ext
        except ImportError as e:
            raise RuntimeError("the extension module _native is missing in %s: build it with "
                               "`python -m paper_2503_15758_amd.build`" % _PKG) from e
        ext.set_error_class(A2DError)
        _native = ext
    return _native


def _check(status):
    if status != 0:
        raise A2DError(status, lib().a2d_last_error().decode())


def _dtype_code(t):
    if t == torch.float32:
        return A2D_F32
    if t == torch.bfloat16:
        return A2D_BF16
    raise A2DError(-2, "dtype %s not supported" % t)


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def _plain(ts, name):
    """What the library writes is always in the plain layout."""
    for t in ts:
        if not (t.is_cuda and t.is_contiguous()):
            raise A2DError(-1, "%s must be contiguous device tensors" % name)


def _layout(t):
    """a2d_layout of a tensor or view of contiguous rows ((0, 0) for the plain layout)."""
    if t is None or t.is_contiguous():
        return Layout(0, 0)
    heads, rows, H = t.shape
    row = t.stride(1) if rows > 1 else H             # a stride over a dimension of extent 1 is arbitrary
    head = t.stride(0) if heads > 1 else rows * row
    return Layout(int(head), int(row))


def tile_desc(Q, K, q_off, kv_off, causal, scale, V=None, O=None, dO=None, flags=0):
    """Descriptor of the tile; the strides of Q, K (and V, O, dO when given) are taken from the tensors."""
    heads, nq, H = Q.shape
    return TileDesc(heads, nq, K.shape[1], H, int(q_off), int(kv_off), int(bool(causal)),
                    float(scale if scale is not None else 1.0 / math.sqrt(H)), _dtype_code(Q.dtype), int(flags),
                    _layout(Q), _layout(K), _layout(V if V is not None else K), _layout(O), _layout(dO))


def workspace_bytes(desc, op, k=0):
    return int(lib().a2d_workspace_bytes(ctypes.byref(desc), op, k))


def partial_fwd(Q, K, V, q_off=0, kv_off=0, causal=False, scale=None, out=None, segments=None,
                accumulate=False):
    """a2d_partial_fwd. Returns (O_part fp32 [heads][nq][H], m, l fp32 [heads][nq])."""
    return (_native or _ext()).partial_fwd(Q, K, V, q_off, kv_off, causal, scale, out, segments, accumulate)


def partial_fwd_norm(Q, K, V, q_off=0, kv_off=0, causal=False, scale=None, out=None, segments=None):
    """a2d_partial_fwd_norm: the normalised partial (O' in Q's dtype, lse' fp32) of a plain or gathered tile."""
    return (_native or _ext()).partial_fwd_norm(Q, K, V, q_off, kv_off, causal, scale, out, segments)


def fix_norm(O_norms, lses, out_dtype=torch.bfloat16, out=None):
    """a2d_fix_norm over k normalised partials. Returns (O in out_dtype, lse fp32)."""
    return (_native or _ext()).fix_norm(O_norms, lses, out_dtype, out)


def fix(O_parts, ms, ls, out_dtype=torch.bfloat16, out=None):
    """a2d_fix over k partial triples. Returns (O [heads][nq][H] in out_dtype, lse fp32)."""
    return (_native or _ext()).fix(O_parts, ms, ls, out_dtype, out)


def attnfix(O_parts, ms, ls, out=None):
    """a2d_attnfix: AttnFix alone over k partial triples. Returns one partial (N, m, l), fp32, not normalised."""
    return (_native or _ext()).attnfix(O_parts, ms, ls, out)


def partial_bwd(Q, K, V, O, dO, lse, q_off=0, kv_off=0, causal=False, scale=None, out=None,
                workspace=None, segments=None, accumulate=False, ds_handover=False, split_groups=False):
    """a2d_partial_bwd. Returns (dQ_part, dK_part, dV_part), all fp32.  ds_handover=True sets
    A2D_DESC_KEEP_DS in the descriptor: the library may keep dS for the dQ contraction instead of
    recomputing it, and the workspace (allocated here when none is given) must then hold
    a2d_workspace_bytes(A2D_OP_PARTIAL_BWD_DS) bytes.  split_groups=True
    (grouped heads only) passes A2D_TILE_SPLIT_GROUPS: a key block may go to several workgroups,
    each summing over a run of the group's query rows (workspace of A2D_OP_PARTIAL_BWD_SPLIT
    size, which includes the dS area)."""
    return (_native or _ext()).partial_bwd(Q, K, V, O, dO, lse, q_off, kv_off, causal, scale, out, workspace, segments,
                                           accumulate, ds_handover, split_groups)


STATIC_MAX_ROWS = 1 << 20


def partial_bwd_static(Q, K, V, O, dO, lse, q_off=0, kv_off=0, causal=False, scale=None, out=None):
    """a2d_partial_bwd_static: a2d_partial_bwd without a workspace argument (the library's own static
    scratch holds delta; heads * nq <= STATIC_MAX_ROWS).  `out` = (dQ_part, dK_part, dV_part) fp32;
    with out given this function allocates nothing either: the partial results of shared walks go into a
    device array of the library (64 MiB, held from the first call that shares a walk on), and the results are
    bitwise those of partial_bwd.  All calls on one GPU share the library's arrays and must be ordered."""
    return (_native or _ext()).partial_bwd_static(Q, K, V, O, dO, lse, q_off, kv_off, causal, scale, out)


def fix_bwd(parts, out_dtype=torch.bfloat16, out=None):
    """a2d_fix_bwd: sum of k fp32 partials, rounded once to out_dtype."""
    return (_native or _ext()).fix_bwd(parts, out_dtype, out)


def mfma_ceiling(iters=20000, random_data=True):
    """Diagnostic (a2d_mfma_ceiling): (dense bf16 TFLOP/s of the MFMA units alone, shader MHz)."""
    n = int(lib().a2d_mfma_ceiling_scratch_bytes())
    scratch = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    tf, mhz = ctypes.c_double(0.0), ctypes.c_double(0.0)
    _check(lib().a2d_mfma_ceiling(int(iters), int(bool(random_data)), _ptr(scratch), scratch.numel(),
                                  ctypes.byref(tf), ctypes.byref(mhz)))
    return tf.value, mhz.value


def forward_mix_ceiling(iters=6000):
    """Diagnostic (a2d_forward_mix_ceiling): (TFLOP/s of the forward loop's model - MFMA + LDS fragment +
    softmax arithmetic per MFMA -, shader MHz)."""
    n = int(lib().a2d_mfma_ceiling_scratch_bytes())
    scratch = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    tf, mhz = ctypes.c_double(0.0), ctypes.c_double(0.0)
    _check(lib().a2d_forward_mix_ceiling(int(iters), _ptr(scratch), scratch.numel(), ctypes.byref(tf), ctypes.byref(mhz)))
    return tf.value, mhz.value


LEAVE_MAILBOX, LEAVE_ARITHMETIC, LEAVE_BARRIER = 1, 2, 4


def backward_mix_ceiling(iters=6000, leave_out=0):
    """Diagnostic (a2d_backward_mix_ceiling): (TFLOP/s of the dK/dV loop's model - paired roles, natural and
    transposing LDS fragments, mailbox, one barrier per step -, shader MHz); leave_out: LEAVE_* bits."""
    n = int(lib().a2d_mfma_ceiling_scratch_bytes())
    scratch = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    tf, mhz = ctypes.c_double(0.0), ctypes.c_double(0.0)
    _check(lib().a2d_backward_mix_ceiling(int(iters), int(leave_out), _ptr(scratch), scratch.numel(),
                                          ctypes.byref(tf), ctypes.byref(mhz)))
    return tf.value, mhz.value


def lds_read_ceiling(iters=20000, transposing=False):
    """Diagnostic (a2d_lds_read_ceiling): (10^12 bytes per second the chip's LDS delivers to wavefronts that
    only read it, shader MHz)."""
    n = int(lib().a2d_mfma_ceiling_scratch_bytes())
    scratch = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    tb, mhz = ctypes.c_double(0.0), ctypes.c_double(0.0)
    _check(lib().a2d_lds_read_ceiling(int(iters), int(bool(transposing)), _ptr(scratch), scratch.numel(),
                                      ctypes.byref(tb), ctypes.byref(mhz)))
    return tb.value, mhz.value


def tile_route(heads, nq, nkv, hdim, dtype=torch.bfloat16, kv_heads=None, q_off=0, kv_off=0, causal=False, segments=None,
               backward=False, ds_handover=False, split_groups=False, scratch=True, compute_units=0):
    """Diagnostic: how a tile call of these sizes goes out, by the library's own plans and without a device (compute_units
    0: those of the current one).  A dict: "kernels" in launch order, "rows" and "lanes" (key lanes) of a forward or dQ
    workgroup, "keys" of a dK/dV workgroup, "parts_q" and "parts_kv" (workgroups that share a walk), "phased" (a forward's
    wavefronts in opposite phases), "apart" (dK and dV of a backward of few rows in workgroups of their own).  scratch: whether
    there is memory for partial results (this module's calls; not those of the C boundary)."""
    flags = 1 * bool(backward) | 2 * bool(ds_handover) | 4 * bool(split_groups) | 8 * bool(scratch)
    return _ext().tile_route(heads, kv_heads or heads, nq, nkv, hdim, dtype, q_off, kv_off, causal, segments, flags,
                             compute_units)


def force_generic(on):
    """a2d_debug_force_generic: route every tile call to the vector-ALU kernels (debugging aid)."""
    lib().a2d_debug_force_generic(int(bool(on)))


def copy_probe(dst, src):
    """a2d_copy_probe: plain device copy of src into dst (contiguous device tensors of equal byte size)."""
    _plain([dst, src], "dst, src")
    n = src.numel() * src.element_size()
    if n != dst.numel() * dst.element_size():
        raise A2DError(-1, "dst and src differ in size")
    _check(lib().a2d_copy_probe(_ptr(dst), _ptr(src), n, _stream()))
    return dst


def _loaded_hip_runtime():
    """Path of the HIP runtime ALREADY mapped into this process (the one liba2d.so and torch use):
    events must come from that copy, not from a second one a search by name might load."""
    with open("/proc/self/maps") as f:
        for line in f:
            if "libamdhip64.so" in line:
                return line.split()[-1]
    raise RuntimeError("no HIP runtime is loaded in this process")


class KernelTrace:
    """a2d_debug_trace on the calling thread: `with KernelTrace(n) as tr:` records up to n HIP events
    (created here through the HIP runtime the library is linked against); after a device
    synchronisation tr.intervals_ms() gives the time between consecutive recorded events."""

    def __init__(self, n):
        self.n = int(n)
        lib()
        self._hip = ctypes.CDLL(_loaded_hip_runtime())
        self._hip.hipEventCreate.argtypes = [ctypes.POINTER(ctypes.c_void_p)]
        self._hip.hipEventDestroy.argtypes = [ctypes.c_void_p]
        self._hip.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_void_p, ctypes.c_void_p]
        self._ev = (ctypes.c_void_p * self.n)()
        for i in range(self.n):
            e = ctypes.c_void_p()
            if self._hip.hipEventCreate(ctypes.byref(e)) != 0:
                raise A2DError(-5, "hipEventCreate failed")
            self._ev[i] = e
        self.count = 0

    def __enter__(self):
        lib().a2d_debug_trace(self._ev, self.n)
        return self

    def __exit__(self, *exc):
        self.count = int(lib().a2d_debug_trace_count())
        lib().a2d_debug_trace(None, 0)
        return False

    def intervals_ms(self):
        """[t(event i+1) - t(event i)] for the recorded events; call after the device has finished them."""
        out = []
        for i in range(self.count - 1):
            ms = ctypes.c_float()
            if self._hip.hipEventElapsedTime(ctypes.byref(ms), self._ev[i], self._ev[i + 1]) != 0:
                raise A2DError(-5, "hipEventElapsedTime failed")
            out.append(ms.value)
        return out

    def close(self):
        for i in range(self.n):
            if self._ev[i]:
                self._hip.hipEventDestroy(self._ev[i])
                self._ev[i] = None


def version():
    return lib().a2d_version().decode()
