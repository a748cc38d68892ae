"""Where the memory for the partial results of shared walks comes from: replays of captured calls that share walks, a
stream captured without torch's allocator, a full device, and the calls of the C boundary, which never share."""
import ctypes
import math
import warnings

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def a2d():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15758_amd import binding
    binding.lib()
    return binding


class Tile:
    """Few row blocks against a long walk, both ways round: forward, dQ and dK / dV all share walks."""

    def __init__(self, a2d, dtype, nq, nkv, heads=2, H=128):
        self.a2d = a2d
        gen = torch.Generator(device="cuda")
        gen.manual_seed(31)
        make = lambda n: torch.randn(heads, n, H, generator=gen, device="cuda").to(dtype)
        self.Q, self.dO, self.O, self.K, self.V = make(nq), make(nq), make(nq) * 0.1, make(nkv), make(nkv)
        self.lse = torch.randn(heads, nq, generator=gen, device="cuda") * 0.3 + math.log(nkv)
        f32 = dict(dtype=torch.float32, device="cuda")
        self.scale = 1.0 / math.sqrt(H)
        self.fwd = (torch.empty(heads, nq, H, **f32), torch.empty(heads, nq, **f32), torch.empty(heads, nq, **f32))
        self.bwd = (torch.empty(heads, nq, H, **f32), torch.empty(heads, nkv, H, **f32), torch.empty(heads, nkv, H, **f32))
        self.d = a2d.tile_desc(self.Q, self.K, 0, 0, False, self.scale)
        self.ws = torch.empty(a2d.workspace_bytes(self.d, a2d.OP_PARTIAL_BWD), dtype=torch.uint8, device="cuda")

    def step(self):
        self.a2d.partial_fwd(self.Q, self.K, self.V, 0, 0, False, self.scale, out=self.fwd)
        self.a2d.partial_bwd(self.Q, self.K, self.V, self.O, self.dO, self.lse, 0, 0, False, self.scale, out=self.bwd,
                             workspace=self.ws)
        return self.fwd + self.bwd

    def unshared(self):
        """The same step through the C boundary, which has no scratch memory to share walks with."""
        L, p = self.a2d.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
        out = tuple(torch.empty_like(t) for t in self.fwd + self.bwd)
        qkv, st = [p(self.Q), p(self.K), p(self.V)], ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert L.a2d_partial_fwd(ctypes.byref(self.d), *qkv, *map(p, out[:3]), None, 0, st) == 0
        assert L.a2d_partial_bwd(ctypes.byref(self.d), *qkv, p(self.O), p(self.dO), p(self.lse), *map(p, out[3:]),
                                 p(self.ws), self.ws.numel(), st) == 0
        torch.cuda.synchronize()
        return out


SHAPES = [(torch.bfloat16, 140, 6000), (torch.bfloat16, 6000, 140), (torch.float32, 40, 1500)]
allocations = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]


def differing(xs, ys, tol=None):
    """Numbers of the outputs that are not the same bits (tol: that are further apart, in the 2-norm)."""
    if tol is None:
        return [i for i, (x, y) in enumerate(zip(xs, ys)) if not torch.equal(x, y)]
    return [i for i, (x, y) in enumerate(zip(xs, ys)) if not float((x - y).norm() / y.norm()) < tol]


def shared(t):
    """The step's results, which differ from the unshared ones by the order of their sums only."""
    want = tuple(x.clone() for x in t.step())
    alone = t.unshared()
    assert differing(want, alone), "the shape does not share walks"
    # bf16: a part takes its exponentials against a maximum of its own, so P and dS are rounded anew - each term by at
    # most 2^-9 of itself on either side
    assert not differing(want, alone, 2 * 2.0 ** -9 if t.Q.dtype == torch.bfloat16 else 1e-5)
    return want


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%s_%dx%d" % (str(s[0])[6:], s[1], s[2]))
def test_shared_walks_replay_from_a_graph(a2d, shape):
    print("graph case", shape, flush=True)
    t = Tile(a2d, *shape)
    want = shared(t)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        t.step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        t.step()
    for replay in range(3):
        for x in t.fwd + t.bwd:
            x.fill_(float("nan"))
        junk = [torch.full((4 << 20,), float("nan"), device="cuda") for _ in range(8)]   # eager work on torch's memory
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert not differing(t.fwd + t.bwd, want), "replay %d differs from the eager step" % replay
        del junk


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%s_%dx%d" % (str(s[0])[6:], s[1], s[2]))
def test_a_foreign_capture_takes_no_memory(a2d, shape):
    """A stream captured by the program itself: memory from torch's allocator would be handed out again before the
    graph replays, so the calls share no walks there."""
    print("foreign capture case", shape, flush=True)
    t = Tile(a2d, *shape)
    alone = t.unshared()
    hip = ctypes.CDLL(a2d._loaded_hip_runtime())
    side, graph, run = torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_void_p()
    stream = ctypes.c_void_p(side.cuda_stream)
    with torch.cuda.stream(side):
        t.step()                                   # (kernels loaded, LDS limits raised)
        torch.cuda.synchronize()
        before = allocations()
        assert hip.hipStreamBeginCapture(stream, ctypes.c_int(1)) == 0       # hipStreamCaptureModeThreadLocal
        try:
            t.step()
        finally:
            ended = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
        assert ended == 0 and allocations() == before
    assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        for x in t.fwd + t.bwd:
            x.fill_(float("nan"))
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(run, stream) == 0
        torch.cuda.synchronize()
        assert not differing(t.fwd + t.bwd, alone)
    assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0
    shared(t)                                      # and eagerly they share again


def test_no_memory_is_said_aloud(a2d):
    """Without memory for the partial results a call runs, unshared, and warns."""
    t = Tile(a2d, *SHAPES[0])
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        shared(t)
    alone = t.unshared()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    held = []
    try:
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)   # no new segments
        for size in (16 << 20, 2 << 20, 1 << 20, 1 << 16, 512):     # and what is free in those there are is taken
            while True:
                try:
                    held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
                except torch.cuda.OutOfMemoryError:
                    break
        with pytest.warns(RuntimeWarning, match="share"):
            t.step()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        held.clear()
    torch.cuda.synchronize()
    assert not differing(t.fwd + t.bwd, alone)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%s_%dx%d" % (str(s[0])[6:], s[1], s[2]))
def test_static_call_of_the_boundary(a2d, shape):
    """a2d_partial_bwd_static gives a C caller bitwise what a2d_partial_bwd gives it, and the torch binding's static
    call what the binding's other call gives."""
    print("static case", shape, flush=True)
    t = Tile(a2d, *shape)
    p = lambda x: ctypes.c_void_p(x.data_ptr())
    out = tuple(torch.empty_like(x) for x in t.bwd)
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert a2d.lib().a2d_partial_bwd_static(ctypes.byref(t.d), p(t.Q), p(t.K), p(t.V), p(t.O), p(t.dO), p(t.lse),
                                            *map(p, out), st) == 0
    torch.cuda.synchronize()
    assert not differing(out, t.unshared()[3:])
    before = allocations()
    got = a2d.partial_bwd_static(t.Q, t.K, t.V, t.O, t.dO, t.lse, 0, 0, False, t.scale, out=out)
    assert allocations() == before
    assert not differing(got, shared(t)[3:])
