"""What a program that uses this library has it do, as measurable cases.

`listed()` gives the fixed cases, `draw(rng)` one more of the same ranges, `prepare(case, seed)` what the program
holds before the call (inputs, output buffers, workspace), `run(state)` one pass through the public entry points of
`paper_2503_15758_amd.binding` and `paper_2503_15758_amd.grid`, `work(case)` the bytes and operations a pass cannot do
without and `tolerance(case)` how far two correct implementations of the same precision may be apart.

Kinds of cases (key "op"):
  fwd      one query block against `blocks` key/value blocks that follow one another in the sequence: a tile call for
           the first, accumulating tile calls for the others (one block: the plain tile of one device of the grid)
  gathered one query block against a gathered key/value row, sub-blocks ("segs") of their own global offsets, in the
           normalised partial format
  bwd      the gradient call of one tile, from the saved O and lse of the query block
  fix      AttnFix over k partial triples; fix_bwd: the sum of k gradient partials
  grid     forward and backward of a whole sequence over the emulated grid
Heads "kv_heads" < "heads": grouped queries.  "packed": Q, K, V, O, dO are views of the [rows][heads][H] tensors a
model keeps (K and V of one [rows][2][heads][H] projection).
"""
import math

import torch

from paper_2503_15758_amd import binding as a2d
from paper_2503_15758_amd import grid as emulation

HEAD_SIZES = (64, 80, 96, 128)
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _tile(name, op, heads, nq, nkv, hdim, **more):
    c = {"name": name, "op": op, "dtype": "bf16", "heads": heads, "kv_heads": heads, "nq": nq, "nkv": nkv,
         "hdim": hdim, "causal": False, "q_off": 0, "kv_off": 0, "sigma": 1.0, "packed": False}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one fp32 tile of a 256-token sequence on a 2 x 2 grid (workload c1)
        _tile("fwd fp32 2x128x128", "fwd", 2, 128, 128, 64, dtype="f32", blocks=1),
        # a short sequence over a small grid, forward and backward: many small calls
        {"name": "grid 512 tokens 2x2", "op": "grid", "dtype": "bf16", "heads": 2, "kv_heads": 2, "seq": 512, "grid": 2,
         "hdim": 128, "causal": True, "layout": "contiguous"},
        # a tile of 2048 rows of a 16-head model (workload c2): too few query blocks to fill the chip
        _tile("fwd 16x2048x2048", "fwd", 16, 2048, 2048, 128, blocks=1),
        # that model's whole sequence on its 4 x 4 grid under the causal mask, in the paper's cyclic layout
        {"name": "grid 8192 tokens 4x4", "op": "grid", "dtype": "bf16", "heads": 16, "kv_heads": 16, "seq": 8192, "grid": 4,
         "hdim": 128, "causal": True, "layout": "cyclic"},
        # 175B-like tiles (workload c3): a query block against an unmasked key block, then its diagonal one
        _tile("fwd 96x4096x4096 two blocks", "fwd", 96, 4096, 4096, 128, causal=True, q_off=4096, blocks=2),
        # the gradients of the unmasked tile of that workload, dS kept for dQ
        _tile("bwd 96x4096x4096", "bwd", 96, 4096, 4096, 128, keep_ds=True),
        # long-context prefill (workload c5): long rows, peaky logits
        _tile("fwd 8x16384x16384 peaky", "fwd", 8, 16384, 16384, 128, sigma=4.0, blocks=1),
        # 2.7B-like heads (H = 80) read in place from packed activations, odd sizes, the mask's diagonal through
        # the tile; the smallest workspace, so the scores are recomputed for dQ
        _tile("bwd 32x1999x2777 packed", "bwd", 32, 1999, 2777, 80, causal=True, q_off=778, packed=True, keep_ds=False),
        # grouped queries against a gathered key row of unequal sub-blocks, normalised partials
        _tile("fwd 40/8x1300 gathered", "gathered", 40, 1300, 2561, 128, kv_heads=8, causal=True, q_off=2600,
              segs="0:512,900:777,2600:1272"),
        # the merge of a grid row of 8 partials (workload c3), and of a grid column of 4 gradient partials (c2)
        {"name": "fix 8x96x4096", "op": "fix", "k": 8, "heads": 96, "rows": 4096, "hdim": 128, "out": "bf16"},
        {"name": "fix_bwd 4x16x2048", "op": "fix_bwd", "k": 4, "heads": 16, "rows": 2048, "hdim": 128, "out": "bf16"},
        # fp32 gradients of a ragged tile with an offset diagonal
        _tile("bwd fp32 16x700x900", "bwd", 16, 700, 900, 96, dtype="f32", causal=True, q_off=300, kv_off=100, keep_ds=False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# the most a drawn case computes: below the largest listed one also where a shape is a slow one
_MOST_FLOPS = {"bf16": 8e11, "f32": 1.0e10}
_MOST_BYTES = 1.7e9


def _draw_heads(rng, most):
    if rng.random() < 0.3:                      # grouped queries
        kv = _log_int(rng, 1, 12)
        group = rng.choice([2, 3, 4, 8, 12])
        if kv * group <= most:
            return kv * group, kv
    h = _log_int(rng, 1, most)
    return h, h


def _draw_tile(rng, op):
    fp32 = op != "gathered" and rng.random() < 0.25
    heads, kv = _draw_heads(rng, 16 if fp32 else 96)
    lo, hi = (64, 1024) if fp32 else (128, 16384)
    c = _tile("", op, heads, _log_int(rng, lo, hi), _log_int(rng, lo, hi), rng.choice(HEAD_SIZES), kv_heads=kv,
              dtype="f32" if fp32 else "bf16", causal=rng.random() < 0.5, sigma=4.0 if not fp32 and rng.random() < 0.15 else 1.0,
              packed=rng.random() < 0.25)
    del c["name"]
    if c["causal"]:                             # the diagonal starts anywhere from the first key to past the last
        c["kv_off"] = rng.choice([0, 0, 100])
        c["q_off"] = c["kv_off"] + rng.choice([0, max(0, c["nkv"] - c["nq"]), rng.randint(0, c["nkv"])])
    if op == "fwd":
        c["blocks"] = rng.choice([1, 1, 2, 3])
    elif op == "bwd":
        c["keep_ds"] = not fp32 and rng.random() < 0.6
        if c["causal"]:
            c["q_off"] = max(c["q_off"], c["kv_off"])       # every query sees a key: its lse is finite
        c["sigma"] = 1.0
    else:
        n = rng.randint(2, 8)
        cuts = sorted(rng.sample(range(16, c["nkv"] - 15), n - 1))
        rows = [b - a for a, b in zip([0] + cuts, cuts + [c["nkv"]])]
        off, segs = 0, []
        for r in rows:
            off += rng.choice([0, 0, rng.randint(1, 500)])
            segs.append("%d:%d" % (off, r))
            off += r
        c["segs"] = ",".join(segs)
        c["kv_off"] = 0
        c["q_off"] = rng.randint(0, off) if c["causal"] else 0
    return c


def draw(rng):
    op = rng.choice(["fwd", "fwd", "fwd", "gathered", "bwd", "bwd", "bwd", "fix", "fix_bwd", "grid"])
    while True:
        if op in ("fwd", "gathered", "bwd"):
            c = _draw_tile(rng, op)
        elif op == "grid":
            g = rng.choice([2, 2, 3, 4])
            heads, kv = _draw_heads(rng, 16)
            c = {"op": "grid", "dtype": "bf16", "heads": heads, "kv_heads": kv, "seq": g * _log_int(rng, 64, 2048),
                 "grid": g, "hdim": rng.choice(HEAD_SIZES), "causal": rng.random() < 0.7,
                 "layout": rng.choice(["cyclic", "contiguous"])}
        else:
            c = {"op": op, "k": rng.choice([2, 3, 4, 6, 8, 16]), "heads": _log_int(rng, 1, 96),
                 "rows": _log_int(rng, 128, 16384), "hdim": rng.choice(HEAD_SIZES),
                 "out": "bf16" if rng.random() < 0.75 else "f32"}
        w = work(c)
        if w["bytes"] <= _MOST_BYTES and w["flops"] <= _MOST_FLOPS[c.get("dtype", "bf16")]:
            return c


# ------------------------------------------------------------------------------------------- inputs

def _normal(gen, shape, dtype, sigma=1.0):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    return (x * sigma if sigma != 1.0 else x).to(dtype)


def _segments(c):
    return [tuple(int(v) for v in s.split(":")) for s in c["segs"].split(",")]


def _heads_tensor(gen, heads, rows, hdim, dtype, packed, sigma=1.0):
    """[heads][rows][H]; packed: a view of a [rows][heads][H] tensor."""
    if packed:
        return _normal(gen, (rows, heads, hdim), dtype, sigma).permute(1, 0, 2)
    return _normal(gen, (heads, rows, hdim), dtype, sigma)


def _kv_tensors(gen, c, dtype):
    kv, rows, H = c["kv_heads"], c["nkv"], c["hdim"]
    if c["packed"]:
        x = torch.empty(rows, 2, kv, H, dtype=dtype, device="cuda")
        x[:, 0] = _normal(gen, (rows, kv, H), dtype, c["sigma"])
        x[:, 1] = _normal(gen, (rows, kv, H), dtype)
        return x[:, 0].permute(1, 0, 2), x[:, 1].permute(1, 0, 2)
    return _normal(gen, (kv, rows, H), dtype, c["sigma"]), _normal(gen, (kv, rows, H), dtype)


def _attention(Q, K, V, q_off, kv_off, causal, scale, O, lse):
    """softmax(scale Q K^T) V and its log-sum-exp, head by head in fp32: what the forward saved for the backward."""
    heads, nq, _ = Q.shape
    group = heads // K.shape[0]
    hidden = None
    if causal:
        i = torch.arange(nq, device="cuda").unsqueeze(1) + q_off
        hidden = i < torch.arange(K.shape[1], device="cuda").unsqueeze(0) + kv_off
    for h in range(heads):
        if h % group == 0:
            kt = K[h // group].float().t().contiguous()
            v = V[h // group].float().contiguous()
        s = torch.mm(Q[h].float().contiguous(), kt).mul_(scale)
        if hidden is not None:
            s.masked_fill_(hidden, -math.inf)
        lse[h] = torch.logsumexp(s, 1)
        O[h] = torch.mm(s.sub_(lse[h].unsqueeze(1)).exp_(), v)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    f32 = {"dtype": torch.float32, "device": "cuda"}
    op = c["op"]
    s = {"case": c, "op": op}
    if op in ("fix", "fix_bwd"):
        shape = (c["heads"], c["rows"], c["hdim"])
        s["out"] = DTYPES[c["out"]]
        s["N"] = [torch.randn(shape, generator=gen, **f32) for _ in range(c["k"])]
        if op == "fix":
            # row maxima and sums as tiles of unit-scale scores leave them; a query that sees no key of one tile
            # (the first rows of a masked tile of the cyclic layout) left an empty partial
            s["m"] = [torch.randn(shape[:2], generator=gen, **f32) * 0.4 + 3.5 for _ in range(c["k"])]
            s["l"] = [torch.rand(shape[:2], generator=gen, **f32) * 100 + 50 for _ in range(c["k"])]
            for x, y, z in zip(s["N"], s["m"], s["l"]):
                x *= z.unsqueeze(2) * 0.02
            s["N"][-1][:, 0] = 0.0
            s["m"][-1][:, 0] = -math.inf
            s["l"][-1][:, 0] = 0.0
        return s
    dtype, H = DTYPES[c["dtype"]], c["hdim"]
    s["scale"] = 1.0 / math.sqrt(H)
    if op == "grid":
        s["Q"] = _normal(gen, (c["heads"], c["seq"], H), dtype)
        s["K"] = _normal(gen, (c["kv_heads"], c["seq"], H), dtype)
        s["V"] = _normal(gen, (c["kv_heads"], c["seq"], H), dtype)
        s["dO"] = _normal(gen, (c["heads"], c["seq"], H), dtype)
        return s
    heads, nq = c["heads"], c["nq"]
    s["Q"] = _heads_tensor(gen, heads, nq, H, dtype, c["packed"], c["sigma"])
    if op == "fwd":
        s["KV"] = [_kv_tensors(gen, c, dtype) for _ in range(c["blocks"])]
        s["outs"] = (torch.empty(heads, nq, H, **f32), torch.empty(heads, nq, **f32), torch.empty(heads, nq, **f32))
    elif op == "gathered":
        s["K"], s["V"] = _kv_tensors(gen, c, dtype)
        s["segs"] = _segments(c)
        s["outs"] = (torch.empty(heads, nq, H, dtype=dtype, device="cuda"), torch.empty(heads, nq, **f32))
    else:
        s["K"], s["V"] = _kv_tensors(gen, c, dtype)
        s["dO"] = _heads_tensor(gen, heads, nq, H, dtype, c["packed"])
        s["O"] = torch.empty_like(s["dO"])               # (keeps the strides of a packed dO)
        s["lse"] = torch.empty(heads, nq, **f32)
        _attention(s["Q"], s["K"], s["V"], c["q_off"], c["kv_off"], c["causal"], s["scale"], s["O"], s["lse"])
        s["outs"] = (torch.empty(heads, nq, H, **f32), torch.empty(c["kv_heads"], c["nkv"], H, **f32),
                     torch.empty(c["kv_heads"], c["nkv"], H, **f32))
        s["split"] = c["kv_heads"] != heads
        d = a2d.tile_desc(s["Q"], s["K"], c["q_off"], c["kv_off"], c["causal"], s["scale"], s["V"], s["O"], s["dO"],
                          flags=a2d.DESC_KEEP_DS if c["keep_ds"] else 0)
        if s["split"]:
            need = a2d.workspace_bytes(d, a2d.OP_PARTIAL_BWD_SPLIT, c["kv_heads"])
        else:
            need = a2d.workspace_bytes(d, a2d.OP_PARTIAL_BWD_DS if c["keep_ds"] else a2d.OP_PARTIAL_BWD)
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return s


# --------------------------------------------------------------------------------------------- a pass

def run(s):
    c, op = s["case"], s["op"]
    if op == "fwd":
        for b, (K, V) in enumerate(s["KV"]):
            a2d.partial_fwd(s["Q"], K, V, c["q_off"], c["kv_off"] + b * c["nkv"], c["causal"], s["scale"],
                            out=s["outs"], accumulate=b > 0)
        return s["outs"]
    if op == "gathered":
        return a2d.partial_fwd_norm(s["Q"], s["K"], s["V"], c["q_off"], 0, c["causal"], s["scale"], out=s["outs"],
                                    segments=s["segs"])
    if op == "bwd":
        return a2d.partial_bwd(s["Q"], s["K"], s["V"], s["O"], s["dO"], s["lse"], c["q_off"], c["kv_off"], c["causal"],
                               s["scale"], out=s["outs"], workspace=s["ws"], ds_handover=c["keep_ds"],
                               split_groups=s["split"])
    if op == "fix":
        return a2d.fix(s["N"], s["m"], s["l"], s["out"])
    if op == "fix_bwd":
        return a2d.fix_bwd(s["N"], s["out"])
    O, lse = emulation.forward(s["Q"], s["K"], s["V"], c["grid"], c["causal"], c["layout"], s["scale"])
    dQ, dK, dV = emulation.backward(s["Q"], s["K"], s["V"], O, s["dO"], lse, c["grid"], c["causal"], c["layout"],
                                    s["scale"])
    return {"O": O, "lse": lse, "dQ": dQ, "dK": dK, "dV": dV}


# --------------------------------------------------------------------------- what a pass cannot do without

def _visible(nq, q_off, segs):
    """Scores of `nq` queries from token q_off on against the (kv_off, rows) key runs under the causal mask."""
    total = 0
    for off, rows in segs:
        first = q_off - off + 1                            # keys of the run that query 0 sees, if 0 .. rows
        a = min(nq, max(0, 1 - first))                     # queries before a see none
        b = min(nq, max(a, rows - first + 1))              # queries from b on see all
        total += (b - a) * (first + a + first + b - 1) // 2 + (nq - b) * rows
    return total


def work(case):
    c = case
    op, H = c["op"], c["hdim"]
    if op in ("fix", "fix_bwd"):
        rows, e = c["heads"] * c["rows"], 2 if c["out"] == "bf16" else 4
        if op == "fix":
            return {"bytes": rows * (c["k"] * (H + 2) * 4 + H * e + 4), "flops": rows * c["k"] * (H + 1) * 2}
        return {"bytes": rows * H * (c["k"] * 4 + e), "flops": rows * H * (c["k"] - 1)}
    e, heads, kv = 2 if c["dtype"] == "bf16" else 4, c["heads"], c["kv_heads"]
    if op == "grid":
        n = c["seq"]
        scores = heads * (n * (n + 1) // 2 if c["causal"] else n * n)
        # read: Q, dO, K, V; written: O, dQ, lse, dK, dV
        return {"bytes": n * H * e * (4 * heads + 4 * kv) + heads * n * 4, "flops": 14 * scores * H}
    nq, nkv = c["nq"], c["nkv"]
    blocks = c.get("blocks", 1)
    if op == "gathered":
        segs = _segments(c)
    else:
        segs = [(c["kv_off"] + b * nkv, nkv) for b in range(blocks)]
    scores = heads * (_visible(nq, c["q_off"], segs) if c["causal"] else nq * nkv * blocks)
    q, k = heads * nq, kv * nkv
    if op == "bwd":
        # read: Q, O, dO, lse, K, V; written: dQ, dK, dV (fp32)
        return {"bytes": q * (3 * H * e + 4) + 2 * k * H * e + (q + 2 * k) * H * 4, "flops": 10 * scores * H}
    out = q * (H * e + 4) if op == "gathered" else q * (H + 2) * 4
    return {"bytes": q * H * e + 2 * k * H * e * blocks + out, "flops": 4 * scores * H}


def tolerance(case):
    # bf16 inputs: probabilities and dS are rounded to bf16 before their contractions, merged outputs once more;
    # fp32: sums of up to some thousand terms in 32 bits
    if "out" in case:
        return {"rel": 5e-3} if case["out"] == "bf16" else {"rel": 1e-5}
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}

