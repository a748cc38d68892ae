// The whole-grid launches (see a2d_grid.hpp).  Host code only.
//
// Why batched: a grid of small tiles is bound by everything but the tiles' arithmetic when each tile is
// a call of its own - index gathers of the blocks, stream events, a handful of launches per tile, tiles
// that fill an eighth of the chip.  512 tokens on a 2 x 2 grid took 52 launches and 680 us for 60 us of
// kernels; 8192 tokens x 16 heads on 4 x 4 took 2.8 ms for 1.3 ms' worth of work.
// The forward walks all tiles of a grid row in one workgroup: AttnFix over the row in registers, no partials in
// memory, walks `side` times as long.  8192 tokens x 16 heads on 4 x 4, cyclic: tile launch and merge 441 + 49 us, one
// launch 307 us.  The backward likewise, dQ by grid rows and dK, dV by grid columns, with the scores recomputed for
// dQ: 575 + 460 us against 15 (delta) + 850 (dK, dV, dS) + 346 (dQ) + 153 us (sums), and no gigabytes of dS and partials.
#include "a2d_grid.hpp"

#include <cstring>

#include "a2d_common.hpp"

namespace a2d {
namespace {

int rows_of(const GridProblem& p) { return p.seq / p.side; }
size_t up256(size_t n) { return (n + 255) / 256 * 256; }

int64_t block_step(const GridProblem& p, const a2d_layout& l) { return p.cyclic ? l.row : l.row * rows_of(p); }
a2d_layout block_layout(const GridProblem& p, const a2d_layout& l) {
  return a2d_layout{l.head, p.cyclic ? l.row * p.side : l.row};
}

void describe(const GridProblem& p, a2d_tile_desc* d, SegList* g) {
  memset(d, 0, sizeof(*d));
  memset(g, 0, sizeof(*g));
  d->heads = p.heads;
  d->nq = d->nkv = rows_of(p);
  d->hdim = p.hdim;
  d->causal = p.causal;
  d->scale = p.scale;
  d->dtype = A2D_BF16;
  d->lq = block_layout(p, p.q);
  d->lk = block_layout(p, p.k);
  d->lv = block_layout(p, p.v);
  d->lo = block_layout(p, p.o);
  d->ldo = block_layout(p, p.g);
  g->n = 1;
  g->group = p.heads / p.kv_heads;
  g->parts = 1;
  g->seg[0].rows = rows_of(p);
  g->b.side = p.side;
  g->b.cyclic = p.cyclic;
  g->b.q = block_step(p, p.q);
  g->b.k = block_step(p, p.k);
  g->b.v = block_step(p, p.v);
  g->b.g = block_step(p, p.g);
  g->b.o = block_step(p, p.o);
}

void output(const GridProblem& p, const a2d_layout& l, SegList* g, int x) {
  g->b.out[x] = block_layout(p, l);
  g->b.out_step[x] = block_step(p, l);
}

// Parts of `floats` floats each (few, small blocks: split walks, merged by one more launch) that fit kSplitBytes
int cap_of(size_t floats) {
  const size_t room = kSplitBytes / sizeof(float) / floats;
  return room < 1 ? 1 : room < A2D_MAX_PARTS ? (int)room : A2D_MAX_PARTS;
}
size_t out_floats(const GridProblem& p, int heads) { return (size_t)heads * p.seq * p.hdim; }

// The forward's shape and parts, the backward's parts, from the problem and the compute units (0: of the device).
// false: no device
bool plan_forward(const GridProblem& p, const a2d_tile_desc& d, SegList* g, int cus = 0) {
  if (cus == 0 && device_cus(&cus) != hipSuccess) return false;
  plan_fwd_mfma(d, g, cus, cap_of((size_t)p.heads * p.seq * (p.hdim + 2)));
  return true;
}
bool plan_backward(const GridProblem& p, const a2d_tile_desc& d, const SegList& g, BwdParts* b, int cus = 0) {
  if (cus == 0 && device_cus(&cus) != hipSuccess) return false;
  *b = plan_bwd_mfma(d, g, false, cus, cap_of(2 * out_floats(p, p.kv_heads)), cap_of(out_floats(p, p.heads)));
  return true;
}
// floats of partial results
size_t part_floats(const GridProblem& p, const BwdParts& b) {
  return (b.q > 1 ? b.q * out_floats(p, p.heads) : 0) + (b.kv > 1 ? 2 * b.kv * out_floats(p, p.kv_heads) : 0);
}

}  // namespace

bool grid_supported(const GridProblem& p) {
  if (p.heads < 1 || p.kv_heads < 1 || p.heads % p.kv_heads || p.heads > 65535 || p.side < 1 ||
      p.side > A2D_MAX_PARTS || p.seq < p.side || p.seq % p.side || p.seq > (1 << 22) || !(p.scale > 0.f))
    return false;
  if (p.hdim != 64 && p.hdim != 80 && p.hdim != 96 && p.hdim != 128) return false;
  if ((int64_t)p.heads * p.seq * (p.hdim / 4) >= ((int64_t)1 << 31)) return false;   // 32-bit indices of the merges
  const int group = p.heads / p.kv_heads;
  if ((int64_t)group * rows_of(p) > (1 << 22)) return false;
  const a2d_layout* all[5] = {&p.q, &p.k, &p.v, &p.o, &p.g};
  for (int i = 0; i < 5; ++i) {
    const a2d_layout& l = *all[i];
    const int64_t heads = (i == 1 || i == 2) ? 1 : group;
    if (l.row < p.hdim || l.head < 1 || l.row % 8 || l.head % 8 || l.row > ((int64_t)1 << 30) ||
        l.head > ((int64_t)1 << 40))
      return false;
    if (l.row * (p.cyclic ? p.side : 1) * 2 >= ((int64_t)1 << 24)) return false;
    if (((heads - 1) * l.head + (int64_t)p.seq * l.row) * 2 >= ((int64_t)1 << 32)) return false;
  }
  return true;
}

size_t grid_forward_bytes(const GridProblem& p) {
  a2d_tile_desc d;
  SegList g;
  describe(p, &d, &g);
  if (!plan_forward(p, d, &g) || g.parts == 1) return 0;
  return (size_t)g.parts * p.heads * p.seq * (p.hdim + 2) * sizeof(float);
}

size_t grid_backward_bytes(const GridProblem& p) {
  a2d_tile_desc d;
  SegList g;
  BwdParts b;
  describe(p, &d, &g);
  if (!plan_backward(p, d, g, &b)) return 0;
  return up256((size_t)p.heads * p.seq * sizeof(float)) + part_floats(p, b) * sizeof(float);
}

hipError_t grid_forward(const GridProblem& p, const void* Q, const void* K, const void* V, void* O, float* lse,
                        void* ws, hipStream_t s) {
  a2d_tile_desc d;
  SegList g;
  describe(p, &d, &g);
  if (!plan_forward(p, d, &g)) return hipErrorInvalidDevice;
  const FwdInput none{nullptr, nullptr, nullptr};
  const size_t rows = (size_t)p.heads * p.seq;
  float *N = static_cast<float*>(O), *m = lse, *l = nullptr;   // lines 4-6 of Alg. 1 in one launch ...
  g.norm = g.parts == 1;
  if (g.parts > 1) {                                           // ... or the partials of split walks
    N = static_cast<float*>(ws);
    m = N + g.parts * rows * p.hdim;
    l = m + g.parts * rows;
  }
  hipError_t e = launch_fwd_mfma(PREPARE, d, g, Q, K, V, N, m, l, none, s);
  if (e != hipSuccess) return e;
  trace_mark(s);
  e = launch_fwd_mfma(LAUNCH, d, g, Q, K, V, N, m, l, none, s);
  if (e != hipSuccess || g.parts == 1) return e;
  FixPtrs f;
  memset(&f, 0, sizeof(f));
  for (int z = 0; z < g.parts; ++z) {                          // each [row block][head][row]
    f.o[z] = N + z * rows * p.hdim;
    f.m[z] = m + z * rows;
    f.l[z] = l + z * rows;
  }
  const GridMap parts{p.side, rows_of(p), p.heads, p.cyclic, g.parts};
  return launch_fix_grid(parts, p.hdim, A2D_BF16, f, p.o, O, lse, s);
}

hipError_t grid_backward(const GridProblem& p, const void* Q, const void* K, const void* V, const void* O,
                         const void* dO, const float* lse, void* dQ, void* dK, void* dV, void* ws, hipStream_t s) {
  a2d_tile_desc d;
  SegList g;
  BwdParts bp;
  describe(p, &d, &g);
  if (!plan_backward(p, d, g, &bp)) return hipErrorInvalidDevice;
  output(p, p.dq, &g, 0);
  output(p, p.dk, &g, 1);
  output(p, p.dv, &g, 2);
  float* delta = static_cast<float*>(ws);
  float* more = reinterpret_cast<float*>(static_cast<char*>(ws) + up256((size_t)p.heads * p.seq * sizeof(float)));
  // all lines of Alg. 3 in one launch, delta's in front where the plan has it read, or the partials of split walks and their sums
  const size_t nq = out_floats(p, p.heads), nk = out_floats(p, p.kv_heads);
  void *q = dQ, *k = dK, *v = dV;
  SumSet sets[3];
  int n = 0;
  memset(sets, 0, sizeof(sets));
  const auto split = [&](int parts, int heads, size_t floats, void* out, const a2d_layout& lo) -> void* {
    SumSet& t = sets[n++];
    for (int z = 0; z < parts; ++z) t.p.p[z] = more + z * floats;
    t.gm = GridMap{p.side, rows_of(p), heads, p.cyclic, parts};
    t.out = out;
    t.lo = lo;
    float* const first = more;
    more += parts * floats;
    return first;
  };
  if (bp.q > 1) q = split(bp.q, p.heads, nq, dQ, p.dq);
  if (bp.kv > 1) {
    k = split(bp.kv, p.kv_heads, nk, dK, p.dk);
    v = split(bp.kv, p.kv_heads, nk, dV, p.dv);
  }
  hipError_t e = launch_bwd_one(PREPARE, d, g, Q, K, V, O, dO, lse, delta, (float*)q, (float*)k, (float*)v, bp, s);
  if (e != hipSuccess) return e;
  trace_mark(s);
  e = launch_bwd_one(LAUNCH, d, g, Q, K, V, O, dO, lse, delta, (float*)q, (float*)k, (float*)v, bp, s);
  return e != hipSuccess || n == 0 ? e : launch_sum_grid(n, sets, p.hdim, A2D_BF16, s);
}

bool grid_route(const GridProblem& p, bool backward, int cus, Route* out) {
  if (!grid_supported(p)) return false;
  a2d_tile_desc d;
  SegList g;
  describe(p, &d, &g);
  if (!backward) {
    if (!plan_forward(p, d, &g, cus)) return false;
    route_fwd(d, g, out);
    if (g.parts > 1) out->kernel[out->kernels++] = "fix_grid_kernel";
    return true;
  }
  BwdParts b;
  if (!plan_backward(p, d, g, &b, cus)) return false;
  route_bwd(d, b, out);
  if (b.kv > 1 || b.q > 1) out->kernel[out->kernels++] = "sum_grid_kernel";
  return true;
}

}  // namespace a2d
