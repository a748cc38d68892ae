// The whole-grid launches (see a2d_grid.hpp).  Host code only.
//
// Why batched: a grid of small tiles is bound by everything but the tiles' arithmetic when each tile is
// a call of its own - index gathers of the blocks, stream events, a handful of launches per tile, tiles
// that fill an eighth of the chip.  512 tokens on a 2 x 2 grid took 52 launches and 680 us for 60 us of
// kernels; 8192 tokens x 16 heads on 4 x 4 took 2.8 ms for 1.3 ms' worth of work.
// The forward walks all tiles of a grid row in one workgroup: AttnFix over the row in registers, no partials in
// memory, walks four times as long.  8192 tokens x 16 heads on 4 x 4, cyclic: tile launch and merge 441 + 49 us, one
// launch 329 us.
#include "a2d_grid.hpp"

#include <cstring>

#include "a2d_common.hpp"

namespace a2d {
namespace {

// dS kept at a time by the batched backward: enough tiles to fill the chip many times over, and small
// beside what a grid's own partials take
constexpr size_t kGridDsBytes = (size_t)2 << 30;

int rows_of(const GridProblem& p) { return p.seq / p.side; }
int tri_of(const GridProblem& p) { return p.causal && !p.cyclic; }
int slots_of(const GridProblem& p) { return tri_of(p) ? p.side * (p.side + 1) / 2 : p.side * p.side; }
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
  g->b.n = g->b.slots = slots_of(p);
  g->b.side = p.side;
  g->b.tri = tri_of(p);
  g->b.cyclic = p.cyclic;
  g->b.q = block_step(p, p.q);
  g->b.k = block_step(p, p.k);
  g->b.v = block_step(p, p.v);
  g->b.g = block_step(p, p.g);
  g->b.o = block_step(p, p.o);
}

// tiles whose dS is kept at a time
int chunk_of(const GridProblem& p, const a2d_tile_desc& d, const SegList& g) {
  const size_t per_tile = bwd_ds_bytes(d, g);
  const size_t n = per_tile ? kGridDsBytes / per_tile : 1;
  return n < 1 ? 1 : n > (size_t)slots_of(p) ? slots_of(p) : (int)n;
}

GridMap map_of(const GridProblem& p, int heads, int dir, int parts) {
  return GridMap{p.side, rows_of(p), heads, p.cyclic, tri_of(p) ? dir : 0, parts, p.side};
}

// Parts of the tiles' walks (few, small tiles): the merges of the grid take the parts along, so that only
// their bytes count.  At most what the merges can take, and kSplitBytes of partials.
int cap_of(const GridProblem& p, size_t floats) {
  const int64_t room = (int64_t)(kSplitBytes / sizeof(float) / floats), most = A2D_MAX_PARTS / p.side;
  return room < 1 || most < 1 ? 1 : (int)(room < most ? room : most);
}
size_t out_floats(const GridProblem& p, int heads) { return (size_t)slots_of(p) * heads * rows_of(p) * p.hdim; }

// The forward's shape and parts, the backward's parts.  Both depend on the problem alone (the chunks
// of the backward share its parts).  false: no device
bool plan_forward(const GridProblem& p, const a2d_tile_desc& d, SegList* g) {
  int cus = 0;
  if (device_cus(&cus) != hipSuccess) return false;
  const size_t floats = (size_t)p.heads * p.seq * (p.hdim + 2);
  const size_t room = kSplitBytes / sizeof(float) / floats;
  plan_fwd_mfma(d, g, cus, room < 1 ? 1 : room < A2D_MAX_PARTS ? (int)room : A2D_MAX_PARTS);
  return true;
}
bool plan(const GridProblem& p, const a2d_tile_desc& d, SegList* g, BwdParts* b) {
  int cus = 0;
  if (device_cus(&cus) != hipSuccess) return false;
  *b = plan_bwd_mfma(d, *g, true, cus, cap_of(p, 2 * out_floats(p, p.kv_heads)), cap_of(p, out_floats(p, p.heads)));
  return true;
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
  a2d_tile_desc d;
  SegList g;
  describe(p, &d, &g);
  return bwd_ds_bytes(d, g) > 0;
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
  if (!plan(p, d, &g, &b)) return 0;
  const size_t stats = 2 * up256((size_t)p.heads * p.seq * sizeof(float));
  const size_t parts = (b.q * out_floats(p, p.heads) + 2 * b.kv * out_floats(p, p.kv_heads)) * sizeof(float);
  return stats + up256(parts) + (size_t)chunk_of(p, d, g) * bwd_ds_bytes(d, g);
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
  const GridMap parts{p.side, rows_of(p), p.heads, p.cyclic, 0, g.parts, 1};
  return launch_fix_grid(parts, p.hdim, A2D_BF16, f, p.o, O, lse, s);
}

hipError_t grid_backward(const GridProblem& p, const void* Q, const void* K, const void* V, const void* O,
                         const void* dO, const float* lse, void* dQ, void* dK, void* dV, void* ws, hipStream_t s) {
  a2d_tile_desc d;
  SegList g;
  describe(p, &d, &g);
  const size_t rows = rows_of(p), slots = slots_of(p);
  const size_t stat = up256((size_t)p.heads * p.seq * sizeof(float));
  char* w = static_cast<char*>(ws);
  float* delta = reinterpret_cast<float*>(w);
  float* lse_blk = reinterpret_cast<float*>(w + stat);
  float* dq = reinterpret_cast<float*>(w + 2 * stat);
  BwdParts bp;
  if (!plan(p, d, &g, &bp)) return hipErrorInvalidDevice;
  g.parts = 1;
  float* dk = dq + bp.q * out_floats(p, p.heads);
  float* dv = dk + bp.kv * out_floats(p, p.kv_heads);
  const size_t parts = (bp.q * out_floats(p, p.heads) + 2 * bp.kv * out_floats(p, p.kv_heads)) * sizeof(float);
  void* ds = w + 2 * stat + up256(parts);
  const int chunk = chunk_of(p, d, g), total = slots_of(p);
  for (int pass = 0; pass < 2; ++pass) {                       // everything that can fail on the host first
    if (pass == 1) {
      trace_mark(s);
      const hipError_t e = launch_delta_grid(map_of(p, p.heads, 0, 1), p.hdim, p.o, p.g, (const bf16_t*)O,
                                             (const bf16_t*)dO, lse, delta, lse_blk, s);
      if (e != hipSuccess) return e;
    }
    for (int t = 0; t < total; t += chunk) {                   // Alg. 3 line 3, every tile
      g.b.first = t;
      g.b.n = total - t < chunk ? total - t : chunk;
      const hipError_t e = launch_bwd_mfma(pass == 0 ? PREPARE : LAUNCH, d, g, Q, K, V, O, dO, lse_blk, delta, dq, dk, dv,
                                           ds, bp, s);
      if (e != hipSuccess) return e;
    }
  }
  SumSet sets[3];
  memset(sets, 0, sizeof(sets));
  for (int x = 0; x < p.side; ++x) {
    for (int z = 0; z < bp.q; ++z)
      sets[0].p.p[x * bp.q + z] = dq + (size_t)(z * (int)slots + col_slot(g.b, x, x) - x) * p.heads * rows * p.hdim;
    for (int z = 0; z < bp.kv; ++z) {
      const size_t at = (size_t)(z * (int)slots + row_slot(g.b, x, 0)) * p.kv_heads * rows * p.hdim;
      sets[1].p.p[x * bp.kv + z] = dk + at;
      sets[2].p.p[x * bp.kv + z] = dv + at;
    }
  }
  sets[0].gm = map_of(p, p.heads, 1, bp.q);
  sets[1].gm = sets[2].gm = map_of(p, p.kv_heads, 2, bp.kv);
  sets[0].out = dQ;
  sets[1].out = dK;
  sets[2].out = dV;
  sets[0].lo = p.dq;
  sets[1].lo = p.dk;
  sets[2].lo = p.dv;
  return launch_sum_grid(3, sets, p.hdim, A2D_BF16, s);        // Alg. 3 lines 4-5
}

}  // namespace a2d
