// bf16 MFMA backward of calls with few rows and keys, in one launch and without partial results: the counterpart of
// a2d_fwd_small.hip.
//
// Two kinds of workgroups side by side, both with 32 rows that all eight wavefronts hold and a walk that they share
// by slabs of 32: dQ workgroups (32 queries; the slabs are keys) and dK / dV workgroups (32 keys; the slabs are
// queries).  A wavefront stages its slabs in LDS of its own and keeps partial accumulators of the 32 rows; the
// eight are added up through LDS at the end.  No barrier during the walk, no sums in memory, no second launch.
// dK / dV workgroups compute delta of the rows they stage, from O.
// Where all of them run at once with dK and dV in workgroups of their own, these are (S is computed once more): one accumulator leaves
// the registers for a turn of loads ahead, and half of the sums to add up at the end.  A turn of dK / dV was 1.9 us, now 1.3, and the sums
// 2.9, now 1.4 (2 heads, 512 tokens on 2 x 2, H = 128).  Beyond one workgroup a compute unit the work counts, not the latency: 4 heads, 838 tokens,
// H = 80 23.8 us together, 29.1 apart, 17 x 192 x 365 10.0 / 11.7.
//
// What bounds it: launch, argument and first-load latencies below two rounds of slabs; then the 16-byte loads of the
// staging, which every 32 rows or keys do for all they meet (24 a lane and round for dK / dV; 2.7 us a round at H = 128,
// its MFMAs take 0.9; delta from unpacked products was a third of its vector instructions, 3.0 us).  The 32 rows' own operands come in
// once for all wavefronts, through LDS: fragments loaded by each of the eight are 24 instructions of 64 scattered pieces, 3 us before the first
// slab of a dQ workgroup could be used, 1.5 now.  Registers: dK, dV and one slab of loads fill the 256 of a wavefront at H = 128,
// so there the second slab is loaded under the first contraction only, and the fixed operands are read from LDS.
// (The second slab straight into LDS: 0.88 to 1.0 on long walks of few workgroups, since the wait for the first one's registers is then a
// wait for it too.)
// Measured, against workgroups of 128 and more rows with their walks in parts: H = 64 8 x 512 x 512 19.1 -> 8.2 us, 4 x 1024 x
// 1024 22.6 -> 11.3, 1 x 128 x 128 10.1 -> 4.7; H = 128 26.9 -> 12.4, 28.5 -> 18.3, 13.4 -> 6.0, 2 x 2048 x 2048 36.6 -> 30.
#include "a2d_bwd.hpp"

namespace a2d {
namespace {

using namespace mfma;

constexpr int LANES = 8;                           // wavefronts
// Kinds of workgroups: dQ of 32 queries; dK and dV of 32 keys, or one of the two
enum Kind32 { ROWS_DQ, KEYS_BOTH, KEYS_DK, KEYS_DV };
// LDS rows of 256 bytes (H = 64: 128); chunk c of 16 bytes of row r lies at c ^ mix(r), so that a natural read (16 rows, one
// chunk), a transposing one (four rows, four chunks) and a store (a whole row) each meet every bank once.
template <int HR>
struct Lds {
  static constexpr int CHUNKS = HR == 64 ? 8 : 16, ROW = 16 * CHUNKS, SLAB = 32 * ROW;
  static __device__ __forceinline__ int mix(int r) { return CHUNKS == 16 ? ((r & 3) << 2) | ((r >> 2) & 3) : ((r & 2) << 1) | ((r >> 2) & 3); }
  // every wavefront's { first, second slab } | the workgroup's fixed rows: K, V or Q, dO | every wavefront's { lse, -delta } of a slab
  static constexpr int FIXED_AT = LANES * 2 * SLAB, STAT_AT = FIXED_AT + 2 * SLAB, STAT_BYTES = 2 * 32 * 4;
  static constexpr int BYTES = STAT_AT + LANES * STAT_BYTES;
};

typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) float lds_float;

// Per slab: S from the first slab (K, or Q) and the fixed rows' Q, or K; dP from the second (V, or dO) and their dO, or V;
// dQ += K^T dS, or dV += dO^T P and dK += Q^T dS.
// GRID: rows of a whole emulated grid, walked as in dq_rows and dkdv_pairs.  id: the workgroup's number among its kind.
template <int HR, int KIND, int GRID, bool AHEAD>
__device__ __forceinline__ void small_rows(
    int id, char* const lds, const a2d_tile_desc& d, const SegList& g, const bf16_t* __restrict__ Q,
    const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ O,
    const bf16_t* __restrict__ dO, const float* __restrict__ lse, float* __restrict__ dQ, float* __restrict__ dK,
    float* __restrict__ dV) {
  constexpr int HD = padded_head(HR), H = HR, KS = (HR + 15) / 16, CT = HD / 32;
  constexpr bool PLAIN = GRID == 0, CYCLIC = GRID == 2, KV = KIND != ROWS_DQ, HAS_DK = KIND == KEYS_BOTH || KIND == KEYS_DK,
                 HAS_DV = KIND == KEYS_BOTH || KIND == KEYS_DV, HAS_DP = KIND != KEYS_DV;
  constexpr int CHUNKS = Lds<HR>::CHUNKS, ROW = Lds<HR>::ROW, SLAB = Lds<HR>::SLAB, FIXED_AT = Lds<HR>::FIXED_AT, STAT_AT = Lds<HR>::STAT_AT;
  constexpr auto mix = Lds<HR>::mix;
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int kl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int half = lane >> 5, l32 = lane & 31;
  const float c = d.scale * kLog2e;
  const int by_size = GRID ? d.causal : g.by_size, sides = GRID ? g.b.side : 1;
  const int side = CYCLIC ? sides : 1;             // row blocks, or columns, that are walked in turn

  // ---- the workgroup's rows: block `blk` of 32 of key/value head `kvh` (query head `head`), of row block or column `place`
  const int nb = ((KV ? d.nkv : d.nq) + 31) / 32, group = g.group;
  int kvh, blk, head;
  if (!xcd_map(id, d.heads / group, sides * (KV ? 1 : group) * nb, by_size != 0, kvh, blk, KV ? 0 : kXcdCus)) return;
  head = kvh;                                      // (no divisions by one: they delay the first loads)
  if (group > 1) {
    head = kvh * group;
    if constexpr (!KV) {
      const int by = GRID || by_size ? group : nb, q = blk / by, r = blk - q * by;
      head += GRID || by_size ? r : q;
      blk = GRID || by_size ? q : r;
    }
  }
  int place = 0;
  if constexpr (GRID != 0) {
    const GridBlock gb = KV ? grid_column(g.b, nb, blk) : grid_block(g.b, nb, blk);
    place = gb.r;
    blk = gb.blk;
  }
  const int r0 = 32 * (KV ? blk : nb - 1 - blk);   // (heavy blocks first under a causal mask)
  const int row = r0 + l32, row_ld = min(row, (KV ? d.nkv : d.nq) - 1);
  const bool row_ok = row < (KV ? d.nkv : d.nq);
  Q += (int64_t)head * d.lq.head + (GRID && !KV ? place * g.b.q : 0);
  O += (int64_t)head * d.lo.head + (GRID && !KV ? place * g.b.o : 0);
  dO += (int64_t)head * d.ldo.head + (GRID && !KV ? place * g.b.g : 0);
  K += (int64_t)kvh * d.lk.head + (GRID && KV ? place * g.b.k : 0);
  V += (int64_t)kvh * d.lv.head + (GRID && KV ? place * g.b.v : 0);

  // ---- staging of slabs: a lane moves one 16-byte chunk of ST_N rows (chunks past the head size: its last one once more,
  // into columns whose results are not stored; a branch around them costs 3 % at H = 96).  AHEAD: all of a turn's loads are under
  // way during the turn before (two accumulators leave registers for one slab at a time; and where a compute unit runs several
  // workgroups one after the other, or dK / dV need all the memory gives, one slab at a time is the better order: 13 heads, 404 tokens
  // on 2 x 2, H = 128 24.6 us with all ahead in the dQ workgroups, 23.9 without, 6 x 1589 x 1902, H = 64 39.1 / 37.1).  dQ beside dK and dV
  // apart: at H = 64 alone, where it is worth 1 %; at H = 80 and more walks of many keys lose up to a tenth by it, those of few a hundredth at most
  // without (ahead / not: 2 x 197 x 1353, H = 80 13.5 / 12.4, H = 128 15.5 / 14.1, 1 x 560 x 1680, H = 128 19.0 / 17.3, 4 x 181 x 550, H = 80 8.6 / 8.0).
  constexpr int ST_ROWS = 64 / CHUNKS, ST_N = 32 / ST_ROWS;
  const int st_row = lane / CHUNKS, st_chunk = lane % CHUNKS;
  const unsigned first_area = lds_base + kl * 2 * SLAB;
  unsigned st_at = first_area + st_row * ROW + 16 * (st_chunk ^ mix(st_row));
  u32x4 xr[ST_N], yr[AHEAD ? ST_N : 1], zr[HAS_DK ? ST_N : 1];       // the first slab's rows, the second's (else in xr too), those of O
  // rows at, at + row_bytes, .. of a slab, from row `first` on; those from `last` on re-read row `last`
  auto load = [&](u32x4 (&x)[ST_N], gptr_t base, unsigned at, unsigned row_bytes, int first, int last) {
    const int ln = lane_again(), st_row = ln / CHUNKS, st_chunk = min(ln % CHUNKS, H / 8 - 1);
#pragma unroll
    for (int p = 0; p < ST_N; ++p)
      x[p] = gload_b128(base, at + __umul24((unsigned)min(first + st_row + ST_ROWS * p, last), row_bytes) + 16 * st_chunk);
  };
  auto store = [&](const u32x4 (&x)[ST_N], int second) {
#pragma unroll
    for (int p = 0; p < ST_N; ++p)                 // (mix of row st_row + ST_ROWS p: that of st_row, bits flipped)
      *reinterpret_cast<lds_u32x4*>((uintptr_t)((st_at ^ (CHUNKS == 16 ? 16 * (p & 3) : 32 * (p & 1))) + second * SLAB +
                                                p * ST_ROWS * ROW)) = x[p];
  };
  // fragment reads: natural fragment x, transposed fragment of column tile t, rows 16 u ..
  unsigned nat_at = first_area + l32 * ROW + 16 * (half ^ mix(l32));
  const int g16 = lane >> 4, j16 = lane & 15, tr_row = 4 * (g16 >> 1) + (j16 >> 2);
  unsigned tr_at = first_area + tr_row * ROW + 16 * ((2 * (g16 & 1) + ((j16 & 3) >> 1)) ^ mix(tr_row)) + 8 * (j16 & 1);
  auto natural = [&](int second, int x) { return lds_load_b128((nat_at ^ (32 * x)) + second * SLAB); };
  auto transposed = [&](int second, int u, int t) {
    const unsigned at = second * SLAB + 16 * u * ROW;
    return lds_load_tr((tr_at ^ (64 * t)) + at, (tr_at ^ (64 * t) ^ 32) + at + 8 * ROW);
  };

  // ---- the fixed rows' operands, which come in once for all wavefronts: then in registers, or (two accumulators to hold) in LDS
  constexpr bool FIXED_LDS = KIND == KEYS_BOTH || (AHEAD && HD > 96);
  const unsigned to_fixed = FIXED_AT - kl * 2 * SLAB;
  bf16x8 f1[FIXED_LDS ? 1 : KS], f2[FIXED_LDS ? 1 : KS];
  auto fixed_lds = [&](int x, int second) { return lds_load_b128((nat_at ^ (32 * x)) + to_fixed + second * SLAB); };
  auto fixed1 = [&](int x) { return FIXED_LDS ? fixed_lds(x, 0) : f1[FIXED_LDS ? 0 : x]; };
  auto fixed2 = [&](int x) { return FIXED_LDS ? fixed_lds(x, 1) : f2[FIXED_LDS ? 0 : x]; };
  float lse2 = 0.f, del = 0.f;                     // of the lane's query (dQ)

  // ---- the walk: entry e, e + LANES, .. of (sub-block, slab) as in fwd_small_kernel (dQ), or of (query head, slab, row block)
  const int nq = GRID == 1 ? sides * d.nq : d.nq, head_rows = nq * side;
  const int key_rows = GRID == 1 ? sides * d.nkv : d.nkv;
  int sb = 0, j = 0, n = 0, start = 0, rows = key_rows, nfull = 0, my_vis = 0;      // dQ: as in fwd_small_kernel
  int64_t rel = 0;
  const int segs = PLAIN ? g.n : side, shift_from = CYCLIC && d.causal ? place : segs;
  const int last_row = min(r0 + 31, d.nq - 1);
  auto vis_count = [&](int i) -> int {
    if (GRID == 1) return d.causal ? place * d.nq + i + 1 : rows;
    if (GRID == 2) return d.causal ? i + 1 : rows;
    if (!d.causal) return rows;
    const int64_t v = (int64_t)i + rel + 1;
    return v <= 0 ? 0 : (v < rows ? (int)v : rows);
  };
  auto enter_segment = [&]() {
    nfull = vis_count(r0);
    my_vis = vis_count(row_ld);
  };
  auto open_segment = [&](int s) {
    for (n = 0; s < segs; ++s) {
      if (PLAIN) {
        start = g.seg[s].start;
        rows = g.seg[s].rows;
        rel = g.seg[s].rel;
      }
      n = (vis_count(last_row) + 31) / 32;
      if (n > 0) break;
    }
    sb = s;
  };
  auto advance = [&](int by) {
    if constexpr (CYCLIC) {
      const int q = by / segs;
      j += q;
      sb += by - q * segs;
      if (sb >= segs) { sb -= segs; ++j; }
      if (j >= n) sb = segs;
    } else {
      j += by;
      while (A2D_SELDOM(j >= n)) {
        if (sb >= segs) break;
        j -= n;
        open_segment(sb + 1);
      }
    }
  };
  const unsigned x_row = __builtin_amdgcn_readfirstlane((unsigned)(KV ? d.lq.row : d.lk.row) * 2);
  const unsigned y_row = __builtin_amdgcn_readfirstlane((unsigned)(KV ? d.ldo.row : d.lv.row) * 2);
  const unsigned x_blk = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)((KV ? g.b.q : g.b.k) * 2)) : x_row;
  const unsigned y_blk = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)((KV ? g.b.g : g.b.v) * 2)) : y_row;
  const unsigned o_row = KV ? __builtin_amdgcn_readfirstlane((unsigned)d.lo.row * 2) : 0;
  const gptr_t x_base = uniform_gptr(KV ? Q : K), y_base = uniform_gptr(KV ? dO : V), o_base = uniform_gptr(O);

  // dK / dV: which rows see which keys, as in dkdv_wide
  const int col_first = GRID == 1 && d.causal ? place * d.nkv : 0;
  auto seg_first_row = [&](int s, int r) -> int {
    const int64_t f = (int64_t)(r - g.seg[s].start) - g.seg[s].rel;
    return f <= 0 ? 0 : (f >= d.nq ? d.nq : (int)f);
  };
  int i_start = 0, w_all = 0, nsteps = 0, total = 0, my_first = nq;
  int e = kl, eh = 0, es = 0, er = 0;              // this entry, its query head of the group, slab, row block
  auto locate = [&]() {
    eh = group > 1 ? e / (nsteps * side) : 0;
    es = group > 1 ? e - eh * (nsteps * side) : e;
    if constexpr (CYCLIC) {
      er = es % side;
      es /= side;
    }
  };
  const int late = CYCLIC && d.causal ? place : 0;
  if constexpr (KV) {
    int lo = nq, hi = 0;
    if (!d.causal) lo = 0;
    else if (GRID) {
      lo = col_first + r0;
      hi = col_first + min(r0 + 32, d.nkv) - 1;
    } else {
      for (int s = 0; s < g.n; ++s) {
        const int x = max(r0, g.seg[s].start), y = min(min(r0 + 32, d.nkv), g.seg[s].start + g.seg[s].rows);
        if (x >= y) continue;
        lo = min(lo, seg_first_row(s, x));
        hi = max(hi, seg_first_row(s, y - 1));
      }
    }
    i_start = lo / 32 * 32;
    w_all = r0 + 32 > d.nkv ? nq : hi;
    nsteps = (nq - i_start + 31) / 32;
    total = nsteps * side * group;
    if (row_ok) {                                  // the first row that sees the lane's key; no row sees padding keys
      my_first = GRID && d.causal ? col_first + row : 0;
      if (!GRID && d.causal)
        for (int s = 0; s < g.n; ++s)
          if (row >= g.seg[s].start && row < g.seg[s].start + g.seg[s].rows) my_first = seg_first_row(s, row);
    }
    if (e < total) locate();
  } else {
    open_segment(0);
    if (sb < segs) advance(kl);
    if (sb < segs) enter_segment();
  }
  float stat = 0.f;                                // lse of query l32 of the slab (dK / dV)
  const float* lse_at = lse + (int64_t)head * (GRID ? sides : 1) * d.nq;
  auto here = [&]() { return KV ? e < total : sb < segs; };
  auto load_first = [&]() {
    if constexpr (KV) {
      const int i0 = i_start + 32 * es;
      load(xr, x_base, eh * (unsigned)(d.lq.head * 2) + (CYCLIC ? er * x_blk : 0u), x_row, i0, nq - 1);
      const int i = min(i0 + l32, nq - 1);
      stat = lse_at[eh * head_rows + (CYCLIC ? i * side + er : i)];
    } else {
      if (CYCLIC) start = sb;
      load(xr, x_base, start * x_blk, x_row, 32 * j, rows - 1);
    }
  };

  auto load_second = [&](u32x4 (&y)[ST_N]) {       // and O
    if constexpr (KV) {
      const int i0 = i_start + 32 * es;
      load(y, y_base, eh * (unsigned)(d.ldo.head * 2) + (CYCLIC ? er * y_blk : 0u), y_row, i0, nq - 1);
      if constexpr (HAS_DK) load(zr, o_base, eh * (unsigned)(d.lo.head * 2) + (CYCLIC ? er * (unsigned)(g.b.o * 2) : 0u), o_row, i0, nq - 1);
    } else {
      load(y, y_base, start * y_blk, y_row, 32 * j, rows - 1);
    }
  };
  // sum over the lanes that hold a row's chunks, in the order of dq_rows (one delta for all gradients)
  auto row_total = [](float t, int lanes) {
    t += lane_swap<0xB1>(t);
    t += lane_swap<0x4E>(t);
    t += lane_swap<0x141>(t);
    return lanes == 16 ? t + lane_swap<0x140>(t) : t;
  };
  {                                                // a thread moves a chunk of both
    const int fr = threadIdx.x >> 4, fc = threadIdx.x & 15, at_row = min(r0 + fr, (KV ? d.nkv : d.nq) - 1), at_col = 8 * min(fc, H / 8 - 1);
    const bf16_t* const p1 = KV ? K + (int64_t)at_row * d.lk.row : Q + (int64_t)at_row * d.lq.row;
    const bf16_t* const p2 = KV ? V + (int64_t)at_row * d.lv.row : dO + (int64_t)at_row * d.ldo.row;
    const u32x4 a = *reinterpret_cast<const u32x4*>(p1 + at_col);
    u32x4 b = {}, o = {};
    float l = 0.f;
    if constexpr (HAS_DP) b = *reinterpret_cast<const u32x4*>(p2 + at_col);
    if constexpr (!KV) {
      o = *reinterpret_cast<const u32x4*>(O + (int64_t)at_row * d.lo.row + at_col);
      l = lse_at[GRID ? grid_token(g.b, d.nq, place, at_row) : at_row];
    }
    // (Behind this branch the compiler waits for the slab too, not for the fixed rows alone, in front of the barrier.  Without it wavefronts that
    // have no entry load for nothing: grids and walks of eight slabs and more 1 to 2 % faster, shorter ones up to a tenth slower, 2 x 96 x 113,
    // H = 80 5.8 -> 6.4 us, 26 x 290 x 91, H = 96 10.3 -> 10.7.)
    if (here()) {
      load_first();
      if constexpr (AHEAD) load_second(yr);
    }
    if (8 * fc < H) {
      const unsigned at = lds_base + FIXED_AT + fr * ROW + 16 * (fc ^ mix(fr));
      *reinterpret_cast<lds_u32x4*>((uintptr_t)at) = a;
      if constexpr (HAS_DP) *reinterpret_cast<lds_u32x4*>((uintptr_t)(at + SLAB)) = b;
    }
    if constexpr (!KV) {                           // delta and lse, one lane's for all
      const float t = row_total(8 * fc < H ? dot8(o, b, 0.f) : 0.f, 16);
      *reinterpret_cast<lds_float*>((uintptr_t)(lds_base + STAT_AT + 4 * fr)) = t;
      *reinterpret_cast<lds_float*>((uintptr_t)(lds_base + STAT_AT + 128 + 4 * fr)) = l == -INFINITY ? INFINITY : l * kLog2e;   // +inf: exp2(s - lse2) = 0
    }
  }
  __syncthreads();
  if constexpr (!KV) {
    del = *reinterpret_cast<lds_float*>((uintptr_t)(lds_base + STAT_AT + 4 * l32));
    lse2 = *reinterpret_cast<lds_float*>((uintptr_t)(lds_base + STAT_AT + 128 + 4 * l32));
  }
  if constexpr (!FIXED_LDS) {
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      f1[x] = fixed_lds(x, 0);
      if constexpr (HAS_DP) f2[x] = fixed_lds(x, 1);
    }
  }

  f32x16 acc[HAS_DP ? CT : 1], acc2[HAS_DV ? CT : 1];      // dQ, or dK; dV
#pragma unroll
  for (int t = 0; t < CT; ++t) acc[HAS_DP ? t : 0] = acc2[HAS_DV ? t : 0] = zero16();
  const unsigned stat_at = lds_base + STAT_AT + kl * Lds<HR>::STAT_BYTES;

  // slab . fixed rows, the operands two ahead of their use
  auto contract = [&](int second, auto fixed, f32x16& r) {
    bf16x8 a[2], b[2];
    auto ld = [&](auto X) {
      constexpr int x = decltype(X)::value;
      if constexpr (x < KS) {
        a[x % 2] = natural(second, x);
        b[x % 2] = fixed(x);
      }
    };
    static_for<0, 2>(ld);
    static_for<0, KS>([&](auto X) {
      constexpr int x = decltype(X)::value;
      r = mma(a[x % 2], b[x % 2], r);
      ld(std::integral_constant<int, x + 2>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  while (here()) {
    // (fragment addresses are computed at each use: kept over the loop they cost 30 registers)
    asm volatile("" : "+v"(st_at), "+v"(nat_at), "+v"(tr_at));
    const int i0 = KV ? i_start + 32 * es : 0;
    const int sh = KV && CYCLIC && er < late ? 1 : 0;
    const int k0 = KV ? 0 : 32 * j + (CYCLIC && sb > shift_from);
    // -delta = -rowsum(dO o O), CHUNKS lanes a row
    auto own_delta = [&](const u32x4 (&y)[ST_N]) {
      const int ln = lane_again();
#pragma unroll
      for (int p = 0; p < ST_N; ++p) {
        float t = dot8(zr[HAS_DK ? p : 0], y[p], 0.f);
        if (8 * CHUNKS != H) t = ln % CHUNKS * 8 < H ? t : 0.f;
        *reinterpret_cast<lds_float*>((uintptr_t)(stat_at + 128 + 4 * (ln / CHUNKS + ST_ROWS * p))) = -row_total(t, CHUNKS);   // (all lanes of a row)
      }
    };
    const int sb_now = sb;
    bool masked;
    int first = 0;
    unsigned limit = 0;
    auto next = [&]() {                            // the next slab
      if constexpr (KV) {
        masked = i0 - sh < w_all || i0 + 32 > nq;
        first = i0 - sh + 4 * half - my_first;
        limit = max(nq - sh - my_first, 0);
        e += LANES;
        if (e < total) locate();
      } else {
        masked = k0 + 32 > nfull;
        advance(LANES);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (here()) {
        load_first();
        if constexpr (AHEAD) load_second(yr);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    store(xr, 0);
    if constexpr (KV) {
      if (half == 0)
        *reinterpret_cast<lds_float*>((uintptr_t)(stat_at + 4 * l32)) =
            i0 + l32 >= nq || stat == -INFINITY ? INFINITY : stat * kLog2e;
    }
    if constexpr (AHEAD) {
      store(yr, 1);
      if constexpr (HAS_DK) own_delta(yr);
      next();
    } else {
      load_second(xr);
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s = zero16();
    contract(0, [&](int x) { return fixed1(x); }, s);
    asm volatile("" : "+v"(s));                    // (here, not where it is first used)
    if constexpr (!AHEAD) {
      store(xr, 1);
      if constexpr (HAS_DK) own_delta(xr);
      next();
    }
    f32x16 dp = zero16();
    if constexpr (HAS_DK) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = lds_load_f32x4(stat_at + 128 + 32 * q + 16 * half);
#pragma unroll
        for (int i = 0; i < 4; ++i) dp[4 * q + i] = v[i];
      }
    }
    if constexpr (HAS_DP) contract(1, [&](int x) { return fixed2(x); }, dp);
    // register r <-> row or key 8 (r >> 2) + 4 half + (r & 3) of the slab
    if (masked) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int at = 8 * (r >> 2) + (r & 3);
        if (KV ? (unsigned)(first + at) >= limit : k0 + 4 * half + at >= my_vis) s[r] = -INFINITY;
      }
    }
    bf16x8 pb[2], sb8[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 l = {lse2, lse2, lse2, lse2};
      if constexpr (KV) l = lds_load_f32x4(stat_at + 32 * q + 16 * half);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * q + i;
        const float p = fast_exp2(fmaf(s[r], c, -l[i]));
        if constexpr (HAS_DV) pb[r >> 3][r & 7] = (bf16_t)p;
        if constexpr (HAS_DP) sb8[r >> 3][r & 7] = (bf16_t)(p * (KV ? dp[r] : dp[r] - del));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // (fragments two ahead of their use; dV, then dQ or dK)
    constexpr int N2 = HAS_DV ? 2 * CT : 0, N = N2 + (HAS_DP ? 2 * CT : 0);
    bf16x8 a[2];
    auto ld = [&](auto I) {
      constexpr int i = decltype(I)::value, y = i < N2 ? i : i - N2;
      if constexpr (i < N) a[i % 2] = transposed(i < N2, y / CT, y % CT);
    };
    static_for<0, 2>(ld);
    static_for<0, N>([&](auto I) {
      constexpr int i = decltype(I)::value, y = i < N2 ? i : i - N2;
      if constexpr (i < N2) acc2[HAS_DV ? y % CT : 0] = mma(a[i % 2], pb[y / CT], acc2[HAS_DV ? y % CT : 0]);
      else acc[HAS_DP ? y % CT : 0] = mma(a[i % 2], sb8[y / CT], acc[HAS_DP ? y % CT : 0]);
      ld(std::integral_constant<int, i + 2>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    if (!KV && !CYCLIC && sb != sb_now && sb < segs) enter_segment();
  }

  // ---- the wavefronts' sums: pieces of four columns, [wavefront][piece][lane]; each adds up and stores its share of them
  static_assert(LANES * CT * 4 * 1024 <= Lds<HR>::BYTES, "the pieces must fit");
  f32x4* const x = reinterpret_cast<f32x4*>(lds);
  const int ln = lane_again(), to = r0 + (ln & 31), col0 = 4 * (ln >> 5);
  const bool to_ok = to < (KV ? d.nkv : d.nq);
  auto finish = [&](const f32x16 (&a)[CT], float mul, float* out, bf16_t* out16, bool add) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        x[(kl * 4 * CT + t * 4 + q) * 64 + ln] = f32x4{a[t][4 * q], a[t][4 * q + 1], a[t][4 * q + 2], a[t][4 * q + 3]};
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (4 * CT + LANES - 1) / LANES; ++i) {
      const int piece = kl + LANES * i, col = 32 * (piece >> 2) + 8 * (piece & 3) + col0;
      if (piece >= 4 * CT || col >= H || !to_ok) continue;
      f32x4 v = x[piece * 64 + ln];
#pragma unroll
      for (int k = 1; k < LANES; ++k) {
        const f32x4 w = x[(k * 4 * CT + piece) * 64 + ln];
        v[0] += w[0]; v[1] += w[1]; v[2] += w[2]; v[3] += w[3];
      }
      if constexpr (GRID != 0) {
        bf16x4 b;
#pragma unroll
        for (int k = 0; k < 4; ++k) b[k] = (bf16_t)(v[k] * mul);
        *reinterpret_cast<bf16x4*>(out16 + col) = b;
      } else {
        f32x4* const o = reinterpret_cast<f32x4*>(out + col);
        f32x4 r = {v[0] * mul, v[1] * mul, v[2] * mul, v[3] * mul};
        if (add) {
          const f32x4 old = *o;
          r[0] += old[0]; r[1] += old[1]; r[2] += old[2]; r[3] += old[3];
        }
        *o = r;
      }
    }
  };
  const auto out16 = [&](float* p, int w, int h) {
    return reinterpret_cast<bf16_t*>(p) + h * g.b.out[w].head + place * g.b.out_step[w] + to * g.b.out[w].row;
  };
  if constexpr (KV) {
    const int64_t at = ((int64_t)kvh * d.nkv + to) * H;
    if constexpr (HAS_DV) finish(acc2, 1.0f, dV + (GRID ? 0 : at), GRID ? out16(dV, 2, kvh) : nullptr, false);
    if constexpr (HAS_DK) finish(acc, d.scale, dK + (GRID ? 0 : at), GRID ? out16(dK, 1, kvh) : nullptr, false);
  } else {
    finish(acc, d.scale, dQ + (GRID ? 0 : ((int64_t)head * d.nq + to) * H), GRID ? out16(dQ, 0, head) : nullptr, g.acc != 0);
  }
}

// SPLIT: dK and dV of 32 keys in workgroups of their own (`first` of them each, then those for dQ); else `first` workgroups of the kind
// that goes first, then the others
template <int HR, int GRID, bool SPLIT>
__global__ __launch_bounds__(64 * LANES, 1) void bwd_small_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, const bf16_t* __restrict__ O, const bf16_t* __restrict__ dO,
    const float* __restrict__ lse, float* __restrict__ dQ, float* __restrict__ dK, float* __restrict__ dV, int first,
    int q_first) {
  warm_arguments<9 * 8 + 8>();
  extern __shared__ __attribute__((aligned(256))) char lds[];
  const int at = blockIdx.x;
  if constexpr (SPLIT) {
    if (at < first) small_rows<HR, KEYS_DK, GRID, true>(at, lds, d, g, Q, K, V, O, dO, lse, dQ, dK, dV);
    else if (at < 2 * first) small_rows<HR, KEYS_DV, GRID, true>(at - first, lds, d, g, Q, K, V, O, dO, lse, dQ, dK, dV);
    else small_rows<HR, ROWS_DQ, GRID, HR == 64>(at - 2 * first, lds, d, g, Q, K, V, O, dO, lse, dQ, dK, dV);
  } else {
    const int id = at < first ? at : at - first;
    if ((at < first) == (q_first != 0)) small_rows<HR, ROWS_DQ, GRID, false>(id, lds, d, g, Q, K, V, O, dO, lse, dQ, dK, dV);
    else small_rows<HR, KEYS_BOTH, GRID, false>(id, lds, d, g, Q, K, V, O, dO, lse, dQ, dK, dV);
  }
}

template <int HR, int GRID, bool SPLIT>
hipError_t go_split(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                    const void* O, const void* dO, const float* lse, float* dQ, float* dK, float* dV, int q_first, hipStream_t s) {
  constexpr int bytes = Lds<HR>::BYTES;
  if (ph == PREPARE) return ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_small_kernel<HR, GRID, SPLIT>), bytes);
  const int side = GRID ? g.b.side : 1, kv_heads = d.heads / g.group;
  const int n_kv = xcd_grid(kv_heads, side * ((d.nkv + 31) / 32)), n_q = xcd_grid(kv_heads, side * g.group * ((d.nq + 31) / 32));
  A2D_LAUNCH((bwd_small_kernel<HR, GRID, SPLIT>), dim3((SPLIT ? 2 : 1) * n_kv + n_q), dim3(64 * LANES), bytes, s, d, g,
             (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, (const bf16_t*)dO, lse, dQ, dK, dV,
             !SPLIT && q_first ? n_q : n_kv, q_first);
  return hipGetLastError();
}
template <int HR, int GRID>
hipError_t go(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
              const void* O, const void* dO, const float* lse, float* dQ, float* dK, float* dV, int q_first, int split, hipStream_t s) {
  return split ? go_split<HR, GRID, true>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, s)
               : go_split<HR, GRID, false>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, s);
}
template <int GRID>
hipError_t go_h(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                const void* O, const void* dO, const float* lse, float* dQ, float* dK, float* dV, int q_first, int split, hipStream_t s) {
  switch (d.hdim) {
    case 128: return go<128, GRID>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s);
    case 96: return go<96, GRID>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s);
    case 80: return go<80, GRID>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s);
    default: return go<64, GRID>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s);
  }
}

}  // namespace

hipError_t launch_bwd_small(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                            const void* V, const void* O, const void* dO, const float* lse, float* dQ, float* dK,
                            float* dV, int q_first, int split, hipStream_t s) {
  return g.b.side == 0 ? go_h<0>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s)
         : g.b.cyclic  ? go_h<2>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s)
                       : go_h<1>(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, q_first, split, s);
}

}  // namespace a2d
