// The dK/dV workgroup of 128 keys, in pairs of wavefronts (see a2d_bwd_mfma.hip for the kernels).
#pragma once
#include <type_traits>

#include "a2d_bwd.hpp"

namespace a2d {
namespace mfma {

constexpr int DK_THREADS = 512;
constexpr int DK_KEYS = 128;      // keys per workgroup
constexpr int DK_NBUF = 4;        // tile buffers: gradient waves' step, score waves' step, next, incoming
// LDS: [buf]{ Q tile, dO tile } (dual layout, 32 rows each) | [buf]{ lse*log2e [32], delta [32] } |
//      (the latter negated) | [slot][pair] probabilities handed from the score wave to the gradient wave (fp32)
constexpr int DK_STAT = DK_NBUF * DK_BUF;
constexpr int DK_MBOX = DK_STAT + DK_NBUF * DK_STAT_BUF;
constexpr int DK_MBOX_PIECE = 32 * 32 * 4;
constexpr int DK_MBOX_SLOT = 4 * DK_MBOX_PIECE;
constexpr int DK_LDS = DK_MBOX + 2 * DK_MBOX_SLOT;

// Per-wavefront state.  The two roles run the same contraction code on different operands:
//   score wave (role 0):    frag = K^T fragments, natural reads from the Q tile,
//                           transposed reads from the dO tile, acc = dV^T
//   gradient wave (role 1): frag = V^T fragments, natural reads from the dO tile,
//                           transposed reads from the Q tile, acc = dK^T
template <int HD>
struct DkCtx {
  f32x16 acc[HD / 32];
  bf16x8 frag[HD / 16];
  unsigned nat_e, nat_o, tr_lo, tr_hi;   // dual-layout bases in the tile buffer of this wave's step
  unsigned stat;        // lse (role 0) or delta (role 1) row of that buffer, + 16 * half
  unsigned mbox;        // this lane's place in the pair's mailbox, slot of this wave's step
  float c;
  int my_first;         // first local query row that sees this lane's key
  int half;
};

// Fragment addresses inside the wave's tile buffer (per-lane base + immediate)
#define A2D_NAT(X) lds_load_b128((((X) & 1) ? cx.nat_o : cx.nat_e) + 64 * ((X) >> 1))
#define A2D_TR(U, HT) \
  lds_load_tr(cx.tr_lo + (U) * 16 * DUAL_LD + 64 * (HT), cx.tr_hi + (U) * 16 * DUAL_LD + 64 * (HT))
#define A2D_FENCE __builtin_amdgcn_sched_barrier(0);

// First contraction of a 32-query x 32-key step (S = Q K^T or dP = dO V^T): HD / 16 MFMAs over
// H.  The natural fragments travel through a ring of four: dk_first_pre requests fragments
// 0..3, the body requests the others while it consumes those.  (The fences keep the compiler
// from sinking the requests down to their uses.)
template <int HD>
__device__ __forceinline__ void dk_first_pre(const DkCtx<HD>& cx, bf16x8 (&n)[4]) {
  n[0] = A2D_NAT(0); n[1] = A2D_NAT(1); n[2] = A2D_NAT(2); n[3] = A2D_NAT(3);
  A2D_FENCE
}
// `init` is the starting value of the sum (zero for S, -delta for dP - delta).  One chain (an MFMA
// accumulates onto the result of the one issued just before it without waiting: 33 cycles apart, as
// independent ones): adding up two costs 4-7 % of the call at H = 64 to 96; at H = 128 the two
// chains measured up to 2 % faster.
// KS: the slices that hold data (a head size of 80 fills five of the padded six)
template <int HD, int KS = HD / 16>
__device__ __forceinline__ f32x16 dk_first(const DkCtx<HD>& cx, bf16x8 (&n)[4], f32x16 init) {
  constexpr bool TWO = HD == 128;
  f32x16 s = init, s2 = zero16();
  static_for<0, KS>([&](auto X) {
    constexpr int x = decltype(X)::value;
    if constexpr (TWO && (x & 1)) s2 = mma(n[x & 3], cx.frag[x], s2); else s = mma(n[x & 3], cx.frag[x], s);
    if constexpr (x + 4 < KS) { n[x & 3] = A2D_NAT(x + 4); A2D_FENCE }
  });
  if constexpr (TWO) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] += s2[r];
  }
  return s;
}

// The 32 per-query statistics of the step (lse for the score wave, delta for the gradient wave)
// and the partner's probabilities, requested ahead of the first contraction.
template <int HD>
__device__ __forceinline__ void dk_stat_pre(const DkCtx<HD>& cx, f32x4 (&st)[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) st[g] = lds_load_f32x4(cx.stat + 8 * g * 4);
  A2D_FENCE
}
template <int HD>
__device__ __forceinline__ void dk_mbox_pre(const DkCtx<HD>& cx, f32x4 (&pm)[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) pm[g] = lds_load_f32x4(cx.mbox + g * 1024);
  A2D_FENCE
}

// score wave: P = exp2(c S - lse2), masked; handed on in fp32 and kept as bf16 B fragments.
// register r <-> query qs0 + 8*(r>>2) + 4*half + (r&3); lane <-> key.  (Queries from nq on are re-reads of the
// last one: their statistic of +inf makes p = 0 only while q.k is finite.)
template <bool MASK, int HD>
__device__ __forceinline__ void dk_probs(const DkCtx<HD>& cx, const f32x4 (&st)[4], f32x16& s,
                                         bf16x8 (&bf)[2], int qs0, int nq) {
  const int first = qs0 + 4 * cx.half - cx.my_first;
  const unsigned limit = max(nq - cx.my_first, 0);            // (padding keys: none)
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 p4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float p = fast_exp2(fmaf(s[4 * g + e], cx.c, -st[g][e]));
      if (MASK && (unsigned)(first + 8 * g + e) >= limit) p = 0.f;
      s[4 * g + e] = p;
      p4[e] = p;
    }
    *reinterpret_cast<__attribute__((address_space(3))) f32x4*>((uintptr_t)(cx.mbox + g * 1024)) = p4;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) bf[u] = pack8(s, 8 * u);
}

// gradient wave: dS = P o (dP - delta) from the partner's probabilities; `dpd` is dP - delta
// already (the contraction started from -delta)
__device__ __forceinline__ void dk_dscores(const f32x4 (&pm)[4], f32x16& dpd, bf16x8 (&bf)[2]) {
  f32x16& dp = dpd;
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) dp[4 * g + e] = pm[g][e] * dp[4 * g + e];
#pragma unroll
  for (int u = 0; u < 2; ++u) bf[u] = pack8(dp, 8 * u);
}

// Second contraction of a step (dV^T += dO^T P or dK^T += Q^T dS): 2 * HD / 32 MFMAs, A operands
// from the LDS transpose read, again through a ring (one fragment per 32-column tile of H):
// dk_second_pre requests those of the first 16 query rows (before the exponentials, so they
// arrive meanwhile), the body those of the second 16.
template <int HD>
__device__ __forceinline__ void dk_second_pre(const DkCtx<HD>& cx, bf16x8 (&t)[HD / 32]) {
  static_for<0, HD / 32>([&](auto HT) { constexpr int ht = decltype(HT)::value; t[ht] = A2D_TR(0, ht); });
  A2D_FENCE
}
template <int HD>
__device__ __forceinline__ void dk_second(DkCtx<HD>& cx, bf16x8 (&t)[HD / 32], const bf16x8 (&bf)[2]) {
  constexpr int CT = HD / 32;
  static_for<0, CT>([&](auto HT) {
    constexpr int ht = decltype(HT)::value;
    cx.acc[ht] = mma(t[ht], bf[0], cx.acc[ht]);
    t[ht] = A2D_TR(1, ht);
    A2D_FENCE
  });
  static_for<0, CT>([&](auto HT) {
    constexpr int ht = decltype(HT)::value;
    cx.acc[ht] = mma(t[ht], bf[1], cx.acc[ht]);
  });
}
#undef A2D_FENCE
#undef A2D_TR
#undef A2D_NAT

// HR: head size = row length in memory (64, 80, 96 or 128); the LDS tiles and fragments are laid out
// for the padded head size HD = padded_head(HR) (64, 96 or 128).
// GROUPED: several query heads per key/value head (g.group > 1); the plain kernel is compiled
// without the bookkeeping that walks them.
// WRITE_DS: the gradient waves also leave dS in the workspace `dS` (layout above) for the
// contraction-only dQ kernel.
// PLAIN: Q and dO are in the plain layout (row stride H, head stride nq * H): the staging offsets
// are then compile-time multiples and one offset serves both tensors (3 % on the recomputing path).
// GRID: all key blocks of an emulated grid, as in bwd_dkdv_wide_kernel.
// OWN_DELTA: computes delta = rowsum(dO o O) of the rows it stages, from O, in the order of sums of delta_kernel (the
// same bits); `delta` is not read.
// id: the workgroup's number among those of the tile.
template <int HR, bool GROUPED, bool WRITE_DS, bool PLAIN, int GRID, bool OWN_DELTA>
__device__ __forceinline__ void dkdv_pairs(
    int id, char* const lds, const a2d_tile_desc& d, const SegList& g, const int parts, const bf16_t* __restrict__ Q,
    const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ O,
    const bf16_t* __restrict__ dO, const float* __restrict__ lse, const float* __restrict__ delta,
    float* __restrict__ dK, float* __restrict__ dV, bf16_t* __restrict__ dS) {
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  int head, blk;
  // `head` is the KEY/VALUE head; its g.group query heads are consecutive rows of Q, dO, lse, delta.
  // With parts > 1 that many workgroups share a key block: workgroup `part` walks its share of the
  // steps over the group's query rows and leaves its sums in partial buffer `part` (dK, dV then point
  // at parts buffers of [key/value heads][nkv][H], added up by a sum kernel afterwards).
  static_assert(!GRID || (GROUPED && !WRITE_DS && !PLAIN), "the grid's form");
  constexpr bool CYCLIC = GRID == 2;
  const int group = GROUPED ? g.group : 1, kv_heads = GROUPED ? d.heads / g.group : d.heads;
  const int nkb = (d.nkv + DK_KEYS - 1) / DK_KEYS;
  int unit;
  if (!xcd_map(id, kv_heads * parts, (GRID ? g.b.side : 1) * nkb, (GRID ? d.causal : g.by_size) != 0, unit, blk)) return;
  const Split up = split_by(unit, parts);
  head = up.q;
  const int part = up.r;
  const int qh0 = GROUPED ? head * g.group : head;           // the first query head, as a head of Q
  const GridBlock gb = GRID ? grid_column(g.b, nkb, blk) : GridBlock{0, blk};
  const int col = gb.r;                                      // of the grid
  blk = gb.blk;
  if (!GRID || parts > 1) {
    const int64_t first = ((int64_t)part * (GRID ? g.b.side : 1) + col) * kv_heads * d.nkv * HR;
    dK += first;
    dV += first;
  }
  const int side = CYCLIC ? __builtin_amdgcn_readfirstlane(g.b.side) : 1;      // row blocks that are walked in turn
  const int nq = GRID == 1 ? g.b.side * d.nq : d.nq, head_rows = nq * side;    // rows of a run; of a query head
  const int col_first = GRID == 1 && d.causal ? col * d.nkv : 0;               // the row that sees the column's first key
  constexpr int HD = padded_head(HR), H = HR, KS = HD / 16, CT = HD / 32;
  constexpr int KSR = (HR + 15) / 16;       // slices of H that hold data
  const int k0 = blk * DK_KEYS;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int pair = wave & 3, role = wave >> 2;   // wavefronts w and w + 4 share 32 keys
  const int l32 = lane & 31;
  Q += (int64_t)qh0 * d.lq.head;
  dO += (int64_t)qh0 * d.ldo.head;
  if (OWN_DELTA) O += (int64_t)qh0 * d.lo.head;
  K += (int64_t)head * d.lk.head + (GRID ? col * g.b.k : 0);
  V += (int64_t)head * d.lv.head + (GRID ? col * g.b.v : 0);
  lse += (int64_t)qh0 * head_rows;
  if (!OWN_DELTA) delta += (int64_t)qh0 * head_rows;

  DkCtx<HD> cx;
  cx.half = lane >> 5;
  cx.c = d.scale * kLog2e;
  // ---- K^T (score wave) or V^T (gradient wave) B fragments of the pair's 32 keys: lane = key,
  // h = 16 x + 8 half + 0..7.  Keys beyond nkv re-read the last key; the mask zeroes their
  // probabilities.
  const int key = k0 + pair * 32 + l32;
  {
    const bf16_t* src = (role ? V : K) + (int64_t)min(key, d.nkv - 1) * (role ? d.lv.row : d.lk.row) + 8 * cx.half;
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      if (16 * x < H) cx.frag[x] = *reinterpret_cast<const bf16x8*>(src + 16 * x);
      else cx.frag[x] = bf16x8{};                              // columns past the head size are zero
    }
  }
#pragma unroll
  for (int t = 0; t < CT; ++t) cx.acc[t] = zero16();

  // Query i sees key kk of key/value sub-block s iff i >= kk - rel[s].  seg_first_row(sb, r): first
  // local query row that sees local key r of sub-block sb (nq if none does).
  auto seg_first_row = [&](int sb, int r) -> int {
    const int64_t f = (int64_t)(r - g.seg[sb].start) - g.seg[sb].rel;
    return f <= 0 ? 0 : (f >= d.nq ? d.nq : (int)f);
  };
  // smallest / largest such row over the local keys a .. b - 1 (inside a sub-block it grows with
  // the key, so only the ends of the covered part of each sub-block matter).  Each sub-block's
  // table entries are read once, with no load depending on another.
  auto first_row_range = [&](int a, int b, int& lo, int& hi) {
    lo = nq; hi = 0;
    if (!d.causal) { lo = 0; return; }
    if (GRID) { lo = col_first + a; hi = col_first + b - 1; return; }
    for (int sb = 0; sb < g.n; ++sb) {
      const int x = max(a, g.seg[sb].start), y = min(b, g.seg[sb].start + g.seg[sb].rows);
      if (x >= y) continue;
      lo = min(lo, seg_first_row(sb, x));
      hi = max(hi, seg_first_row(sb, y - 1));
    }
  };
  int wg_lo, wg_hi;
  first_row_range(k0, min(k0 + DK_KEYS, d.nkv), wg_lo, wg_hi);
  // The walk: nsteps steps of BQ rows per query head, the group's heads one after the other.  A part
  // takes an equal run of it: `total` steps from step s0 of head h0 of the group on.
  // (cyclic grids: step s of every row block before step s + 1 of any)
  int i_start = (wg_lo / BQ) * BQ;
  int nsteps = (nq - i_start + BQ - 1) / BQ;
  int total = nsteps * side * group, s0 = 0, r0 = 0, h0 = 0;
  if (parts > 1) {
    const int all = total, first = (int)((int64_t)part * all / parts);
    total = (int)((int64_t)(part + 1) * all / parts) - first;
    if (!GROUPED) {
      i_start += first * BQ;
      nsteps = total;
    } else if (nsteps > 0) {
      h0 = first / (nsteps * side);
      s0 = first - h0 * (nsteps * side);
      if (CYCLIC) { r0 = s0 % side; s0 /= side; }
    }
    if (total == 0) nsteps = 0;
  }
  const int wk_first = k0 + pair * 32, wk_end = min(wk_first + 32, d.nkv);
  cx.my_first = nq;                                           // padding keys see nothing
  if (key < d.nkv) {
    cx.my_first = GRID && d.causal ? col_first + key : 0;
    if (!GRID && d.causal) {
      for (int sb = 0; sb < g.n; ++sb)                        // uniform loop, per-lane select
        if (key >= g.seg[sb].start && key < g.seg[sb].start + g.seg[sb].rows) cx.my_first = seg_first_row(sb, key);
    }
  }
  int w_any = nq, w_all = nq;       // rows below w_any see none of the pair's keys, rows from w_all on all
  if (wk_first < wk_end) {
    first_row_range(wk_first, wk_end, w_any, w_all);
    if (wk_end < wk_first + 32) w_all = nq;                   // padding keys in the pair: always masked
  }
  // cyclic: the row blocks before the column see a key a row later than the others
  const int late = CYCLIC && d.causal ? col : 0;

  // ---- The gradient waves run ONE STEP BEHIND the score waves: in iteration j the score wave
  // computes S, P, dV of step j and leaves P in mailbox slot j & 1, while the gradient wave of
  // the same SIMD computes dP, dS, dK of step j - 1 from slot (j - 1) & 1.  Inside an iteration
  // the two never wait for each other; the single barrier per iteration publishes the mailbox
  // and a tile.  Step s lives in tile buffer s % 4: during iteration j buffers (j - 1) % 4 and
  // j % 4 are being computed on, (j + 1) % 4 is complete already - so that every wave can
  // request the first fragments of its NEXT step before the barrier and start the following
  // iteration with its operands in registers - and (j + 2) % 4 is being filled.  The score wave
  // starts on buffer 0 / slot 0, the gradient wave one behind.
  {
    DualAddr a;
    a.init(lane, lds_base + (role ? (DK_NBUF - 1) * DK_BUF : 0));
    const unsigned nat_tile = role ? DK_TILE : 0, tr_tile = role ? 0 : DK_TILE;
    cx.nat_e = a.nat_e + nat_tile; cx.nat_o = a.nat_o + nat_tile;
    cx.tr_lo = a.tr_lo + tr_tile;  cx.tr_hi = a.tr_hi + tr_tile;
  }
  cx.stat = lds_base + DK_STAT + (role ? (DK_NBUF - 1) * DK_STAT_BUF + BQ * 4 : 0) + 16 * cx.half;
  cx.mbox = lds_base + DK_MBOX + (role ? DK_MBOX_SLOT : 0) + pair * DK_MBOX_PIECE + lane * 16;
  int cur = role ? DK_NBUF - 1 : 0;   // tile buffer of this wave's step

  // ---- staging of a 32-row step: thread moves chunk (tid & 15) of row (tid >> 4) of both tiles.
  // Global latency is longer than an iteration: step j + 4 is requested in iteration j and
  // written to LDS in iteration j + 2, through two register sets.  Rows beyond nq re-read the
  // last row; their lse entry is +inf, which makes exp2(s - lse) = 0 (also for rows whose lse is
  // -inf).  Steps beyond the last re-stage the last one (into a buffer nobody reads any more):
  // unconditional loads and stores keep the compiler's wait counters exact.
  static_assert(DK_THREADS == BQ * 16, "staging map: one 16-byte chunk of each tile per thread");
  const int st_row = tid >> 4, st_ch = tid & 15;
  const gptr_t q_base = uniform_gptr(Q), g_base = uniform_gptr(dO);
  const int st_off = dual_store_off(st_row, st_ch);
  u32x4 qreg[2], greg[2], oreg[2];
  float stat[2] = {0.f, 0.f};
  bool stat_ok[2] = {false, false}, row_ok[2] = {false, false};
  // (a chunk past the row's end - head sizes below 128 - re-reads the row's last chunk and is
  // stored as zeros or, past the padded head size, not at all: every lane issues every load)
  const int ld_ch = min(st_ch, H / 8 - 1);
  const bool ch_data = st_ch * 8 < H, ch_tile = st_ch * 8 < HD;
  // (load_step is called for steps 0, 1, 2, ... in order; with grouped heads ld_s / ld_row0 /
  // ld_left follow the next step's position - its step inside the query head, the head's first
  // row - without a division)
  // (ld_qh / ld_gh: byte offset of the query head's first row of Q / dO from the group's first head)
  int ld_s = s0, ld_r = r0, ld_row0 = h0 * head_rows, ld_left = total - 1;
  const unsigned q_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.row * 2);
  const unsigned g_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.ldo.row * 2);
  const unsigned q_head_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.head * 2);
  const unsigned g_head_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.ldo.head * 2);
  const unsigned q_blk_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.q * 2)) : 0;
  const unsigned g_blk_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.g * 2)) : 0;
  unsigned ld_qh = h0 * q_head_bytes, ld_gh = h0 * g_head_bytes;
  const gptr_t o_base = uniform_gptr(OWN_DELTA ? O : dO);
  const unsigned o_row_bytes = OWN_DELTA ? __builtin_amdgcn_readfirstlane((unsigned)d.lo.row * 2) : 0;
  const unsigned o_head_bytes = OWN_DELTA ? __builtin_amdgcn_readfirstlane((unsigned)d.lo.head * 2) : 0;
  const unsigned o_blk_bytes = OWN_DELTA && CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.o * 2)) : 0;
  unsigned ld_oh = h0 * o_head_bytes;
  auto load_step = [&](int step, auto set_tag) {
    constexpr int SET = decltype(set_tag)::value;
    const int i0 = i_start + (GROUPED ? ld_s : min(step, nsteps - 1)) * BQ;
    if constexpr (PLAIN) {
      const unsigned off = (unsigned)((ld_row0 + min(i0 + st_row, d.nq - 1)) * (H * 2) + ld_ch * 16);
      qreg[SET] = gload_b128(q_base, off);
      greg[SET] = gload_b128(g_base, off);
    } else {
      const unsigned r = (unsigned)min(i0 + st_row, nq - 1);
      qreg[SET] = gload_b128(q_base, ld_qh + (CYCLIC ? ld_r * q_blk_bytes : 0u) + __umul24(r, q_row_bytes) + ld_ch * 16);
      greg[SET] = gload_b128(g_base, ld_gh + (CYCLIC ? ld_r * g_blk_bytes : 0u) + __umul24(r, g_row_bytes) + ld_ch * 16);
      if constexpr (OWN_DELTA) {
        oreg[SET] = gload_b128(o_base, ld_oh + (CYCLIC ? ld_r * o_blk_bytes : 0u) + __umul24(r, o_row_bytes) + ld_ch * 16);
        row_ok[SET] = i0 + st_row < nq;
      }
    }
    // raw statistic loads only: converting here would make the wave wait for everything just
    // issued.  Every thread loads one (only the first 64 values are used) so that each set is
    // the same number of loads in every wavefront.
    const int ir = min(i0 + (tid & (BQ - 1)), nq - 1);
    const int i = ld_row0 + (CYCLIC ? ir * side + ld_r : ir);
    stat[SET] = !OWN_DELTA && (tid & BQ) ? delta[i] : lse[i];
    stat_ok[SET] = (i0 + (tid & (BQ - 1))) < nq;
    if constexpr (GROUPED) {   // next step; the last one repeats
      bool more = ld_left > 0;
      ld_left -= more ? 1 : 0;
      if constexpr (CYCLIC) {
        const bool last = ld_r + 1 == side;
        ld_r = more ? (last ? 0 : ld_r + 1) : ld_r;
        more = more && last;
      }
      const bool wrap = ld_s + 1 == nsteps;
      ld_row0 += (more && wrap) ? head_rows : 0;
      ld_qh += (more && wrap) ? q_head_bytes : 0u;
      ld_gh += (more && wrap) ? g_head_bytes : 0u;
      if (OWN_DELTA) ld_oh += (more && wrap) ? o_head_bytes : 0u;
      ld_s = more ? (wrap ? 0 : ld_s + 1) : ld_s;
    }
  };
  auto store_step = [&](int buf, auto set_tag) {
    constexpr int SET = decltype(set_tag)::value;
    char* b = lds + buf * DK_BUF;
    if (HD == 128 || ch_tile) {
      const u32x4 zero = {0, 0, 0, 0};
      *reinterpret_cast<u32x4*>(b + st_off) = (HD == 128 || ch_data) ? qreg[SET] : zero;
      *reinterpret_cast<u32x4*>(b + DK_TILE + st_off) = (HD == 128 || ch_data) ? greg[SET] : zero;
    }
    if constexpr (OWN_DELTA) {
      // this thread's 16-byte chunk of the row, then the chunks 1, 2, 4, 8 apart (16 lanes hold a row; every lane of
      // a quad, then of half a row has its sum, so that mirroring stands for the exchange 4 and 8 apart)
      float t = dot8(oreg[SET], greg[SET], 0.f);
      if (HD != HR || HR != 128) t = ch_data ? t : 0.f;
      t += lane_swap<0xB1>(t);                                 // quad_perm 1, 0, 3, 2
      t += lane_swap<0x4E>(t);                                 // quad_perm 2, 3, 0, 1
      t += lane_swap<0x141>(t);                                // mirrored in 8 lanes
      t += lane_swap<0x140>(t);                                // mirrored in 16 lanes
      if (st_ch == 0) reinterpret_cast<float*>(lds + DK_STAT + buf * DK_STAT_BUF)[BQ + st_row] = row_ok[SET] ? -t : 0.f;
    }
    if (tid < (OWN_DELTA ? BQ : 2 * BQ)) {
      float v = stat[SET];
      if (tid < BQ) v = (!stat_ok[SET] || v == -INFINITY) ? INFINITY : v * kLog2e;
      else v = stat_ok[SET] ? -v : 0.f;                        // -delta: where the sum of dP starts
      reinterpret_cast<float*>(lds + DK_STAT + buf * DK_STAT_BUF)[tid] = v;
    }
  };
  using set0 = std::integral_constant<int, 0>;
  using set1 = std::integral_constant<int, 1>;

  if (nsteps > 0) {
    load_step(0, set0{}); load_step(1, set1{});
    wait_vmem_all();                                 // (the K / V rows and the first steps together)
    store_step(0, set0{}); store_step(1, set1{});
    load_step(2, set0{}); load_step(3, set1{});
  }
  __syncthreads();

  // dS hand-over: this pair's 32 keys are piece T = pair & 1 of key block 2 blk + (pair >> 1)
  const unsigned ds_row_stride = (unsigned)ds_key_blocks(d.nkv) * DS_TILE_BYTES;
  const unsigned ds_lane_off = (unsigned)(2 * blk + (pair >> 1)) * DS_TILE_BYTES + (pair & 1) * 2048 +
                               (l32 >> 4) * 1024 + ((lane >> 5) * 16 + (l32 & 15)) * 16;
  gwptr_t ds_base = nullptr;
  if constexpr (WRITE_DS)
    ds_base = uniform_gwptr(reinterpret_cast<char*>(dS) + qh0 * ds_head_bytes(d.nq, d.nkv));

  // A step is skipped (by both wavefronts of its pair) when none of its rows sees any of the
  // pair's keys; it is masked unless every row sees every key.
  // (step = position in the whole walk, s = its step inside its run of rows, r its row block)
  // (rows past nq do not count: a pair without keys, w_any = nq, is never active - it has no
  // place in the dS workspace either)
  auto shift = [&](int r) { return CYCLIC && r < late ? 1 : 0; };
  auto active = [&](int step, int s, int r) {
    return step >= 0 && step < total && min(i_start + s * BQ + BQ - 1, nq - 1) - shift(r) >= w_any;
  };
  int cs = s0, cr = r0;                                         // s, r of the iteration's step j
  auto next_step = [&](int& s, int& r) {
    if (CYCLIC) {
      const bool last = r + 1 == side;
      r = last ? 0 : r + 1;
      if (!last) return;
    }
    s = (GROUPED && s + 1 == nsteps) ? 0 : s + 1;
  };
  // dS row tile of step j, counted over the group's heads
  int c_rt = (GROUPED ? h0 * ds_row_tiles(d.nq) + s0 : 0) + i_start / BQ;
  // (a head's steps end at its last row tile; the next head's start i_start / BQ tiles into its own)
  auto next_rt = [&](int rt, int s) { return (GROUPED && s + 1 == nsteps) ? rt + 1 + i_start / BQ : rt + 1; };
  auto advance = [&](int slot_delta) {   // to this wave's next step: tile buffer and mailbox slot
    const int adv = (cur == DK_NBUF - 1) ? -(DK_NBUF - 1) : 1;
    cur += adv;
    cx.nat_e += adv * DK_BUF; cx.nat_o += adv * DK_BUF; cx.tr_lo += adv * DK_BUF; cx.tr_hi += adv * DK_BUF;
    cx.stat += adv * DK_STAT_BUF;
    cx.mbox += slot_delta;
  };

  // The two roles go through an iteration in opposite phase, so that on every SIMD one wave's
  // element-wise work coincides with the other's MFMAs:
  //   score wave     S (8 MFMAs)          | exponentials          | dV (8 MFMAs)
  //   gradient wave  dS of step j - 1     | dK of step j - 1      | dP of step j (8 MFMAs each)
  // In iteration j, SET is the register set that holds step j + 2 and then receives step j + 4.
  if (nsteps > 0 && role == 0) {
    // first natural fragments and lse values of the coming step, requested an iteration ahead
    bf16x8 n[4];
    f32x4 st[4];
    dk_first_pre(cx, n);
    dk_stat_pre(cx, st);
    auto iteration = [&](int j, auto set_tag) {
      constexpr int SET = decltype(set_tag)::value;
      store_step((j + 2) % DK_NBUF, set_tag);
      load_step(j + 4, set_tag);
      if (active(j, cs, cr)) {
        // (first row, rows of the run: both one less where the keys are seen a row later)
        const int i0 = i_start + cs * BQ - shift(cr), rows = nq - shift(cr);
        bf16x8 t[CT], bf[2];
        f32x16 s = dk_first<HD, KSR>(cx, n, zero16());
        dk_second_pre(cx, t);
        if (i0 >= w_all && i0 + BQ <= rows) dk_probs<false>(cx, st, s, bf, i0, rows);
        else dk_probs<true>(cx, st, s, bf, i0, rows);
        dk_second(cx, t, bf);
      }
      advance(SET ? -DK_MBOX_SLOT : DK_MBOX_SLOT);
      next_step(cs, cr);
      dk_first_pre(cx, n);
      dk_stat_pre(cx, st);
      __syncthreads();
    };
    // nsteps + 1 iterations (the gradient wave's last step), rounded up to an even number: an
    // iteration beyond that finds no step to compute, and straight-line control flow keeps the
    // wait counters exact
    for (int j = 0; j <= total; j += 2) {
      iteration(j, set0{});
      iteration(j + 1, set1{});
    }
  } else if (nsteps > 0) {
    f32x16 dp = zero16();   // dP - delta of the step whose dS, dK come next iteration
    int ps = 0, pr = 0;     // s, r of step j - 1
    int p_rt = 0;           // and its dS row tile
    auto iteration = [&](int j, auto set_tag) {
      constexpr int SET = decltype(set_tag)::value;
      store_step((j + 2) % DK_NBUF, set_tag);
      load_step(j + 4, set_tag);
      if (active(j - 1, ps, pr)) {
        bf16x8 t[CT], bf[2];
        f32x4 pm[4];
        dk_mbox_pre(cx, pm);
        dk_second_pre(cx, t);
        dk_dscores(pm, dp, bf);
        dk_second(cx, t, bf);
        if constexpr (WRITE_DS) {
          // (measured: making these stores unconditional - skipped steps writing to a spill slot,
          // which keeps the compiler's load wait counts exact - is not faster)
          const unsigned off = (unsigned)p_rt * ds_row_stride + ds_lane_off;
          // (register group q: rows 8 q + 4 half + 0..3, i.e. of groups g = half and 2 + half)
          gstore_b128(ds_base, off, __builtin_shufflevector(bf[0], bf[1], 0, 1, 2, 3, 8, 9, 10, 11));
          gstore_b128(ds_base, off + 512, __builtin_shufflevector(bf[0], bf[1], 4, 5, 6, 7, 12, 13, 14, 15));
        }
      }
      advance(SET ? DK_MBOX_SLOT : -DK_MBOX_SLOT);
      p_rt = c_rt;
      c_rt = next_rt(c_rt, cs);
      ps = cs;
      pr = cr;
      next_step(cs, cr);
      if (active(j, ps, pr)) {
        bf16x8 n[4];
        f32x4 st[4];
        dk_first_pre(cx, n);
        dk_stat_pre(cx, st);
        f32x16 init;
#pragma unroll
        for (int r = 0; r < 16; ++r) init[r] = st[r >> 2][r & 3];
        dp = dk_first<HD, KSR>(cx, n, init);
      }
      __syncthreads();
    };
    for (int j = 0; j <= total; j += 2) {
      iteration(j, set0{});
      iteration(j + 1, set1{});
    }
  }

  if (GRID && parts == 1) {
    if (key < d.nkv) {
      const int x = role ? 1 : 2;                                // dK, dV
      bf16_t* const out = reinterpret_cast<bf16_t*>(role ? dK : dV) + head * g.b.out[x].head + col * g.b.out_step[x] +
                          key * g.b.out[x].row;
      store_acc_t<CT>(out, cx.acc, cx.half, role ? d.scale : 1.0f, H);
    }
  } else if (key < d.nkv) {
    const int64_t row = (int64_t)head * d.nkv + key;
    if (role == 0) store_acc_t<CT>(dV + row * H, cx.acc, cx.half, 1.0f, H);
    else store_acc_t<CT>(dK + row * H, cx.acc, cx.half, d.scale, H);
  }
}

}  // namespace mfma
}  // namespace a2d
