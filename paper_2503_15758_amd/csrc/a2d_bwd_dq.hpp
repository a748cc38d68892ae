// The workgroup that recomputes the scores for dQ (see a2d_bwd_mfma.hip for the kernels).
#pragma once
#include <type_traits>

#include "a2d_bwd.hpp"

namespace a2d {
namespace mfma {

constexpr int BKS = 64;           // keys per step
// LDS: [buf]{ K tile (dual layout), V tile (natural reads only: rows of the head's bytes + 16) }
__host__ __device__ constexpr int vt_ld(int hd) { return hd * 2 + 16; }
constexpr int DQ_VT = DUAL64_BYTES;
__host__ __device__ constexpr int dq_buf(int hd) { return DUAL64_BYTES + BKS * vt_ld(hd); }
__host__ __device__ constexpr int dq_lds(int hd) { return 2 * dq_buf(hd); }
// fragment ring depth (registers are tight above H = 64: 256 per wavefront)
__host__ __device__ constexpr int dq_ring(int hd) { return hd == 64 ? 4 : 2; }

template <int HD>
struct DqCtx {
  f32x16 dq[HD / 32];
  bf16x8 qf[HD / 16], gf[HD / 16];
  DualAddr ka;          // K tile of the current buffer
  unsigned vnat;        // natural-fragment base in the V tile of the current buffer
  float c, lse2, del;
  int my_vis;           // number of leading local keys this lane's query row sees
  int half;
};

// one 32-key x 32-query piece: T selects the half of the 64-key step.  HD / 16 slices of H in the
// two first contractions (S^T and dP^T, alternating), 2 * HD / 32 MFMAs in dQ^T += K^T dS^T
// (step I: 16-key group I / CT, column tile I % CT); fragments run two steps ahead of their use.
// (KS: the slices that hold data - a head size of 80 fills five of the padded six)
template <int T, bool MASK, int HD, int KS = HD / 16>
__device__ __forceinline__ void dq_piece(DqCtx<HD>& cx, int key0) {
  constexpr int CT = HD / 32, VT_LD = vt_ld(HD), DQ_RING = dq_ring(HD);
  constexpr int RB = T * 32 * DUAL_LD;
  constexpr int VB = T * 32 * VT_LD;
  bf16x8 kr[DQ_RING], vr[DQ_RING], kt[DQ_RING];
  auto ld1 = [&](auto X) {
    constexpr int x = decltype(X)::value;
    kr[x % DQ_RING] = dual_nat<x>(cx.ka, RB);
    vr[x % DQ_RING] = lds_load_b128(cx.vnat + VB + 32 * x);
    __builtin_amdgcn_sched_barrier(0);
  };
  // K^T fragments; the first ones are on their way during the exponentials
  auto ld2 = [&](auto I) {
    constexpr int i = decltype(I)::value;
    kt[i % DQ_RING] = lds_load_tr(cx.ka.tr_lo + RB + (i / CT) * 16 * DUAL_LD + 64 * (i % CT),
                                  cx.ka.tr_hi + RB + (i / CT) * 16 * DUAL_LD + 64 * (i % CT));
    __builtin_amdgcn_sched_barrier(0);
  };
  static_for<0, DQ_RING>(ld1);
  f32x16 s = zero16(), dp = zero16();
  static_for<0, KS>([&](auto X) {
    constexpr int x = decltype(X)::value;
    s = mma(kr[x % DQ_RING], cx.qf[x], s);
    dp = mma(vr[x % DQ_RING], cx.gf[x], dp);
    if constexpr (x + DQ_RING < KS) ld1(std::integral_constant<int, x + DQ_RING>{});
    else ld2(std::integral_constant<int, x + DQ_RING - KS>{});
  });
  // register r <-> key key0 + 8*(r>>2) + 4*half + (r&3); lane <-> query
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float p = fast_exp2(fmaf(s[r], cx.c, -cx.lse2));
    if (MASK && (key0 + 8 * (r >> 2) + 4 * cx.half + (r & 3) >= cx.my_vis)) p = 0.f;
    dp[r] = p * (dp[r] - cx.del);
  }
  bf16x8 dsb[2];
  dsb[0] = pack8(dp, 0);
  dsb[1] = pack8(dp, 8);
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, 2 * CT>([&](auto I) {
    constexpr int i = decltype(I)::value;
    cx.dq[i % CT] = mma(kt[i % DQ_RING], dsb[i / CT], cx.dq[i % CT]);
    if constexpr (i + DQ_RING < 2 * CT) ld2(std::integral_constant<int, i + DQ_RING>{});
  });
}

// WAVES wavefronts (32 query rows each) per workgroup: 8 fill a compute unit with one workgroup;
// 4 (two workgroups per compute unit) are used when there are too few 256-row blocks to give
// every compute unit one.
// KL key lanes of WAVES / KL wavefronts: with KL = 2 a 128-row workgroup of eight wavefronts walks
// the key blocks in two lanes (alternate blocks, own tile buffers) whose dQ sums are added through
// LDS at the end - for tiles with at most one 128-row block per compute unit, so that a SIMD still
// holds two wavefronts.
// HR: head size (64, 80, 96 or 128), HD its padded size, as in the dK/dV kernel.
// GRID: all query blocks of an emulated grid, walked as in fwd_mfma_kernel; dQ goes to rows of the sequence's
// (of a split walk: a partial, [part][row block][head][row]).
// id: the workgroup's number among those of the tile.
template <int WAVES, int HR, int KL, int GRID>
__device__ __forceinline__ void dq_rows(
    int id, char* const lds_all, const a2d_tile_desc& d, const SegList& g, const int parts, const bf16_t* __restrict__ Q,
    const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ O,
    const bf16_t* __restrict__ dO, const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dQ) {
  constexpr int RW = WAVES / KL;           // wavefronts of one key lane
  constexpr int DQ_ROWS = 32 * RW;         // query rows per workgroup
  constexpr int DQ_THREADS = 64 * RW;      // threads of one key lane (they stage its tiles)
  constexpr int HD = padded_head(HR), H = HR;
  constexpr int KS = HD / 16, CT = HD / 32, VT_LD = vt_ld(HD), DQ_BUF = dq_buf(HD);
  constexpr int KSR = (HR + 15) / 16;      // slices of H that hold data
  const int kl = KL == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / DQ_THREADS);
  char* const lds = lds_all + kl * (2 * DQ_BUF);
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int nqb = (d.nq + DQ_ROWS - 1) / DQ_ROWS;
  // (the query blocks of the query heads that share a key/value head are placed as one unit)
  int unit, blk;
  const int by_size = GRID ? d.causal : g.by_size;
  if (!xcd_map(id, d.heads / g.group * parts, (GRID ? g.b.side : 1) * g.group * nqb, by_size != 0, unit, blk,
               kXcdCus * 8 / WAVES)) return;
  // (unit = part `part` of the walks over one key/value head; blocks numbered by size first when the
  // workgroups are ordered by size)
  const Split up = split_by(unit, parts);
  const int kvh = up.q, part = up.r;
  const Split in_group = query_head(blk, g.group, nqb, GRID || by_size);
  const int head = kvh * g.group + in_group.r;
  blk = in_group.q;
  const GridBlock gb = GRID ? grid_block(g.b, nqb, blk) : GridBlock{0, blk};
  const int row_blk = gb.r;                            // of the grid
  blk = gb.blk;
  const int q0 = (nqb - 1 - blk) * DQ_ROWS;            // heavy blocks first under a causal mask
  const int tid = (int)threadIdx.x - kl * DQ_THREADS;  // within the key lane
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l32 = lane & 31;
  Q += (int64_t)head * d.lq.head + (GRID ? row_blk * g.b.q : 0);
  O += (int64_t)head * d.lo.head + (GRID ? row_blk * g.b.o : 0);
  dO += (int64_t)head * d.ldo.head + (GRID ? row_blk * g.b.g : 0);
  K += (int64_t)kvh * d.lk.head;
  V += (int64_t)kvh * d.lv.head;

  DqCtx<HD> cx;
  cx.half = lane >> 5;
  cx.c = d.scale * kLog2e;
  const int q_row = q0 + wave * 32 + l32;
  const bool q_ok = q_row < d.nq;
  const int q_ld = min(q_row, d.nq - 1);         // rows beyond nq re-read the last row, lse2 = +inf
  {
    const int64_t off = (int64_t)q_ld * d.lq.row + 8 * cx.half, goff = (int64_t)q_ld * d.ldo.row + 8 * cx.half;
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      if (16 * x < H) {
        cx.qf[x] = *reinterpret_cast<const bf16x8*>(Q + off + 16 * x);
        cx.gf[x] = *reinterpret_cast<const bf16x8*>(dO + goff + 16 * x);
      } else {                                                 // columns past the head size are zero
        cx.qf[x] = bf16x8{};
        cx.gf[x] = bf16x8{};
      }
    }
  }
  // (lse and delta: of the tile, or of the whole sequence)
  const int64_t stat_at = GRID ? (int64_t)head * g.b.side * d.nq + grid_token(g.b, d.nq, row_blk, q_ld)
                               : (int64_t)head * d.nq + q_ld;
  const float lse_i = lse[stat_at];
  // delta = rowsum(dO o O) of the wavefront's rows, left for the dK/dV kernel where that runs after this one
  bf16x8 of[KS];
#pragma unroll
  for (int x = 0; x < KS; ++x) {
    if (16 * x < H) of[x] = *reinterpret_cast<const bf16x8*>(O + (int64_t)q_ld * d.lo.row + 8 * cx.half + 16 * x);
    else of[x] = bf16x8{};
  }

  // visibility per key/value sub-block s: query i sees the first vis_count(i, s) keys of it
  auto vis_count = [&](int i, int s) -> int {
    if (GRID == 1) return d.causal ? row_blk * d.nq + i + 1 : g.b.side * d.nkv;
    if (GRID == 2) return d.causal ? i + 1 : d.nkv;    // (of columns up to the row block's own, see shift_from)
    if (!d.causal) return g.seg[s].rows;
    const int64_t v = (int64_t)i + g.seg[s].rel + 1;
    return v <= 0 ? 0 : (v < g.seg[s].rows ? (int)v : g.seg[s].rows);
  };
  const int blk_last = min(q0 + DQ_ROWS, d.nq) - 1;
  const int w_first = min(q0 + wave * 32, d.nq - 1);
  const int w_last = min(q0 + wave * 32 + 31, d.nq - 1);
  // key blocks of sub-block s that some row of the workgroup sees; the walk over (sub-block, block)
  auto seg_blocks = [&](int s) { return (vis_count(blk_last, s) + BKS - 1) / BKS; };
  int nvis_wave = 0, nfull_wave = 0;               // of the current sub-block
  auto enter_segment = [&](int s) {
    nvis_wave = vis_count(w_last, s);
    nfull_wave = vis_count(w_first, s);
    cx.my_vis = vis_count(q_ld, s);
  };
#pragma unroll
  for (int t = 0; t < CT; ++t) cx.dq[t] = zero16();

  cx.ka.init(lane, lds_base);
  cx.vnat = lds_base + DQ_VT + l32 * VT_LD + 16 * cx.half;

  // ---- staging, in two halves of 32 key rows: thread moves chunk (tid & 15) of rows
  // (tid >> 4) + ST_ROWS p of a half.  Rows beyond nkv re-read the last row (finite values,
  // masked out).
  constexpr int ST_ROWS = DQ_THREADS / 16, ST_N = 32 / ST_ROWS;
  const int st_row = tid >> 4, st_ch = tid & 15;
  u32x4 kreg[ST_N], vreg[ST_N];
  // half hf of block j of the sub-block of seg_rows keys that starts at local key seg_start
  // (a chunk past the row's end - head sizes below 128 - re-reads the row's last chunk and is
  // stored as zeros or, past the padded head size, not at all)
  const int ld_ch = min(st_ch, H / 8 - 1);
  const bool ch_data = st_ch * 8 < H, ch_tile = st_ch * 8 < HD;
  // (row strides in bytes, pinned in registers: read from the kernel arguments inside the loop they
  // would be scalar loads, which share a wait counter with the LDS reads in flight.  A head's rows
  // span less than 4 GiB - the API layer checks it - so row index times stride fits 32 bits.)
  const unsigned k_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lk.row * 2);
  const unsigned v_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lv.row * 2);
  // (cyclic grids: seg_start is the number of the grid's column, whose first row that is in the sequence)
  const unsigned k_col_bytes = GRID == 2 ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.k * 2)) : k_row_bytes;
  const unsigned v_col_bytes = GRID == 2 ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.v * 2)) : v_row_bytes;
  auto load_half = [&](int seg_start, int seg_rows, int j, int hf) {
    const gptr_t kb = uniform_gptr(reinterpret_cast<const char*>(K) + (seg_start * k_col_bytes + (unsigned)(j * BKS) * k_row_bytes));
    const gptr_t vb = uniform_gptr(reinterpret_cast<const char*>(V) + (seg_start * v_col_bytes + (unsigned)(j * BKS) * v_row_bytes));
    const int last = seg_rows - 1 - j * BKS;       // rows beyond the sub-block re-read its last row
#pragma unroll
    for (int p = 0; p < ST_N; ++p) {
      const unsigned r = (unsigned)min(32 * hf + st_row + ST_ROWS * p, last);
      kreg[p] = gload_b128(kb, __umul24(r, k_row_bytes) + ld_ch * 16);
      vreg[p] = gload_b128(vb, __umul24(r, v_row_bytes) + ld_ch * 16);
    }
  };
  auto store_half = [&](int buf, int hf) {
    char* b = lds + buf * DQ_BUF;
    if (HD == 128 || ch_tile) {
      const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
      for (int p = 0; p < ST_N; ++p) {
        const int row = 32 * hf + st_row + ST_ROWS * p;
        *reinterpret_cast<u32x4*>(b + dual_store_off(row, st_ch)) = (HD == 128 || ch_data) ? kreg[p] : zero;
        *reinterpret_cast<u32x4*>(b + DQ_VT + row * VT_LD + st_ch * 16) = (HD == 128 || ch_data) ? vreg[p] : zero;
      }
    }
  };

  // Walk over the entries (sub-block, key block): lane part * KL + kl of parts * KL takes every
  // (parts * KL)-th entry.  The sub-block table lives in kernel-argument memory, and scalar loads
  // share a wait counter with the LDS reads in flight, so it is only touched when a walk moves to
  // another sub-block; in between its values sit in registers.  An entry is (sub-block sb, block j
  // of its nblk); sb == g.n: past the end.
  // (cyclic grids: block j of all columns before block j + 1 of any)
  constexpr bool PLAIN = GRID == 0, CYCLIC = GRID == 2;
  const int stride = KL * parts, segs = PLAIN ? g.n : CYCLIC ? __builtin_amdgcn_readfirstlane(g.b.side) : 1;
  const int grid_rows = GRID == 1 ? g.b.side * d.nkv : d.nkv;
  auto seg_start = [&](int s) { return PLAIN ? g.seg[s].start : s; };
  auto seg_rows = [&](int s) { return PLAIN ? g.seg[s].rows : grid_rows; };
  const int jump = CYCLIC ? stride / segs : 0, jump_rest = stride - jump * segs;
  auto open_segment = [&](int s, int& sb, int& nblk) {           // first sub-block from s on with visible keys
    while (s < segs && seg_blocks(s) == 0) ++s;
    sb = s;
    if (s < segs) nblk = seg_blocks(s);
  };
  auto advance = [&](int by, int& sb, int& j, int& nblk) {
    if constexpr (CYCLIC) {
      if (sb >= segs) return;
      const int q = by == stride ? jump : by / segs;
      j += q;
      sb += by == stride ? jump_rest : by - q * segs;
      if (sb >= segs) { sb -= segs; ++j; }
      if (j >= nblk) sb = segs;
    } else {
      j += by;
      while (sb < segs && j >= nblk) { j -= nblk; open_segment(sb + 1, sb, nblk); }
    }
  };
  // cyclic: query i sees the keys kk <= i of columns up to its row block's own, kk < i of the others - the mask of the
  // former with the keys numbered one higher
  const int shift_from = CYCLIC && d.causal ? row_blk : segs;
  int sb, j = 0, nblk = 0;                         // this key lane's current entry
  open_segment(0, sb, nblk);
  advance(part * KL, sb, j, nblk);
  int lead_sb = sb, lead_j = j, lead_nblk = nblk;  // key lane 0's: every lane of the workgroup loops while it exists
  if (KL > 1) advance(kl, sb, j, nblk);
  int nx_start = 0, nx_rows = 0;                   // start / rows of the next entry's sub-block
  if (sb < segs) {
    enter_segment(sb);
    nx_start = seg_start(sb); nx_rows = seg_rows(sb);
    load_half(nx_start, nx_rows, j, 0);
  }
  wait_vmem_all();                                 // (the rows of Q, dO, O and the first half together)
  cx.lse2 = (!q_ok || lse_i == -INFINITY) ? INFINITY : lse_i * kLog2e;      // +inf: exp2(s - lse2) = 0
  {
    // (the order of sums of delta_kernel, so that both dQ paths give the same dK, dV: 16-byte chunks,
    // then chunks 1, 2, 4, 8 apart; this lane holds the chunks 2 x + half)
    float t[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      t[x] = 0.f;
      if (x >= KS) continue;
      t[x] = dot8(__builtin_bit_cast(u32x4, of[x]), __builtin_bit_cast(u32x4, cx.gf[x]), 0.f);
      t[x] += __shfl_xor(t[x], 32, 64);
    }
    cx.del = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
  }
  if (delta && part == 0 && kl == 0 && cx.half == 0 && q_ok) delta[stat_at] = cx.del;
  if (sb < segs) {
    store_half(0, 0);
    load_half(nx_start, nx_rows, j, 1); store_half(0, 1);
  }
  __syncthreads();

  int buf = 0;
  while ((KL == 1 ? sb : lead_sb) < segs) {
    int nsb = sb, nj = j, nnblk = nblk;
    advance(stride, nsb, nj, nnblk);
    const bool more = nsb < segs;
    if (CYCLIC) nx_start = nsb;
    else if (A2D_SELDOM(more && nsb != sb)) { nx_start = seg_start(nsb); nx_rows = seg_rows(nsb); }
    const bool here = KL == 1 || sb < segs;         // this lane has a block in this round
    const int k0 = j * BKS + (CYCLIC && sb > shift_from);      // local to the sub-block
    if (A2D_OFTEN(more)) load_half(nx_start, nx_rows, nj, 0);
    if (here && k0 < nvis_wave) {
      if (k0 + 32 > nfull_wave) dq_piece<0, true, HD, KSR>(cx, k0); else dq_piece<0, false, HD, KSR>(cx, k0);
    }
    if (A2D_OFTEN(more)) { store_half(buf ^ 1, 0); load_half(nx_start, nx_rows, nj, 1); }
    if (here && k0 + 32 < nvis_wave) {
      if (k0 + 64 > nfull_wave) dq_piece<1, true, HD, KSR>(cx, k0 + 32); else dq_piece<1, false, HD, KSR>(cx, k0 + 32);
    }
    if (A2D_OFTEN(more)) store_half(buf ^ 1, 1);
    const int tog = buf ? -DQ_BUF : DQ_BUF;
    cx.ka.shift(tog);
    cx.vnat += tog;
    __syncthreads();
    if (!CYCLIC && A2D_SELDOM(more && nsb != sb)) enter_segment(nsb);
    if (KL > 1) advance(stride, lead_sb, lead_j, lead_nblk);
    sb = nsb; j = nj; nblk = nnblk;
    buf ^= 1;
  }
  if constexpr (KL == 2) {
    // lane 1 hands its sums to lane 0 through LDS (the tiles are no longer read: every wavefront
    // has passed the walk's last barrier); layout [row wavefront][value][lane]: conflict free
    static_assert(RW * CT * 16 * 256 <= KL * 2 * DQ_BUF, "the exchange area must fit the tile buffers");
    float* xch = reinterpret_cast<float*>(lds_all) + wave * (CT * 16 * 64) + lane;
    if (kl == 1) {
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) xch[(16 * t + r) * 64] = cx.dq[t][r];
    }
    __syncthreads();
    if (kl == 1) return;
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) cx.dq[t][r] += xch[(16 * t + r) * 64];
  }
  if (GRID && parts == 1) {
    bf16_t* const out = reinterpret_cast<bf16_t*>(dQ) + head * g.b.out[0].head + row_blk * g.b.out_step[0];
    if (q_ok) store_acc_t<CT>(out + q_row * g.b.out[0].row, cx.dq, cx.half, d.scale, H);
  } else if (q_ok) {
    const int64_t slot = (int64_t)part * (GRID ? g.b.side : 1) + row_blk;
    store_acc_t<CT>(dQ + ((slot * d.heads + head) * d.nq + q_row) * H, cx.dq, cx.half, d.scale, H, !GRID && g.acc != 0);
  }
}

}  // namespace mfma
}  // namespace a2d
