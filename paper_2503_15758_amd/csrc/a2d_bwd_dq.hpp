// The workgroup that recomputes the scores for dQ (see a2d_bwd_mfma.hip for the kernels).
#pragma once
#include <type_traits>

#include "a2d_bwd.hpp"

namespace a2d {
namespace mfma {

constexpr int BKS = 64;           // keys per step
// LDS: [buf]{ K tile, V tile }, in blocks
__host__ __device__ constexpr int dq_buf(int hd) { return 2 * BKS * 2 * hd; }
// of a key lane (eight wavefronts also store 16 rows each at a time)
__host__ __device__ constexpr int dq_lds(int hd) { return 2 * dq_buf(hd); }
__host__ __device__ constexpr int dq_launch_lds(int hd, int kl) {
  return kl * dq_lds(hd) > 8 * acc_area(hd / 16) ? kl * dq_lds(hd) : 8 * acc_area(hd / 16);
}
// fragment ring depth (registers are tight above H = 64: 256 per wavefront)
__host__ __device__ constexpr int dq_ring(int hd) { return hd == 64 ? 4 : 2; }

template <int HR>
struct DqCtx {
  static constexpr int KS = padded_head(HR) / 32, HT = HR / 16;
  f32x4 dq[HT][2];              // column tiles x the wavefront's two tiles of 16 query rows
  bf16x8 qf[KS][2], gf[KS][2];  // slices of H x row tiles
  f32x4 start[2];               // -delta: what dP starts from, so that the contraction yields dP - delta
  Blocks16 ka;                  // K tile of the current buffer (the V tile stands dq_buf / 2 behind it)
  float c, lse2[2];
  int my_vis[2];                // number of leading local keys this lane's query rows see
  int grp;
};

// one 32-key x 32-query piece: T selects the half of the 64-key step.  S^T and dP^T in tiles of 16 keys (kt) x 16 queries
// (qt), lane = query, registers = keys 16 kt + 4 grp + 0..3; the two key tiles' registers are the eight contraction
// indices of a lane in dQ^T += K^T dS^T.  An A fragment serves both query tiles (slot i of the first contractions: slice
// i >> 1 of H, key tile i & 1); fragments run DQ_RING slots ahead of their use.
// masked: some of the wavefront's rows do not see all of its keys.
template <int T, int HR>
__device__ __forceinline__ void dq_piece(DqCtx<HR>& cx, int key0, bool masked) {
  constexpr int HD = padded_head(HR), DQ_RING = dq_ring(HD);
  constexpr int KS = DqCtx<HR>::KS, HT = DqCtx<HR>::HT, N = 2 * KS;
  constexpr int RB = T * 2 * KS * BLOCK, VT = dq_buf(HD) / 2;
  bf16x8 kr[DQ_RING], vr[DQ_RING], kt[DQ_RING];
  auto ld1 = [&](auto X) {
    constexpr int x = decltype(X)::value;
    const unsigned at = cx.ka.nat + RB + ((x & 1) * KS + (x >> 1)) * BLOCK;
    kr[x % DQ_RING] = lds_load_b128(at);
    vr[x % DQ_RING] = lds_load_b128(at + VT);
    __builtin_amdgcn_sched_barrier(0);
  };
  // K^T fragments; the first ones are on their way during the exponentials
  auto ld2 = [&](auto I) {
    constexpr int i = decltype(I)::value;
    const unsigned at = (i & 1 ? cx.ka.tr_o : cx.ka.tr_e) + RB + (i >> 1) * BLOCK;
    kt[i % DQ_RING] = lds_load_tr(at, at + KS * BLOCK);
    __builtin_amdgcn_sched_barrier(0);
  };
  static_for<0, DQ_RING>(ld1);
  f32x4 s[2][2], dp[2][2];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int q = 0; q < 2; ++q) { s[k][q] = f32x4{0.f, 0.f, 0.f, 0.f}; dp[k][q] = cx.start[q]; }
  static_for<0, N>([&](auto X) {
    constexpr int x = decltype(X)::value, k = x & 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      s[k][q] = mma16(kr[x % DQ_RING], cx.qf[x >> 1][q], s[k][q]);
      dp[k][q] = mma16(vr[x % DQ_RING], cx.gf[x >> 1][q], dp[k][q]);
    }
    if constexpr (x + DQ_RING < N) ld1(std::integral_constant<int, x + DQ_RING>{});
    else ld2(std::integral_constant<int, x + DQ_RING - N>{});
  });
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e >> 2][q][e & 3] = fast_exp2(fmaf(s[e >> 2][q][e & 3], cx.c, -cx.lse2[q]));
  if (A2D_SELDOM(masked)) {
    asm volatile("" ::: "memory");                 // keep this a branch
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (key0 + 16 * (e >> 2) + 4 * cx.grp + (e & 3) >= cx.my_vis[q]) s[e >> 2][q][e & 3] = 0.f;
  }
  bf16x8 dsb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) dsb[q][e] = (bf16_t)(s[e >> 2][q][e & 3] * dp[e >> 2][q][e & 3]);
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, HT>([&](auto I) {
    constexpr int i = decltype(I)::value;
#pragma unroll
    for (int q = 0; q < 2; ++q) cx.dq[i][q] = mma16(kt[i % DQ_RING], dsb[q], cx.dq[i][q]);
    if constexpr (i + DQ_RING < HT) ld2(std::integral_constant<int, i + DQ_RING>{});
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
  constexpr int KS = DqCtx<HR>::KS, HT = DqCtx<HR>::HT, DQ_BUF = dq_buf(HD);
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
  Q += (int64_t)head * d.lq.head + (GRID ? row_blk * g.b.q : 0);
  O += (int64_t)head * d.lo.head + (GRID ? row_blk * g.b.o : 0);
  dO += (int64_t)head * d.ldo.head + (GRID ? row_blk * g.b.g : 0);
  K += (int64_t)kvh * d.lk.head;
  V += (int64_t)kvh * d.lv.head;

  DqCtx<HR> cx;
  cx.grp = lane >> 4;
  cx.c = uniform(d.scale * kLog2e);
  const int q_row = q0 + wave * 32 + (lane & 15);      // of the first row tile
  // rows beyond nq re-read the last row, lse2 = +inf; columns past the head size are zero
  int64_t stat_at[2];                                  // (lse and delta: of the tile, or of the whole sequence)
  float lse_i[2];
  bf16x8 of[KS][2];                                    // delta = rowsum(dO o O)
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = min(q_row + 16 * q, d.nq - 1);
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      const int at = 32 * x + 8 * cx.grp, ld = min(at, H - 8);
      cx.qf[x][q] = *reinterpret_cast<const bf16x8*>(Q + (int64_t)r * d.lq.row + ld);
      cx.gf[x][q] = *reinterpret_cast<const bf16x8*>(dO + (int64_t)r * d.ldo.row + ld);
      of[x][q] = *reinterpret_cast<const bf16x8*>(O + (int64_t)r * d.lo.row + ld);
      if (32 * x + 32 > H && at >= H) cx.qf[x][q] = cx.gf[x][q] = of[x][q] = bf16x8{};
    }
    stat_at[q] = GRID ? (int64_t)head * g.b.side * d.nq + grid_token(g.b, d.nq, row_blk, r) : (int64_t)head * d.nq + r;
    lse_i[q] = lse[stat_at[q]];
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
#pragma unroll
    for (int q = 0; q < 2; ++q) cx.my_vis[q] = vis_count(min(q_row + 16 * q, d.nq - 1), s);
  };
#pragma unroll
  for (int t = 0; t < HT; ++t) cx.dq[t][0] = cx.dq[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  cx.ka.init(lane, lds_base);

  // ---- staging, straight into LDS: of eight wavefronts 0 .. 3 load a row tile of K each and 4 .. 7 one of V, each of four
  // one of both.  Block j of the sub-block of seg_rows keys that starts at local key seg_start; rows beyond its end
  // re-read its last row: finite values, masked out of the scores.
  // (Row strides in bytes, pinned in registers: read from the kernel arguments inside the loop they
  // would be scalar loads, which share a wait counter with the LDS reads in flight.  A head's rows
  // span less than 4 GiB - the API layer checks it - so row index times stride fits 32 bits.)
  // (cyclic grids: seg_start is the number of the grid's column, whose first row that is in the sequence)
  constexpr int LD_N = RW == 8 ? 1 : 2;            // matrices of a wavefront
  const int ld_first = RW == 8 ? wave >> 2 : 0, ld_tile = wave & 3, ld_row = 16 * ld_tile + (lane >> 2);
  const int ld_chunk = (lane & 3) ^ block_swap(lane >> 4);
  const char* ld_base[LD_N];
  unsigned ld_row_bytes[LD_N], ld_col_bytes[LD_N];
#pragma unroll
  for (int x = 0; x < LD_N; ++x) {
    const bool v = ld_first + x != 0;
    ld_base[x] = reinterpret_cast<const char*>(v ? V : K);
    ld_row_bytes[x] = __builtin_amdgcn_readfirstlane((unsigned)(v ? d.lv.row : d.lk.row) * 2);
    ld_col_bytes[x] = GRID == 2 ? __builtin_amdgcn_readfirstlane((unsigned)((v ? g.b.v : g.b.k) * 2)) : ld_row_bytes[x];
  }
  auto load_tile = [&](int seg_start, int seg_rows, int j, int boff) {
    const int r = min(ld_row, seg_rows - 1 - j * BKS);
#pragma unroll
    for (int x = 0; x < LD_N; ++x) {
      const gptr_t base = uniform_gptr(ld_base[x] + (seg_start * ld_col_bytes[x] + (unsigned)(j * BKS) * ld_row_bytes[x]));
      dma_blocks<KS, H>(lds_base + boff + (4 * (ld_first + x) + ld_tile) * KS * BLOCK, base,
                        __umul24(r, ld_row_bytes[x]) + 16 * ld_chunk, ld_chunk);
    }
  };
  if constexpr (H != HD) {                         // columns past the head size are zero for good
    for (int i = tid; i < 4 * BKS * (HD - H) / 8; i += DQ_THREADS) {
      const int row = i % BKS, x = i / BKS, tile = x / ((HD - H) / 8), ch = H % 32 / 8 + x % ((HD - H) / 8);
      *reinterpret_cast<u32x4*>(lds + tile * (DQ_BUF / 2) + ((row >> 4) * KS + H / 32) * BLOCK + (row & 15) * 64 +
                                16 * (ch ^ block_swap((row & 15) >> 2))) = u32x4{0, 0, 0, 0};
    }
  }

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
    load_tile(nx_start, nx_rows, j, 0);
  }
  wait_vmem_all();                                 // (the rows of Q, dO, O and the first tile together)
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bool ok = q_row + 16 * q < d.nq;
    cx.lse2[q] = (!ok || lse_i[q] == -INFINITY) ? INFINITY : lse_i[q] * kLog2e;      // +inf: exp2(s - lse2) = 0
    // (the order of sums of delta_kernel, so that both dQ paths give the same dK, dV: 16-byte chunks,
    // then chunks 1, 2, 4, 8 apart; this lane holds the chunks 4 x + grp)
    float t[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      t[x] = 0.f;
      if (x >= KS) continue;
      t[x] = dot8(__builtin_bit_cast(u32x4, of[x][q]), __builtin_bit_cast(u32x4, cx.gf[x][q]), 0.f);
      t[x] += __shfl_xor(t[x], 16, 64);
      t[x] += __shfl_xor(t[x], 32, 64);
    }
    const float del = (t[0] + t[1]) + (t[2] + t[3]);
    cx.start[q] = f32x4{-del, -del, -del, -del};
    if (delta && part == 0 && kl == 0 && cx.grp == 0 && ok) delta[stat_at[q]] = del;
  }
  __syncthreads();

  int boff = 0;
  while ((KL == 1 ? sb : lead_sb) < segs) {
    int nsb = sb, nj = j, nnblk = nblk;
    advance(stride, nsb, nj, nnblk);
    const bool more = nsb < segs;
    if (CYCLIC) nx_start = nsb;
    else if (A2D_SELDOM(more && nsb != sb)) { nx_start = seg_start(nsb); nx_rows = seg_rows(nsb); }
    const bool here = KL == 1 || sb < segs;         // this lane has a block in this round
    const int k0 = j * BKS + (CYCLIC && sb > shift_from);      // local to the sub-block
    if (A2D_OFTEN(more)) load_tile(nx_start, nx_rows, nj, DQ_BUF - boff);
    if (here && k0 < nvis_wave) dq_piece<0, HR>(cx, k0, k0 + 32 > nfull_wave);
    if (here && k0 + 32 < nvis_wave) dq_piece<1, HR>(cx, k0 + 32, k0 + 64 > nfull_wave);
    const int tog = boff ? -DQ_BUF : DQ_BUF;
    cx.ka.nat += tog; cx.ka.tr_e += tog; cx.ka.tr_o += tog;
    boff = DQ_BUF - boff;
    wait_vmem_all();
    __syncthreads();
    if (!CYCLIC && A2D_SELDOM(more && nsb != sb)) enter_segment(nsb);
    if (KL > 1) advance(stride, lead_sb, lead_j, lead_nblk);
    sb = nsb; j = nj; nblk = nnblk;
  }
  if constexpr (KL == 2) {
    // lane 1 hands its sums to lane 0 through LDS (the tiles are no longer read: every wavefront
    // has passed the walk's last barrier); layout [row wavefront][value][lane]: conflict free
    static_assert(RW * HT * 8 * 256 <= KL * 2 * DQ_BUF, "the exchange area must fit the tile buffers");
    float* xch = reinterpret_cast<float*>(lds_all) + wave * (HT * 8 * 64) + lane;
    if (kl == 1) {
#pragma unroll
      for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int r = 0; r < 8; ++r) xch[(8 * t + r) * 64] = cx.dq[t][r >> 2][r & 3];
    }
    __syncthreads();
    if (kl == 1) return;
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
      for (int r = 0; r < 8; ++r) cx.dq[t][r >> 2][r & 3] += xch[(8 * t + r) * 64];
  }
  // (KL = 2: inside what this wavefront has read of the exchange)
  char* const area = lds_all + wave * (KL == 2 ? HT * 8 * 256 : acc_area(HT));
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int first = q0 + wave * 32 + 16 * q;
    if (GRID && parts == 1) {
      bf16_t* const out = reinterpret_cast<bf16_t*>(dQ) + head * g.b.out[0].head + row_blk * g.b.out_step[0];
      store_acc16(out + first * g.b.out[0].row, g.b.out[0].row, d.nq - first, area, cx.dq, q, lane, d.scale);
    } else {
      const int64_t slot = (int64_t)part * (GRID ? g.b.side : 1) + row_blk;
      store_acc16(dQ + ((slot * d.heads + head) * d.nq + first) * H, H, d.nq - first, area, cx.dq, q, lane, d.scale,
                  !GRID && g.acc != 0);
    }
  }
}

}  // namespace mfma
}  // namespace a2d
