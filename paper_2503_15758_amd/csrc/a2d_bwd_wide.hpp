// The dK/dV workgroup of 256 keys, for tiles with many keys (see a2d_bwd_wide.hip for the kernel).
#pragma once
#include <type_traits>

#include "a2d_bwd.hpp"

namespace a2d {
namespace mfma {

// Eight wavefronts, two per SIMD, each with 32 keys of its own and all four contractions: both the
// dK^T and dV^T accumulators, K^T fragments in registers and V^T fragments too (H = 128: in LDS).  Against
// the pairs of bwd_dkdv_kernel nothing passes between wavefronts (no mailbox: a fifth of the LDS
// traffic), the two wavefronts of a SIMD run freely against each other, and a step - its barrier,
// its staging, its LDS latencies - holds twice the MFMAs.  In program order the exponentials stand
// under the dP MFMAs and the products dS under the dV MFMAs.  The scores start from -lse / scale
// and dP from -delta, so that p = exp2(c s) and dS = p dP need no further operand.
// Measured per 32 rows x 256 keys, H = 128 / 96 / 80 / 64: 1.51 / 1.22 / 1.17 / 0.99 us against 2.26 / 1.92 /
// 1.86 / 1.58 us in pairs; the call at 96 x 4096 x 4096 H = 128 2.80 -> 2.60 ms (dS kept: 2.60 -> 2.43 ms), at
// 32 x 1999 x 2777 H = 80 causal 217 -> 190 us.
// (One wavefront per SIMD with two tiles of 32 keys, which halves the LDS reads again, issues too
// slowly: 2.8 us at H = 128.)
// Not for tiles with few keys, whose workgroups it halves (see plan_bwd_mfma).
constexpr int WK_KEYS = 256, WK_THREADS = 512;
// LDS: two buffers { Q tile, dO tile } | two of { -lse / scale [32], -delta [32] } | a wavefront's piece
// for turning dS | V (H = 128; rows of 272 bytes)
constexpr int WK_STAT = 2 * DK_BUF;
constexpr int WK_TURN = WK_STAT + 2 * DK_STAT_BUF;
constexpr int WK_TURN_BYTES = 32 * DS_TR_LD;
constexpr int WK_V = WK_TURN + 8 * WK_TURN_BYTES;
constexpr int WK_VLD = 272;
__host__ __device__ constexpr int wk_lds(int hd) { return WK_V + (hd == 128 ? WK_KEYS * WK_VLD : 0); }

// GRID: all key blocks of an emulated grid (g.b).  The workgroup walks the query rows of its whole grid column and
// writes rows of dK and dV of the sequence (of a split walk: a partial, [part][column][head][key]).  Contiguous blocks
// of queries are one run of rows; of cyclic ones, step s of every row block comes before step s + 1 of any.
// id: the workgroup's number among those of the tile.
template <int HR, bool WRITE_DS, int GRID>
__device__ __forceinline__ void dkdv_wide(
    int id, char* const lds, const a2d_tile_desc& d, const SegList& g, const int parts, const bf16_t* __restrict__ Q,
    const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dK, float* __restrict__ dV,
    bf16_t* __restrict__ dS) {
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  constexpr int HD = padded_head(HR), H = HR, CT = HD / 32;
  constexpr int KS = (HR + 15) / 16;               // slices of H that hold data
  constexpr bool V_LDS = HD == 128;
  // At H = 128 the accumulators and K^T leave 96 registers: shorter fragment rings, and per-lane addresses
  // that are used once a step are computed again in every step.
  constexpr bool TIGHT = HD == 128;
  const int kv_heads = d.heads / g.group;
  constexpr bool CYCLIC = GRID == 2;
  const int nkb = (d.nkv + WK_KEYS - 1) / WK_KEYS;
  int unit, blk;
  if (!xcd_map(id, kv_heads * parts, (GRID ? g.b.side : 1) * nkb, (GRID ? d.causal : g.by_size) != 0, unit, blk)) return;
  const Split up = split_by(unit, parts);
  const int head = up.q, part = up.r, qh0 = head * g.group;
  const GridBlock gb = GRID ? grid_column(g.b, nkb, blk) : GridBlock{0, blk};
  const int col = gb.r;                            // of the grid
  blk = gb.blk;
  if (!GRID || parts > 1) {
    const int64_t slot = (int64_t)part * (GRID ? g.b.side : 1) + col;
    dK += slot * kv_heads * d.nkv * H;
    dV += slot * kv_heads * d.nkv * H;
  }
  const int k0 = blk * WK_KEYS;
  const int side = CYCLIC ? __builtin_amdgcn_readfirstlane(g.b.side) : 1;      // row blocks that are walked in turn
  const int nq = GRID == 1 ? g.b.side * d.nq : d.nq, head_rows = nq * side;    // rows of a run; of a query head
  const int col_first = GRID == 1 && d.causal ? col * d.nkv : 0;               // the row that sees the column's first key
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l32 = lane & 31, half = lane >> 5;
  Q += (int64_t)qh0 * d.lq.head;
  dO += (int64_t)qh0 * d.ldo.head;
  K += (int64_t)head * d.lk.head + (GRID ? col * g.b.k : 0);
  V += (int64_t)head * d.lv.head + (GRID ? col * g.b.v : 0);
  lse += (int64_t)qh0 * head_rows;
  delta += (int64_t)qh0 * head_rows;
  const float c = d.scale * kLog2e, inv_scale = 1.0f / d.scale;

  // ---- K^T and V^T fragments of the wavefront's 32 keys: lane = key.  Keys beyond nkv
  // re-read the last key; the mask zeroes their probabilities.
  const int wk = k0 + wave * 32, key = wk + l32;
  bf16x8 kf[KS], vf[KS];
  {
    const int64_t r = min(key, d.nkv - 1);
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      kf[x] = *reinterpret_cast<const bf16x8*>(K + r * d.lk.row + 16 * x + 8 * half);
      vf[x] = *reinterpret_cast<const bf16x8*>(V + r * d.lv.row + 16 * x + 8 * half);
    }
  }
  f32x16 dk[CT], dv[CT];
#pragma unroll
  for (int x = 0; x < CT; ++x) { dk[x] = zero16(); dv[x] = zero16(); }

  // ---- which rows see which keys (as in bwd_dkdv_kernel)
  auto seg_first_row = [&](int sb, int r) -> int {
    const int64_t f = (int64_t)(r - g.seg[sb].start) - g.seg[sb].rel;
    return f <= 0 ? 0 : (f >= d.nq ? d.nq : (int)f);
  };
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
  first_row_range(k0, min(k0 + WK_KEYS, d.nkv), wg_lo, wg_hi);
  const int i_start = (wg_lo / BQ) * BQ;
  int nsteps = (nq - i_start + BQ - 1) / BQ;       // steps per run of rows
  // this part's steps: from step s0 of row block r0 of head h0 of the group on
  int total = nsteps * side * g.group, s0 = 0, r0 = 0, h0 = 0;
  if (parts > 1) {
    const int all = total, first = (int)((int64_t)part * all / parts);
    total = (int)((int64_t)(part + 1) * all / parts) - first;
    if (nsteps > 0) {
      h0 = first / (nsteps * side);
      s0 = first - h0 * (nsteps * side);
      if (CYCLIC) { r0 = s0 % side; s0 /= side; }
    }
  }
  int my_first = nq;                               // first row that sees this lane's key; padding keys see nothing
  if (key < d.nkv) {
    my_first = GRID && d.causal ? col_first + key : 0;
    if (!GRID && d.causal) {
      for (int sb = 0; sb < g.n; ++sb)
        if (key >= g.seg[sb].start && key < g.seg[sb].start + g.seg[sb].rows) my_first = seg_first_row(sb, key);
    }
  }
  int w_any = nq, w_all = nq;                      // rows below w_any see none of the wavefront's keys, from w_all on all
  if (wk < d.nkv) {
    first_row_range(wk, min(wk + 32, d.nkv), w_any, w_all);
    if (wk + 32 > d.nkv) w_all = nq;
  }
  // cyclic: the row blocks before the column see a key a row later than the others
  const int late = CYCLIC && d.causal ? col : 0;

  // ---- staging: thread moves chunk (tid & 15) of row (tid >> 4) of both tiles.  Step
  // j + 2 is requested while step j is computed and written to LDS an iteration later; steps beyond the
  // last re-stage it.  Rows beyond nq re-read the last row with a statistic of -inf (p = 0).
  const gptr_t q_base = uniform_gptr(Q), g_base = uniform_gptr(dO);
  const unsigned q_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.row * 2);
  const unsigned g_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.ldo.row * 2);
  const unsigned q_head_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.head * 2);
  const unsigned g_head_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.ldo.head * 2);
  const unsigned q_blk_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.q * 2)) : 0;
  const unsigned g_blk_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.g * 2)) : 0;
  u32x4 qreg, greg;
  float stat = 0.f;
  bool stat_ok = false;
  int ld_s = s0, ld_r = r0, ld_row0 = h0 * head_rows, ld_left = total - 1;   // the step to be loaded next
  unsigned ld_qh = h0 * q_head_bytes, ld_gh = h0 * g_head_bytes;
  auto load_step = [&]() {
    const int tid = TIGHT ? wave * 64 + lane_again() : threadIdx.x;
    const int st_row = tid >> 4, ld_ch = min(tid & 15, H / 8 - 1);
    const int i0 = i_start + ld_s * BQ;
    const unsigned r = (unsigned)min(i0 + st_row, nq - 1);
    qreg = gload_b128(q_base, ld_qh + (CYCLIC ? ld_r * q_blk_bytes : 0u) + __umul24(r, q_row_bytes) + ld_ch * 16);
    greg = gload_b128(g_base, ld_gh + (CYCLIC ? ld_r * g_blk_bytes : 0u) + __umul24(r, g_row_bytes) + ld_ch * 16);
    const int ir = min(i0 + (tid & (BQ - 1)), nq - 1);
    const int i = ld_row0 + (CYCLIC ? ir * side + ld_r : ir);
    stat = (tid & BQ) ? delta[i] : lse[i];
    stat_ok = (i0 + (tid & (BQ - 1))) < nq;
    bool more = ld_left > 0;
    ld_left -= more ? 1 : 0;
    if constexpr (CYCLIC) {                        // the next row block, then the next step
      const bool last = ld_r + 1 == side;
      ld_r = more ? (last ? 0 : ld_r + 1) : ld_r;
      more = more && last;
    }
    const bool wrap = ld_s + 1 == nsteps;
    ld_row0 += (more && wrap) ? head_rows : 0;
    ld_qh += (more && wrap) ? q_head_bytes : 0u;
    ld_gh += (more && wrap) ? g_head_bytes : 0u;
    ld_s = more ? (wrap ? 0 : ld_s + 1) : ld_s;
  };
  auto store_step = [&](int buf) {
    const int tid = TIGHT ? wave * 64 + lane_again() : threadIdx.x;
    const int st_row = tid >> 4, st_ch = tid & 15;
    const bool ch_data = st_ch * 8 < H, ch_tile = st_ch * 8 < HD;
    char* b = lds + buf * DK_BUF;
    if (HD == 128 || ch_tile) {
      const u32x4 zero = {0, 0, 0, 0};
      const int off = dual_store_off(st_row, st_ch);
      *reinterpret_cast<u32x4*>(b + off) = (HD == 128 || ch_data) ? qreg : zero;
      *reinterpret_cast<u32x4*>(b + DK_TILE + off) = (HD == 128 || ch_data) ? greg : zero;
    }
    if (tid < 2 * BQ) {
      float v = -stat;
      if (tid < BQ) v = (!stat_ok || v == INFINITY) ? -INFINITY : v * inv_scale;
      else v = stat_ok ? v : 0.f;
      reinterpret_cast<float*>(lds + WK_STAT + buf * DK_STAT_BUF)[tid] = v;
    }
  };
  if (total > 0) load_step();
  wait_vmem_all();
  if (total > 0) {
    store_step(0);
    load_step();
  }
  const unsigned v_nat = lds_base + WK_V + (wave * 32 + l32) * WK_VLD + 16 * half;
  if constexpr (V_LDS) {
#pragma unroll
    for (int x = 0; x < KS; ++x)
      *reinterpret_cast<__attribute__((address_space(3))) bf16x8*>((uintptr_t)(v_nat + 32 * x)) = vf[x];
  }
  __syncthreads();

  // dS hand-over: the wavefront's 32 keys are piece wave & 1 of key block 4 blk + wave / 2
  const unsigned ds_row_stride = (unsigned)ds_key_blocks(d.nkv) * DS_TILE_BYTES;
  const unsigned ds_wave_off = (unsigned)(8 * blk + wave) * (DS_TILE_BYTES / 2);
  const unsigned turn = lds_base + WK_TURN + wave * WK_TURN_BYTES;
  gwptr_t ds_base = nullptr;
  if constexpr (WRITE_DS)
    ds_base = uniform_gwptr(reinterpret_cast<char*>(dS) + qh0 * ds_head_bytes(d.nq, d.nkv));

  DualAddr da;
  da.init(lane, lds_base);
  unsigned st_addr = lds_base + WK_STAT + 16 * half;

  // One step.  Fragments (A operands) in the order of their use: Q and dO rows, transposed dO, transposed
  // Q; each is requested RING fragments ahead.
  // (i0: its first row, `rows` those of a run - both one less where the keys are seen a row later)
  auto compute = [&](int i0, int rows, unsigned ds_off, bool masked) {
    constexpr int N1 = KS, N2 = 2 * KS, N3 = N2 + 2 * CT, N4 = N3 + 2 * CT, RING = TIGHT ? 2 : 4;
    bf16x8 a[RING], va[2];
    auto ld = [&](auto I) {
      constexpr int i = decltype(I)::value;
      if constexpr (i < N1) a[i % RING] = dual_nat<i>(da, 0);
      else if constexpr (i < N2) a[i % RING] = dual_nat<i - N1>(da, DK_TILE);
      else if constexpr (i < N4) {
        constexpr int y = i < N3 ? i - N2 : i - N3;
        constexpr int at = (i < N3 ? DK_TILE : 0) + (y / CT) * 16 * DUAL_LD + 64 * (y % CT);
        a[i % RING] = lds_load_tr(da.tr_lo + at, da.tr_hi + at);
      }
    };
    auto ldv = [&](auto X) {
      constexpr int x = decltype(X)::value;
      if constexpr (V_LDS && x < KS) va[x & 1] = lds_load_b128(v_nat + 32 * x);
    };
    static_for<0, RING>(ld);
    f32x16 s, dp;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = lds_load_f32x4(st_addr + 32 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[4 * q + e] = v[e];
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, KS>([&](auto X) {
      constexpr int x = decltype(X)::value;
      s = mma(a[x % RING], kf[x], s);
      ld(std::integral_constant<int, x + RING>{});
      if constexpr (x + 2 >= KS) ldv(std::integral_constant<int, x + 2 - KS>{});
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = lds_load_f32x4(st_addr + BQ * 4 + 32 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) dp[4 * q + e] = v[e];
    }
    bf16x8 pb[2], sb[2];
    // Register r of a tile <-> row i0 + 8 (r >> 2) + 4 half + (r & 3).  Hidden pairs, and rows past the end, are
    // taken out of the finished scores, not by where these start from: q.k may have overflowed there.
    auto mask = [&]() {
      if (masked) {
        const int first = i0 + 4 * half - my_first;
        const unsigned limit = CYCLIC ? max(rows - my_first, 0) : rows - my_first;   // (padding keys: none)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if ((unsigned)(first + 8 * (r >> 2) + (r & 3)) >= limit) s[r] = -INFINITY;
      }
    };
    auto prob = [&](int r) {
      const float p = fast_exp2(s[r] * c);
      s[r] = p;
      pb[r >> 3][r & 7] = (bf16_t)p;
    };
    auto dscore = [&](int r) { sb[r >> 3][r & 7] = (bf16_t)(s[r] * dp[r]); };
    static_for<0, KS>([&](auto X) {
      constexpr int x = decltype(X)::value;
      dp = mma(a[(N1 + x) % RING], V_LDS ? va[x & 1] : vf[x], dp);
      if constexpr (x == 0) mask();
#pragma unroll
      for (int r = 16 * x / KS; r < 16 * (x + 1) / KS; ++r) prob(r);
      ld(std::integral_constant<int, N1 + x + RING>{});
      ldv(std::integral_constant<int, x + 2>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<0, 2 * CT>([&](auto Y) {
      constexpr int y = decltype(Y)::value;
      dv[y % CT] = mma(a[(N2 + y) % RING], pb[y / CT], dv[y % CT]);
#pragma unroll
      for (int r = 16 * y / (2 * CT); r < 16 * (y + 1) / (2 * CT); ++r) dscore(r);
      ld(std::integral_constant<int, N2 + y + RING>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<0, 2 * CT>([&](auto Y) {
      constexpr int y = decltype(Y)::value;
      dk[y % CT] = mma(a[(N3 + y) % RING], sb[y / CT], dk[y % CT]);
      ld(std::integral_constant<int, N3 + y + RING>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (WRITE_DS) {
      const int ln = TIGHT ? lane_again() : lane;
      bf16x8 out[2];
      ds_turn_write(turn, ln & 31, ln >> 5, sb);
      ds_turn_read(turn, ln, out);
      gstore_b128(ds_base, ds_off + 16 * ln, out[0]);
      gstore_b128(ds_base, ds_off + 16 * ln + 1024, out[1]);
    }
  };

  int cs = s0, cr = r0;                            // step inside its run, row block
  int rt = h0 * ds_row_tiles(d.nq) + s0 + i_start / BQ;   // dS row tile, counted over the group's heads
  int buf = 0;
#pragma nounroll
  for (int j = 0; j < total; ++j) {
    store_step(buf ^ 1);
    load_step();
    const int i0 = i_start + cs * BQ;
    const int sh = CYCLIC && cr < late ? 1 : 0;
    if (min(i0 + BQ - 1, nq - 1) - sh >= w_any) {
      const unsigned off = (unsigned)rt * ds_row_stride + ds_wave_off;
      compute(i0 - sh, nq - sh, off, i0 - sh < w_all || i0 + BQ > nq);
    }
    if (!CYCLIC || ++cr == side) {
      const bool wrap = cs + 1 == nsteps;
      rt += wrap ? 1 + i_start / BQ : 1;
      cs = wrap ? 0 : cs + 1;
      cr = 0;
    }
    da.shift(buf ? -DK_BUF : DK_BUF);
    st_addr += buf ? -DK_STAT_BUF : DK_STAT_BUF;
    buf ^= 1;
    __syncthreads();
  }

  if (GRID && parts == 1) {
    if (key < d.nkv) {
      bf16_t* const dkb = reinterpret_cast<bf16_t*>(dK) + head * g.b.out[1].head + col * g.b.out_step[1];
      bf16_t* const dvb = reinterpret_cast<bf16_t*>(dV) + head * g.b.out[2].head + col * g.b.out_step[2];
      store_acc_t<CT>(dvb + key * g.b.out[2].row, dv, half, 1.0f, H);
      store_acc_t<CT>(dkb + key * g.b.out[1].row, dk, half, d.scale, H);
    }
  } else if (key < d.nkv) {
    const int64_t row = (int64_t)head * d.nkv + key;
    store_acc_t<CT>(dV + row * H, dv, half, 1.0f, H);
    store_acc_t<CT>(dK + row * H, dk, half, d.scale, H);
  }
}

}  // namespace mfma
}  // namespace a2d
