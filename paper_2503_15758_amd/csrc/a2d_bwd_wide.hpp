// The dK/dV workgroup of 256 keys, for tiles with many keys (see a2d_bwd_wide.hip for the kernel).
#pragma once
#include <type_traits>

#include "a2d_bwd.hpp"

namespace a2d {
namespace mfma {

// Eight wavefronts, two per SIMD, each with 32 keys of its own and all four contractions: both the
// dK^T and dV^T accumulators, K^T and V^T fragments in registers.  Against
// the pairs of bwd_dkdv_kernel nothing passes between wavefronts (no mailbox: a fifth of the LDS
// traffic), the two wavefronts of a SIMD run freely against each other, and a step - its barrier,
// its staging, its LDS latencies - holds twice the MFMAs.  In program order the exponentials stand
// under the dP MFMAs and the products dS under the dV MFMAs.  The scores start from -lse / scale
// and dP from -delta, so that p = exp2(c s) and dS = p dP need no further operand.
// Against the pairs: the call at 96 x 4096 x 4096 H = 128 2.80 -> 2.60 ms (dS kept: 2.60 -> 2.43 ms), at
// 32 x 1999 x 2777 H = 80 causal 217 -> 190 us.
// Bound by the chip's power at 1.8-1.9 GHz with the matrix units 55 % busy, so the contractions run on
// v_mfma_f32_16x16x32_bf16: an MFMA of 16 x 16 x 32 reads and writes half the accumulators per flop of one of 32 x 32 x 16
// (MFMAs alone on normal operands sustain 1.94-1.99 PFLOP/s against 1.72-1.76), and H = 80 fills five column tiles of 16
// instead of three of 32.  64 x 4096 x 4096, H = 128 / 96 / 80 / 64: 1065 / 749 / 697 / 571 -> 1010 / 727 / 669 / 543 us, 1199 ->
// 1183 with dS.  Each fragment still serves two MFMAs (the 32 keys of a wavefront), so the LDS reads are the same.
// Q and dO go straight into LDS, which leaves the registers that V^T needs at H = 128 (from LDS it was a sixth of
// the reads) and no writes of tiles in front of the barrier; three buffers, so that a step's requests have its whole length.
// Calls at 64 x 4096 x 4096, recomputing: 1608 / 1278 / 1196 / 968 -> 1575 / 1262 / 1167 / 941 us; 96 x 4096 x 4096 with dS 2377 ->
// 2302, 16 x 2048 x 2048 122.1 -> 116.6, 32 x 1999 x 2777 H = 80 causal 162.9 -> 156.3.
// (One wavefront per SIMD with two tiles of 32 keys, which halves the LDS reads again, issues too
// slowly: 2.8 us at H = 128.)
// Not for tiles with few keys, whose workgroups it halves (see plan_bwd_mfma).
constexpr int WK_KEYS = 256, WK_THREADS = 512;
// LDS: three buffers { Q tile, dO tile } in blocks | three of { -lse / scale [32], -delta [32] } | a wavefront's piece
// for turning dS
constexpr int WK_BUFS = 3;
__host__ __device__ constexpr int wk_tile(int hd) { return BQ * 2 * hd; }
__host__ __device__ constexpr int wk_stat(int hd) { return WK_BUFS * 2 * wk_tile(hd); }
__host__ __device__ constexpr int wk_turn(int hd) { return wk_stat(hd) + WK_BUFS * DK_STAT_BUF; }
constexpr int WK_TURN_BYTES = 32 * DS_TR_LD;
__host__ __device__ constexpr int wk_lds(int hd) { return wk_turn(hd) + 8 * WK_TURN_BYTES; }

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
  constexpr int HD = padded_head(HR), H = HR, TILE = wk_tile(HD), BUF = 2 * TILE;
  constexpr int KS = HD / 32, HT = HR / 16;        // slices of H in the first two contractions, column tiles of the others
  // At H = 128 the accumulators, K^T and V^T leave 64 registers: shorter fragment rings, and per-lane addresses
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
  const int l16 = lane & 15, grp = lane >> 4;
  Q += (int64_t)qh0 * d.lq.head;
  dO += (int64_t)qh0 * d.ldo.head;
  K += (int64_t)head * d.lk.head + (GRID ? col * g.b.k : 0);
  V += (int64_t)head * d.lv.head + (GRID ? col * g.b.v : 0);
  lse += (int64_t)qh0 * head_rows;
  delta += (int64_t)qh0 * head_rows;
  const float c = uniform(d.scale * kLog2e), inv_scale = uniform(1.0f / d.scale);

  // ---- K^T and V^T fragments of the wavefront's 32 keys, two tiles of 16: lane = key.  Keys beyond nkv
  // re-read the last key; the mask zeroes their probabilities.  (Columns past the head size are zero.)
  const int wk = k0 + wave * 32, key = wk + l16;   // (of tile 0)
  bf16x8 kf[KS][2], vf[KS][2];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int64_t r = min(key + 16 * kt, d.nkv - 1);
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      const int at = 32 * x + 8 * grp, ld = min(at, H - 8);
      kf[x][kt] = *reinterpret_cast<const bf16x8*>(K + r * d.lk.row + ld);
      vf[x][kt] = *reinterpret_cast<const bf16x8*>(V + r * d.lv.row + ld);
      if (32 * x + 32 > H && at >= H) kf[x][kt] = vf[x][kt] = bf16x8{};
    }
  }
  f32x4 dk[HT][2], dv[HT][2];
#pragma unroll
  for (int x = 0; x < HT; ++x)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) dk[x][kt] = dv[x][kt] = f32x4{0.f, 0.f, 0.f, 0.f};

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
  int my_first[2] = {nq, nq};                      // first row that sees this lane's keys; padding keys see nothing
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int k = key + 16 * kt;
    if (k >= d.nkv) continue;
    my_first[kt] = GRID && d.causal ? col_first + k : 0;
    if (!GRID && d.causal) {
      for (int sb = 0; sb < g.n; ++sb)
        if (k >= g.seg[sb].start && k < g.seg[sb].start + g.seg[sb].rows) my_first[kt] = seg_first_row(sb, k);
    }
  }
  int w_any = nq, w_all = nq;                      // rows below w_any see none of the wavefront's keys, from w_all on all
  if (wk < d.nkv) {
    first_row_range(wk, min(wk + 32, d.nkv), w_any, w_all);
    if (wk + 32 > d.nkv) w_all = nq;
  }
  // cyclic: the row blocks before the column see a key a row later than the others
  const int late = CYCLIC && d.causal ? col : 0;

  // ---- staging, straight into LDS: wavefront w loads the blocks w and w + 8 of { Q tile, dO tile }.  Step j + 2 is
  // requested while step j is computed; steps beyond the last re-stage it.  Rows beyond nq re-read the last row with a
  // statistic of -inf (p = 0).
  const gptr_t q_base = uniform_gptr(Q), g_base = uniform_gptr(dO);
  const unsigned q_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.row * 2);
  const unsigned g_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.ldo.row * 2);
  const unsigned q_head_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.head * 2);
  const unsigned g_head_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.ldo.head * 2);
  const unsigned q_blk_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.q * 2)) : 0;
  const unsigned g_blk_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.g * 2)) : 0;
  float stat = 0.f;                                // (wavefront 0: lse of 32 rows, delta of 32 rows)
  bool stat_ok = false;
  int ld_s = s0, ld_r = r0, ld_row0 = h0 * head_rows, ld_left = total - 1;   // the step to be loaded next
  unsigned ld_qh = h0 * q_head_bytes, ld_gh = h0 * g_head_bytes;
  auto load_step = [&](unsigned at) {              // into the buffer at `at`
    const int ln = TIGHT ? lane_again() : lane;
    const int i0 = i_start + ld_s * BQ, ch = (ln & 3) ^ block_swap(ln >> 4);
#pragma unroll
    for (int p = 0; p < (4 * KS + 7) / 8; ++p) {
      const int b = wave + 8 * p, m = b >= 2 * KS, t = (m ? b - 2 * KS : b) / KS, sl = (m ? b - 2 * KS : b) - t * KS;
      if (4 * KS % 8 != 0 && b >= 4 * KS) break;
      const unsigned r = (unsigned)min(i0 + 16 * t + (ln >> 2), nq - 1);
      const unsigned run = m ? ld_gh + (CYCLIC ? ld_r * g_blk_bytes : 0u) : ld_qh + (CYCLIC ? ld_r * q_blk_bytes : 0u);
      if (H == HD || 32 * sl + 8 * ch < H)
        dma_b128(at + b * BLOCK, m ? g_base : q_base, run + __umul24(r, m ? g_row_bytes : q_row_bytes) + 64 * sl + 16 * ch);
    }
    if (wave == 0) {
      const int ir = min(i0 + (ln & (BQ - 1)), nq - 1);
      const int i = ld_row0 + (CYCLIC ? ir * side + ld_r : ir);
      stat = (ln & BQ) ? delta[i] : lse[i];
      stat_ok = (i0 + (ln & (BQ - 1))) < nq;
    }
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
  auto store_stat = [&](int buf) {
    if (wave == 0) {
      const int ln = TIGHT ? lane_again() : lane;
      float v = -stat;
      if (ln < BQ) v = (!stat_ok || v == INFINITY) ? -INFINITY : v * inv_scale;
      else v = stat_ok ? v : 0.f;
      reinterpret_cast<float*>(lds + wk_stat(HD) + buf * DK_STAT_BUF)[ln] = v;
    }
  };
  if constexpr (H != HD) {                         // columns past the head size are zero for good
    for (int i = tid; i < WK_BUFS * 2 * BQ * (HD - H) / 8; i += WK_THREADS) {
      const int row = i % BQ, x = i / BQ, tile = x / ((HD - H) / 8), ch = H % 32 / 8 + x % ((HD - H) / 8);
      *reinterpret_cast<u32x4*>(lds + tile * TILE + ((row >> 4) * KS + H / 32) * BLOCK + (row & 15) * 64 +
                                16 * (ch ^ block_swap((row & 15) >> 2))) = u32x4{0, 0, 0, 0};
    }
  }
  if (total > 0) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      load_step(lds_base + b * BUF);
      store_stat(b);
    }
  }
  wait_vmem_all();
  __syncthreads();

  // dS hand-over: the wavefront's 32 keys are piece wave & 1 of key block 4 blk + wave / 2
  const unsigned ds_row_stride = (unsigned)ds_key_blocks(d.nkv) * DS_TILE_BYTES;
  const unsigned ds_wave_off = (unsigned)(8 * blk + wave) * (DS_TILE_BYTES / 2);
  const unsigned turn = lds_base + wk_turn(HD) + wave * WK_TURN_BYTES;
  gwptr_t ds_base = nullptr;
  if constexpr (WRITE_DS)
    ds_base = uniform_gwptr(reinterpret_cast<char*>(dS) + qh0 * ds_head_bytes(d.nq, d.nkv));

  Blocks16 da;
  da.init(lane, lds_base);
  unsigned st_addr = lds_base + wk_stat(HD) + 16 * grp;

  // One step: S and dP of the 32 rows in tiles of 16 rows (t) x 16 keys (kt), lane = key, registers = rows 16 t + 4 grp + 0..3.
  // The two row tiles' registers are the eight contraction indices of a lane in dV^T += dO^T P and dK^T += Q^T dS.  An A
  // fragment serves both key tiles.  Fragments in the order of their use: Q and dO rows (slice i >> 1, row tile i & 1),
  // transposed dO, transposed Q; each is requested RING fragments ahead.
  // (i0: its first row, `rows` those of a run - both one less where the keys are seen a row later)
  constexpr int N1 = 2 * KS, N2 = 4 * KS, N3 = N2 + HT, N4 = N3 + HT, RING = TIGHT || N4 % 4 != 0 ? 2 : 4;
  auto compute = [&](int i0, int rows, unsigned ds_off, bool masked) {
    bf16x8 a[RING];
    auto ld = [&](auto I) {
      constexpr int i = decltype(I)::value;
      if constexpr (i < N2) a[i % RING] = lds_load_b128(da.nat + (i < N1 ? 0 : TILE) + ((i & 1) * KS + (i % N1 >> 1)) * BLOCK);
      else if constexpr (i < N4) {
        constexpr int y = i < N3 ? i - N2 : i - N3;
        const unsigned at = (y & 1 ? da.tr_o : da.tr_e) + (i < N3 ? TILE : 0) + (y >> 1) * BLOCK;
        a[i % RING] = lds_load_tr(at, at + KS * BLOCK);
      }
    };
    static_for<0, RING>(ld);
    f32x4 s[2][2], dp[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) s[t][0] = s[t][1] = lds_load_f32x4(st_addr + 64 * t);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, N1>([&](auto I) {
      constexpr int i = decltype(I)::value, x = i >> 1, t = i & 1;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) s[t][kt] = mma16(a[i % RING], kf[x][kt], s[t][kt]);
      ld(std::integral_constant<int, i + RING>{});
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int t = 0; t < 2; ++t) dp[t][0] = dp[t][1] = lds_load_f32x4(st_addr + BQ * 4 + 64 * t);
    bf16x8 pb[2], sb[2];
    // Hidden pairs, and rows past the end, are taken out of the finished scores, not by where these start from: q.k may
    // have overflowed there.
    auto mask = [&]() {
      if (masked) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          const int first = i0 + 4 * grp - my_first[kt];
          const unsigned limit = CYCLIC ? max(rows - my_first[kt], 0) : rows - my_first[kt];   // (padding keys: none)
#pragma unroll
          for (int r = 0; r < 8; ++r)
            if ((unsigned)(first + 16 * (r >> 2) + (r & 3)) >= limit) s[r >> 2][kt][r & 3] = -INFINITY;
        }
      }
    };
    // score r of the lane's 16: key tile r >> 3, element r & 7 of its fragment
    auto prob = [&](int r) {
      const float p = fast_exp2(s[(r >> 2) & 1][r >> 3][r & 3] * c);
      s[(r >> 2) & 1][r >> 3][r & 3] = p;
      pb[r >> 3][r & 7] = (bf16_t)p;
    };
    auto dscore = [&](int r) { sb[r >> 3][r & 7] = (bf16_t)(s[(r >> 2) & 1][r >> 3][r & 3] * dp[(r >> 2) & 1][r >> 3][r & 3]); };
    static_for<0, N1>([&](auto I) {
      constexpr int i = decltype(I)::value, x = i >> 1, t = i & 1;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) dp[t][kt] = mma16(a[(N1 + i) % RING], vf[x][kt], dp[t][kt]);
      if constexpr (i == 0) mask();
#pragma unroll
      for (int r = 16 * i / N1; r < 16 * (i + 1) / N1; ++r) prob(r);
      ld(std::integral_constant<int, N1 + i + RING>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<0, HT>([&](auto Y) {
      constexpr int y = decltype(Y)::value;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) dv[y][kt] = mma16(a[(N2 + y) % RING], pb[kt], dv[y][kt]);
#pragma unroll
      for (int r = 16 * y / HT; r < 16 * (y + 1) / HT; ++r) dscore(r);
      ld(std::integral_constant<int, N2 + y + RING>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<0, HT>([&](auto Y) {
      constexpr int y = decltype(Y)::value;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) dk[y][kt] = mma16(a[(N3 + y) % RING], sb[kt], dk[y][kt]);
      ld(std::integral_constant<int, N3 + y + RING>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (WRITE_DS) {
      const int ln = TIGHT ? lane_again() : lane;
      bf16x8 out[2];
      ds_turn_write16(turn, ln, sb);
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
    const int free = buf == 0 ? 2 : buf - 1;       // the buffer of step j - 1 takes step j + 2
    load_step(lds_base + free * BUF);
    const int i0 = i_start + cs * BQ;
    const int sh = CYCLIC && cr < late ? 1 : 0;
    const bool here = min(i0 + BQ - 1, nq - 1) - sh >= w_any;
    const int next = buf == 2 ? -2 * BUF : BUF;
    if (here) {
      const unsigned off = (unsigned)rt * ds_row_stride + ds_wave_off;
      compute(i0 - sh, nq - sh, off, i0 - sh < w_all || i0 + BQ > nq);
    }
    if (!CYCLIC || ++cr == side) {
      const bool wrap = cs + 1 == nsteps;
      rt += wrap ? 1 + i_start / BQ : 1;
      cs = wrap ? 0 : cs + 1;
      cr = 0;
    }
    da.nat += next; da.tr_e += next; da.tr_o += next;
    st_addr += buf == 2 ? -2 * DK_STAT_BUF : DK_STAT_BUF;
    store_stat(free);
    buf = buf == 2 ? 0 : buf + 1;
    // (the tiles of step j + 2 have arrived; a step's two stores of dS, its last requests, may be under way)
    if (WRITE_DS && here) wait_vmem<2>(); else wait_vmem_all();
    __syncthreads();
  }

#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int k = key + 16 * kt;
    if (k >= d.nkv) continue;
    if (GRID && parts == 1) {
      bf16_t* const dkb = reinterpret_cast<bf16_t*>(dK) + head * g.b.out[1].head + col * g.b.out_step[1];
      bf16_t* const dvb = reinterpret_cast<bf16_t*>(dV) + head * g.b.out[2].head + col * g.b.out_step[2];
      store_acc16(dvb + k * g.b.out[2].row, dv, kt, grp, 1.0f);
      store_acc16(dkb + k * g.b.out[1].row, dk, kt, grp, d.scale);
    } else {
      const int64_t row = (int64_t)head * d.nkv + k;
      store_acc16(dV + row * H, dv, kt, grp, 1.0f);
      store_acc16(dK + row * H, dk, kt, grp, d.scale);
    }
  }
}

}  // namespace mfma
}  // namespace a2d
