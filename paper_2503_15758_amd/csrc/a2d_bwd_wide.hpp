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
// (MFMAs alone on normal operands sustained 1.94-1.99 PFLOP/s against 1.72-1.76 in a probe that is not kept), and H = 80 fills five column tiles of 16
// instead of three of 32.  64 x 4096 x 4096, H = 128 / 96 / 80 / 64: 1065 / 749 / 697 / 571 -> 1010 / 727 / 669 / 543 us, 1199 ->
// 1183 with dS.  Each fragment still serves two MFMAs (the 32 keys of a wavefront), so the LDS reads are the same.
// Q and dO go straight into LDS, which leaves the registers that V^T needs at H = 128 (from LDS it was a sixth of
// the reads) and no writes of tiles in front of the barrier.
// Calls at 64 x 4096 x 4096, recomputing: 1608 / 1278 / 1196 / 968 -> 1575 / 1262 / 1167 / 941 us; 96 x 4096 x 4096 with dS 2377 ->
// 2302, 16 x 2048 x 2048 122.1 -> 116.6, 32 x 1999 x 2777 H = 80 causal 162.9 -> 156.3.
// (One wavefront per SIMD with two tiles of 32 keys, which halves the LDS reads again, issues too
// slowly: 2.8 us at H = 128.)
// Not for tiles with few keys, whose workgroups it halves (see plan_bwd_mfma).
constexpr int WK_KEYS = 256, WK_THREADS = 512;
// A step is 64 query rows, computed 32 at a time: one barrier and one round of requests for twice the MFMAs (without the
// barriers of 32-row steps the kernel was 6 % faster, without their requests 14 %: both wavefronts of a SIMD make these at
// the same time).  64 x 4096 x 4096 as above 1548 / 1239 / 1136 / 912 -> 1522 / 1206 / 1111 / 891 us.
constexpr int WK_ROWS = 64;
// LDS: two buffers { Q tile, dO tile } in blocks | two of { -lse / scale [64], -delta [64] }
__host__ __device__ constexpr int wk_tile(int hd) { return WK_ROWS * 2 * hd; }
constexpr int WK_STAT_BUF = 2 * WK_ROWS * 4;
__host__ __device__ constexpr int wk_stat(int hd) { return 4 * wk_tile(hd); }
__host__ __device__ constexpr int wk_lds(int hd) {
  const int walk = wk_stat(hd) + 2 * WK_STAT_BUF, rows = 8 * acc_area(hd / 16);      // (16 keys of every wavefront go out at a time)
  return walk > rows ? walk : rows;
}

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
  // At H = 128 the accumulators, K^T and V^T leave 64 registers: shorter fragment rings, and per-lane values
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
  const int nsteps = (nq - i_start + WK_ROWS - 1) / WK_ROWS;       // steps per run of rows
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

  // ---- staging, straight into LDS: wavefronts 0 .. 3 load a row tile of Q each, 4 .. 7 of dO; wavefront 0 brings lse,
  // wavefront 1 delta.  Step j + 1 is requested while step j is computed; the last one re-stages itself.  Rows beyond
  // nq re-read the last row (the mask takes them out).  What a step's requests need is carried on by a few scalar
  // additions: both wavefronts of a SIMD stand here right behind the barrier, with no MFMA under way.
  const bool is_g = wave >= 4;
  const int ld_tile = 16 * (wave & 3);
  const bf16_t* const ld_base = is_g ? dO : Q;
  const unsigned ld_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)(is_g ? d.ldo.row : d.lq.row) * 2);
  const char* ld_at = nullptr;                     // the step to be loaded next: the wavefront's first row, ...
  int ld_s = s0, ld_r = r0, ld_h = h0, ld_left = total - 1;   // ... its step, row block and head
  auto open_run = [&]() {
    ld_at = reinterpret_cast<const char*>(ld_base + ld_h * (is_g ? d.ldo.head : d.lq.head) + (CYCLIC ? ld_r * (is_g ? g.b.g : g.b.q) : 0)) +
            (int64_t)(i_start + ld_s * WK_ROWS + ld_tile) * ld_row_bytes;
  };
  const auto stat_of = [&](int buf) { return lds_base + wk_stat(HD) + buf * WK_STAT_BUF + wave * (4 * WK_ROWS); };
  auto load_step = [&](int buf) {
    const int ln = TIGHT ? lane_again() : lane;
    const int i0 = i_start + ld_s * WK_ROWS, ch = (ln & 3) ^ block_swap(ln >> 4);
    int r = ln >> 2;
    const char* at = ld_at;
    if (A2D_SELDOM(i0 + WK_ROWS > nq)) {           // (from the step's first row on)
      at -= ld_tile * ld_row_bytes;
      r = min(r + ld_tile, nq - 1 - i0);
    }
    dma_blocks<KS, H>(lds_base + buf * BUF + wave * KS * BLOCK, uniform_gptr(at), __umul24(r, ld_row_bytes) + 16 * ch, ch);
    if (wave < 2) {
      const unsigned ir = min(i0 + ln, nq - 1);
      dma_b32<0>(stat_of(buf), uniform_gptr((wave == 0 ? lse : delta) + (int64_t)ld_h * head_rows + (CYCLIC ? ld_r : 0)),
                 (CYCLIC ? ir * side : ir) * 4);
    }
    if (ld_left > 0) {                             // the next step: of the next row block, or further down, or of the next head
      --ld_left;
      if (CYCLIC && ++ld_r < side) {
        ld_at += (is_g ? g.b.g : g.b.q) * 2;
      } else {
        ++ld_s;
        if (!CYCLIC && A2D_OFTEN(ld_s < nsteps)) {
          ld_at += (int64_t)ld_row_bytes * WK_ROWS;
        } else {
          if (CYCLIC) ld_r = 0;
          if (ld_s == nsteps) { ld_s = 0; ++ld_h; }
          open_run();
        }
      }
    }
  };
  // What the wavefront has brought of lse or delta becomes what the scores or dP start from, half a step after its request.  (Loaded
  // into a register that waits for its place to be free, it was one register too many at H = 128: kept in scratch, and the
  // wait for it in front of the store is one for the tiles just requested.  Turned where it is read it would cost every
  // wavefront some twenty vector instructions a half step.  With it, and c, 1 / scale and the mask's limits out of the vector registers,
  // nothing is in scratch: us, 8192 tokens of 16 heads on 4 x 4, causal, both passes 1012 -> 992, 96 x 4096 x 4096 with dS 2059 ->
  // 2049.)
  auto turn_stat = [&](int buf) {
    if (wave < 2) {
      auto* const at = reinterpret_cast<__attribute__((address_space(3))) float*>((uintptr_t)(stat_of(buf) + 4 * (TIGHT ? lane_again() : lane)));
      float v = -*at;
      if (wave == 0) v = v == INFINITY ? -INFINITY : v * inv_scale;
      *at = v;
    }
  };
  if constexpr (H != HD) {                         // columns past the head size are zero for good
    for (int i = tid; i < 4 * WK_ROWS * (HD - H) / 8; i += WK_THREADS) {
      const int row = i % WK_ROWS, x = i / WK_ROWS, tile = x / ((HD - H) / 8), ch = H % 32 / 8 + x % ((HD - H) / 8);
      *reinterpret_cast<u32x4*>(lds + tile * TILE + ((row >> 4) * KS + H / 32) * BLOCK + (row & 15) * 64 +
                                16 * (ch ^ block_swap((row & 15) >> 2))) = u32x4{0, 0, 0, 0};
    }
  }
  if (total > 0) {
    open_run();
    load_step(0);
  }
  wait_dma();
  if (total > 0) turn_stat(0);
  __syncthreads();

  // dS hand-over: the wavefront's 32 keys are piece wave & 1 of key block 4 blk + wave / 2
  const unsigned ds_row_stride = (unsigned)ds_key_blocks(d.nkv) * DS_TILE_BYTES;
  const unsigned ds_wave_off = (unsigned)(8 * blk + wave) * (DS_TILE_BYTES / 2);
  gwptr_t ds_base = nullptr;
  if constexpr (WRITE_DS)
    ds_base = uniform_gwptr(reinterpret_cast<char*>(dS) + qh0 * ds_head_bytes(d.nq, d.nkv));

  Blocks16 da;
  da.init(lane, lds_base);
  unsigned st_addr = lds_base + wk_stat(HD) + 16 * grp;

  // Half a step: S and dP of 32 rows in tiles of 16 rows (t) x 16 keys (kt), lane = key, registers = rows 16 t + 4 grp + 0..3.
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
        const unsigned at = (y & 1 ? da.tr_e ^ 32 : da.tr_e) + (i < N3 ? TILE : 0) + (y >> 1) * BLOCK;   // (da.tr_o: made where it is used)
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
    for (int t = 0; t < 2; ++t) dp[t][0] = dp[t][1] = lds_load_f32x4(st_addr + WK_ROWS * 4 + 64 * t);
    bf16x8 pb[2], sb[2];
    // Hidden pairs, and rows past the end, are taken out of the finished scores, not by where these start from: q.k may
    // have overflowed there.
    auto mask = [&]() {
      if (masked) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          int mine = my_first[kt];
          if constexpr (TIGHT) asm volatile("" : "+v"(mine));   // (the limit would be kept for all steps)
          const int first = i0 + 4 * (TIGHT ? lane_again() >> 4 : grp) - mine;
          const unsigned limit = CYCLIC ? max(rows - mine, 0) : rows - mine;   // (padding keys: none)
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
      gstore_b128(ds_base, ds_off + 16 * ln, sb[0]);
      gstore_b128(ds_base, ds_off + 16 * ln + 1024, sb[1]);
    }
  };

  constexpr int HALF = 2 * KS * BLOCK;             // of a tile
  int cs = s0, cr = r0, chd = h0;                  // step inside its run, row block, head
  int buf = 0;
#pragma nounroll
  for (int j = 0; j < total; ++j) {
    load_step(buf ^ 1);
    const int sh = CYCLIC && cr < late ? 1 : 0;
    int stored = 0;                                // vector memory operations since the requests: stores of dS, which may be under way
#pragma nounroll
    for (int h = 0; h < 2; ++h) {
      const int i0 = i_start + cs * WK_ROWS + h * BQ;
      if (i0 < nq && min(i0 + BQ - 1, nq - 1) - sh >= w_any) {
        const unsigned off = (unsigned)(chd * ds_row_tiles(d.nq) + i0 / BQ) * ds_row_stride + ds_wave_off;
        compute(i0 - sh, nq - sh, off, i0 - sh < w_all || i0 + BQ > nq);
        stored += 2;
      }
      const int go = h == 0 ? HALF : buf ? -BUF - HALF : BUF - HALF;
      da.nat += go; da.tr_e += go;
      st_addr += h == 0 ? BQ * 4 : buf ? -WK_STAT_BUF - BQ * 4 : WK_STAT_BUF - BQ * 4;
      if (h == 0 && wave < 2) {                    // (requested half a step ago)
        if (WRITE_DS && stored) wait_dma<2>(); else wait_dma();
        turn_stat(buf ^ 1);
      }
    }
    if (!CYCLIC || ++cr == side) {
      cr = 0;
      if (++cs == nsteps) { cs = 0; ++chd; }
    }
    buf ^= 1;
    // (the next tiles)
    if (WRITE_DS && stored == 4) wait_dma<4>();
    else if (WRITE_DS && stored == 2) wait_dma<2>();
    else wait_dma();
    __syncthreads();
  }

  char* const area = lds + wave * acc_area(HT);
  const int ln = TIGHT ? lane_again() : lane;      // (the one of the start would be kept in scratch until here)
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int first = wk + 16 * kt, n = d.nkv - first;
    if (GRID && parts == 1) {
      bf16_t* const dkb = reinterpret_cast<bf16_t*>(dK) + head * g.b.out[1].head + col * g.b.out_step[1];
      bf16_t* const dvb = reinterpret_cast<bf16_t*>(dV) + head * g.b.out[2].head + col * g.b.out_step[2];
      store_acc16(dvb + first * g.b.out[2].row, g.b.out[2].row, n, area, dv, kt, ln, 1.0f);
      store_acc16(dkb + first * g.b.out[1].row, g.b.out[1].row, n, area, dk, kt, ln, d.scale);
    } else {
      const int64_t at = ((int64_t)head * d.nkv + first) * H;
      store_acc16(dV + at, H, n, area, dv, kt, ln, 1.0f);
      store_acc16(dK + at, H, n, area, dk, kt, ln, d.scale);
    }
  }
}

}  // namespace mfma
}  // namespace a2d
