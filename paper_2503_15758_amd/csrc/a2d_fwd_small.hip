// bf16 MFMA forward tile kernel for short calls: the contractions of a2d_fwd_mfma.hip, 32 or 64 query rows per workgroup.
//
// A call of few query rows leaves most of the chip without work when its blocks are 128 rows, and sharing their
// walks between workgroups costs partial results in memory and a launch that merges them.  Here the eight
// wavefronts of a workgroup hold the SAME 32 rows and take every eighth slab of 32 keys; their (N, m, l) are
// merged through LDS at the end.  Nothing is shared during the walk of 32 rows, so there is no barrier in it: each wavefront
// stages its slabs in a piece of LDS of its own.  (K read straight into the A operands, a lane a row, goes 32 lines at a
// time through an L1 that eight wavefronts share: 13.5 us became 16.4 at 8 x 1024 x 1024, H = 128.)
// What bounds it: launch, argument and first-load latencies below two rounds of slabs; then what a compute unit reads
// from L2, 128 KiB a round at H = 128 (its MFMAs take a third of that time), since every 32 rows read all keys they see.  For
// short calls that is cheaper than partial results and a second launch, for long ones not (see plan_fwd_mfma).
// So that the reads are always under way: operands go straight into LDS, without registers in between, the next K slab as soon
// as this one's scores are there, the next V behind the last product; Q once for the workgroup instead of once for each
// wavefront.  Against a slab by way of registers, requested before the one at hand is computed, and 32 x 32 x 16 MFMAs:
// H = 128 2 x 512 x 512 9.5 -> 7.9 us, 8 x 1024 x 1024 13.1 -> 10.8, 4 x 2048 x 2048 19.7 -> 16; H = 96 4 x 400 x 400 8.0 -> 6.8;
// H = 80 8 x 700 x 900 10.6 -> 9.1; H = 64 2 x 512 x 512 6.2 -> 5.9, 4 x 2048 x 2048 11.9 -> 11.0.  (H = 64 with Q in LDS too is
// 0.3 us slower: there the wavefronts' own loads of Q are the shorter way.)
// Where 32-row blocks no longer run at once, 64 rows in four lanes of two wavefronts that stage their slabs together read half
// as much and need a barrier a round: H = 128 16 x 1024 x 1024 16.2 us against 20.6 in 32 rows, 8 x 2048 x 2048 25.4 / 30.3;
// H = 64 32 x 512 x 512 8.2 / 11.2.
// Against the other forms of today (128 rows in two key lanes, unshared): 4 x 2048 x 2048 33.2 us for 16.2, 8 x 1024 x 1024 20.5
// for 10.8.
#include "a2d_mfma.hpp"

namespace a2d {
namespace {

using namespace mfma;

constexpr int SB = 32, WAVES = 8;                  // keys of a slab, wavefronts
// LDS: eight { K slab, V slab } (in blocks, as in a2d_fwd_mfma.hip) | m, l of every wavefront's rows | the workgroup's Q
constexpr int STAT = WAVES * 16 * 1024;            // (the slabs at H = 128; every wavefront's results at the end)
constexpr int Q_AT = STAT + 2 * WAVES * SB * 4;
constexpr int lds_bytes(int rg, int hd) { return Q_AT + (hd > 64 ? rg * 64 * hd : 0); }
constexpr float kRescaleThreshold = 8.0f;          // log2 units

// RG: groups of 32 rows.  1: eight key lanes, each wavefront its own slab.  2: 64 rows and four lanes of two wavefronts that
// stage a slab together, two buffers each: half the reads from L2, a barrier a round.
// (GRID, arguments and outputs as of fwd_mfma_kernel)
template <int HR, int RG, int GRID>
__global__ __launch_bounds__(64 * WAVES, 1) void fwd_small_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, float* O_part, float* m_out, float* l_out, FwdInput in) {
  constexpr int HD = padded_head(HR), H = HR, KS = HD / 32, HT = HR / 16;
  constexpr int V_AT = 2 * KS * BLOCK, SLAB_BYTES = 2 * V_AT;
  static_assert(WAVES * SLAB_BYTES <= STAT && HT * 2 <= 16, "slabs and results must fit");
  constexpr bool PLAIN = GRID == 0, CYCLIC = GRID == 2;
  warm_arguments<9 * 8>();
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  constexpr int LANES = WAVES / RG, BM = 32 * RG;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kl = wave / RG, rg = wave % RG;        // key lane, row group
  const int grp = lane >> 4, l16 = lane & 15;

  const int nqb = (d.nq + BM - 1) / BM;
  int unit, blk;
  const int by_size = GRID ? d.causal : g.by_size;
  if (!xcd_map(blockIdx.x, d.heads / g.group * g.parts, (GRID ? g.b.side : 1) * g.group * nqb, by_size != 0, unit, blk,
               kXcdCus)) return;
  const Split up = split_by(unit, g.parts);
  const int kvh = up.q, part = up.r;
  const Split in_group = query_head(blk, g.group, nqb, GRID || by_size);
  const int head = kvh * g.group + in_group.r;
  blk = in_group.q;
  const GridBlock gb = GRID ? grid_block(g.b, nqb, blk) : GridBlock{0, blk};
  const int row_blk = gb.r;                        // of the grid
  blk = gb.blk;
  const int q0 = (nqb - 1 - blk) * BM, w0 = q0 + 32 * rg;
  Q += (int64_t)head * d.lq.head + (GRID ? row_blk * g.b.q : 0);
  K += (int64_t)kvh * d.lk.head;
  V += (int64_t)kvh * d.lv.head;
  if (!GRID || !g.norm) {
    const int64_t slot = ((int64_t)part * (GRID ? g.b.side : 1) + row_blk) * d.heads * d.nq;
    O_part += slot * HR;
    m_out += slot;
    l_out += slot;
  }

  // ---- Q comes in once for all wavefronts, through LDS (at H = 64 it is little, and every wavefront loads its fragments);
  // rows beyond nq re-read the last row, columns past the head size are zero
  constexpr bool Q_LDS = HD > 64;
  const int q_row = w0 + l16;                      // of the first of the wavefront's two tiles of 16
  const int ld_chunk = (lane & 3) ^ block_swap(lane >> 4);
  bf16x8 qf[KS][2];
  if constexpr (Q_LDS) {
    const unsigned q_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lq.row * 2);
#pragma unroll
    for (int p = 0; p < (2 * RG * KS + WAVES - 1) / WAVES; ++p) {
      const int b = wave + WAVES * p, tile = b / KS, sl = b - tile * KS;
      if (2 * RG * KS % WAVES != 0 && b >= 2 * RG * KS) break;
      if (H == HD || 32 * sl + 8 * ld_chunk < H)
        dma_b128<0>(lds_base + Q_AT + b * BLOCK, uniform_gptr(reinterpret_cast<const char*>(Q) + 64 * sl),
                    __umul24((unsigned)min(q0 + 16 * tile + (lane >> 2), d.nq - 1), q_row_bytes) + 16 * ld_chunk);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int x = 0; x < KS; ++x)
        qf[x][q] = *reinterpret_cast<const bf16x8*>(Q + (int64_t)min(q_row + 16 * q, d.nq - 1) * d.lq.row + 32 * x + 8 * grp);
  }
  const float c = d.scale * kLog2e;

  // ---- visibility and the walk over (sub-block, slab), as in fwd_mfma_kernel
  const int last_row = min(q0 + BM - 1, d.nq - 1);
  const int segs = PLAIN ? g.n : CYCLIC ? g.b.side : 1, stride = LANES * g.parts;
  const int shift_from = CYCLIC && d.causal ? row_blk : segs;
  // the sub-block to be loaded from (cyclic: start is the grid's column); the keys of it that row i sees
  int start = 0, rows = GRID == 1 ? g.b.side * d.nkv : d.nkv;
  int64_t rel = 0;
  auto vis_count = [&](int i) -> int {
    if (GRID == 1) return d.causal ? row_blk * d.nq + i + 1 : rows;
    if (GRID == 2) return d.causal ? i + 1 : rows;
    if (!d.causal) return rows;
    const int64_t v = (int64_t)i + rel + 1;
    return v <= 0 ? 0 : (v < rows ? (int)v : rows);
  };
  int nfull = 0, nvis = 0, my_vis[2] = {0, 0};     // keys of the current sub-block that all rows see, some row, the lane's
  auto enter_segment = [&]() {
    nfull = vis_count(min(w0, d.nq - 1));
    if (RG > 1) nvis = vis_count(min(w0 + 31, d.nq - 1));
#pragma unroll
    for (int q = 0; q < 2; ++q) my_vis[q] = vis_count(min(q_row + 16 * q, d.nq - 1));
  };
  auto open_segment = [&](int s, int& sb, int& n) {
    for (n = 0; s < segs; ++s) {
      if (PLAIN) {
        start = g.seg[s].start;
        rows = g.seg[s].rows;
        rel = g.seg[s].rel;
      }
      n = (vis_count(last_row) + SB - 1) / SB;
      if (n > 0) break;
    }
    sb = s;
  };
  auto advance = [&](int by, int& sb, int& j, int& n) {
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
        open_segment(sb + 1, sb, n);
      }
    }
  };

  // ---- staging, straight into LDS: a wavefront loads all blocks of its slab, or (RG > 1) those of one row tile.  Rows beyond
  // the sub-block re-read its last one.
  constexpr int ST_N = 2 / RG;                     // row tiles of a wavefront
  const unsigned k_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lk.row * 2);
  const unsigned v_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lv.row * 2);
  const unsigned k_col_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.k * 2)) : k_row_bytes;
  const unsigned v_col_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.v * 2)) : v_row_bytes;
  const int ld_tile = RG > 1 ? rg : 0;
  const unsigned slab = lds_base + kl * RG * SLAB_BYTES;     // (RG > 1: the first of two)
  gptr_t k_from, v_from;                           // of the slab to be loaded
  int ld_last = 0;
  auto locate = [&](int s, int j) {
    if (CYCLIC) start = s;
    k_from = uniform_gptr(reinterpret_cast<const char*>(K) + (start * k_col_bytes + (unsigned)(j * SB) * k_row_bytes));
    v_from = uniform_gptr(reinterpret_cast<const char*>(V) + (start * v_col_bytes + (unsigned)(j * SB) * v_row_bytes));
    ld_last = rows - 1 - j * SB;
  };
  constexpr int LOADS = ST_N * KS;                 // of a K or V slab
  auto load = [&](bool v, unsigned buf) {
#pragma unroll
    for (int t = 0; t < ST_N; ++t) {
      const int tile = ld_tile + t, r = min(16 * tile + (lane >> 2), ld_last);
      const unsigned off = __umul24(r, v ? v_row_bytes : k_row_bytes) + 16 * ld_chunk;
      dma_blocks<KS, H>(slab + buf + (v ? V_AT : 0) + tile * KS * BLOCK, v ? v_from : k_from, off, ld_chunk);
    }
  };
  if constexpr (H != HD) {
    // the columns of Q and the K slabs past the head size are zero for good (those of V are not read)
    for (int i = threadIdx.x; i < (WAVES + RG) * SB * (HD - H) / 8; i += 64 * WAVES) {
      const int row = i % SB, x = i / SB, sl = x / ((HD - H) / 8), ch = H % 32 / 8 + x % ((HD - H) / 8);
      *reinterpret_cast<u32x4*>(lds + (sl < WAVES ? sl * SLAB_BYTES : Q_AT + (sl - WAVES) * V_AT) + ((row >> 4) * KS + H / 32) * BLOCK + (row & 15) * 64 +
                                16 * (ch ^ block_swap((row & 15) >> 2))) = u32x4{0, 0, 0, 0};
    }
  }
  Blocks16 rd;
  rd.init(lane, slab);

  // rounds of the workgroup's first lane, which has the longest walk (RG > 1: all lanes keep its barriers)
  int rounds = 0;
  if constexpr (RG > 1) {
    int all = 0;
    for (int s = 0; s < (PLAIN ? segs : 1); ++s) {
      if (PLAIN) {
        rows = g.seg[s].rows;
        rel = g.seg[s].rel;
      }
      all += (vis_count(last_row) + SB - 1) / SB;
    }
    if (CYCLIC) all *= segs;
    all -= part * LANES;
    rounds = all > 0 ? split_by(all + stride - 1, stride).q : 0;
  }
  int sb, j = 0, n;
  open_segment(0, sb, n);
  if (sb < segs) advance(part * LANES + kl, sb, j, n);
  if (sb < segs) {
    locate(sb, j);
    load(false, 0);
    load(true, 0);
    enter_segment();
  }

  f32x4 o[HT][2];
#pragma unroll
  for (int t = 0; t < HT; ++t) o[t][0] = o[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_lane[2] = {-INFINITY, -INFINITY}, m_ref[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
  if (!GRID && g.acc && part == 0 && kl == 0) {
    // the first wavefront continues the stored partial (rows past nq: the last row's, never stored)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t row = (int64_t)head * d.nq + min(q_row + 16 * q, d.nq - 1);
      m_lane[q] = m_ref[q] = in.m[row] / d.scale;
      l_run[q] = grp == 0 ? in.l[row] : 0.f;
#pragma unroll
      for (int t = 0; t < HT; ++t) o[t][q] = *reinterpret_cast<const f32x4*>(in.N + row * H + 16 * t + 4 * grp);
    }
  }

  bool more = false;                               // there is a next slab
  auto wait_behind = [&] {
    if (more) wait_dma<LOADS>(); else wait_dma();
  };
  if constexpr (Q_LDS) {
    if (sb < segs) wait_dma<2 * LOADS>(); else wait_dma();     // this wavefront's share, then everybody's
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int x = 0; x < KS; ++x) qf[x][q] = lds_load_b128(rd.nat - slab + lds_base + Q_AT + ((2 * rg + q) * KS + x) * BLOCK);
  }
  // S^T and O^T in tiles of 16 x 16, as in fwd_block.  behind: called when the K slab has been read.
  auto compute = [&](unsigned buf, auto&& behind) {
    const unsigned k_at = rd.nat + buf, v_e = rd.tr_e + buf + V_AT, v_o = rd.tr_o + buf + V_AT;
    const int k0 = j * SB + (CYCLIC && sb > shift_from);
    f32x4 s[2][2];
#pragma unroll
    for (int k = 0; k < 2; ++k) s[k][0] = s[k][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < KS; ++x)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const bf16x8 a = lds_load_b128(k_at + (k * KS + x) * BLOCK);
#pragma unroll
        for (int q = 0; q < 2; ++q) s[k][q] = mma16(a, qf[x][q], s[k][q]);
      }
    behind();
    if (k0 + SB > nfull) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 8; ++r)
          if (k0 + 16 * (r >> 2) + 4 * grp + (r & 3) >= my_vis[q]) s[r >> 2][q][r & 3] = -INFINITY;
    }
    bool grow = false;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float mx = m_lane[q];
#pragma unroll
      for (int r = 0; r < 8; ++r) mx = fmaxf(mx, s[r >> 2][q][r & 3]);
      m_lane[q] = mx;
      grow |= (mx - m_ref[q]) * c > kRescaleThreshold;
    }
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
      asm volatile("" ::: "memory");               // (a real branch, as in fwd_block)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float m_row = row_max(m_lane[q]);
        const float m_use = (m_row == -INFINITY) ? 0.f : m_row;
        const float alpha = fast_exp2((m_ref[q] - m_use) * c);
        m_ref[q] = m_row;
        l_run[q] *= alpha;
#pragma unroll
        for (int t = 0; t < HT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[t][q][r] *= alpha;
      }
    }
    bf16x8 pb[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float mc = (m_ref[q] == -INFINITY) ? 0.f : m_ref[q] * c;
      float psum = 0.f;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const float p = fast_exp2(fmaf(s[r >> 2][q][r & 3], c, -mc));
        psum += p;
        pb[q][r] = (bf16_t)p;
      }
      l_run[q] += psum;
    }
    if constexpr (RG == 1) wait_behind();   // V has arrived
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      const unsigned at = (t & 1 ? v_o : v_e) + (t >> 1) * BLOCK;
      const bf16x8 a = lds_load_tr(at, at + KS * BLOCK);
#pragma unroll
      for (int q = 0; q < 2; ++q) o[t][q] = mma16(a, pb[q], o[t][q]);
    }
  };
  if constexpr (RG == 1) {
    // One slab a wavefront: the next K goes where the last one was read from while the exponentials and V P^T are under way,
    // the next V behind those.  (In flight at a time: V and the next K, the next K and V.)
    if (sb < segs) wait_dma<LOADS>();             // (K)
    while (sb < segs) {
      int nsb = sb, nj = j, nn = n;
      advance(stride, nsb, nj, nn);
      more = nsb < segs;
      if (more) locate(nsb, nj);
      compute(0, [&] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more) load(false, 0);
      });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) {
        load(true, 0);
        wait_dma<LOADS>();
      }
      if (!CYCLIC && nsb != sb && more) enter_segment();
      sb = nsb; j = nj; n = nn;
    }
  } else {
    wait_dma();
    __syncthreads();
    unsigned buf = 0;
    for (int r = 0; r < rounds; ++r) {
      int nsb = sb, nj = j, nn = n;
      advance(stride, nsb, nj, nn);
      more = nsb < segs;
      if (more) {
        locate(nsb, nj);
        load(false, SLAB_BYTES - buf);
        load(true, SLAB_BYTES - buf);
      }
      if (sb < segs && j * SB + (CYCLIC && sb > shift_from) < nvis) compute(buf, [] {});
      wait_dma();
      __syncthreads();
      if (!CYCLIC && more && nsb != sb) enter_segment();
      sb = nsb; j = nj; n = nn;
      buf = SLAB_BYTES - buf;
    }
  }

  // ---- the wavefronts' (N, m, l) become one, as partials of one query block do (Alg. 2)
  // (the lanes of a wavefront's first 32 hold its rows' sums in turn; row_pair hands all lanes those of their two rows)
  float* const xm = reinterpret_cast<float*>(lds + STAT) + rg * 32 + (lane & 31);
  float* const xl = xm + WAVES * 32;
  float m_row[2], l_row[2], f[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    m_row[q] = row_max(m_lane[q]);
    f[q] = (m_row[q] == -INFINITY) ? 0.f : fast_exp2((m_ref[q] - m_row[q]) * c);
    l_row[q] = row_sum(l_run[q]) * f[q];
  }
  if (lane < 32) {
    xm[kl * BM] = m_row[grp & 1];
    xl[kl * BM] = l_row[grp & 1];
  }
  __syncthreads();
  f32x4* const x = reinterpret_cast<f32x4*>(lds);
  const bool norm = g.norm != 0;
  float m_new = -INFINITY, l_tot = 0.f, use[2], fn[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < LANES; ++k) m_new = fmaxf(m_new, xm[k * BM]);
  const float m_use = m_new == -INFINITY ? 0.f : m_new;        // (2^-inf = 0 for the wavefronts that saw nothing)
  row_pair(m_use, use);
  if (norm || kl == 0) {
#pragma unroll
    for (int k = 0; k < LANES; ++k) l_tot += xl[k * BM] * fast_exp2((xm[k * BM] - m_use) * c);
    row_pair(l_tot > 0.f ? 1.0f / l_tot : 0.f, fn);
  }
  if (kl == 0 && lane < 32 && w0 + lane < d.nq) {
    const int r = w0 + lane;
    const int64_t row = GRID && norm ? (int64_t)head * g.b.side * d.nq + grid_token(g.b, d.nq, row_blk, r) : (int64_t)head * d.nq + r;
    if (norm) m_out[row] = l_tot > 0.f ? m_new * d.scale + logf(l_tot) : -INFINITY;
    else {
      m_out[row] = m_new * d.scale;                // -inf stays -inf (scale > 0)
      l_out[row] = l_tot;
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float a = f[q] * fast_exp2((m_row[q] - use[q]) * c);
    // Every wavefront leaves its pieces of four columns, [wavefront][piece][lane], and adds up and stores 16 / LANES of its
    // row group's.
#pragma unroll
    for (int t = 0; t < HT; ++t)
      x[(wave * 16 + 2 * t + q) * 64 + lane] = f32x4{o[t][q][0] * a, o[t][q][1] * a, o[t][q][2] * a, o[t][q][3] * a};
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16 / LANES; ++i) {
    const int piece = kl + LANES * i, q = piece & 1, col = 16 * (piece >> 1) + 4 * grp, r = q_row + 16 * q;   // (LANES is even)
    if (piece >= 2 * HT || r >= d.nq) continue;
    f32x4 v = x[(rg * 16 + piece) * 64 + lane];
#pragma unroll
    for (int k = 1; k < LANES; ++k) {
      const f32x4 w = x[((k * RG + rg) * 16 + piece) * 64 + lane];
      v[0] += w[0]; v[1] += w[1]; v[2] += w[2]; v[3] += w[3];
    }
    const int64_t o_at = GRID && norm ? head * d.lo.head + row_blk * g.b.o + r * d.lo.row : ((int64_t)head * d.nq + r) * H;
    if (norm) {
      const float by = q ? fn[1] : fn[0];
      bf16x4 b;
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = (bf16_t)(v[e] * by);
      *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(O_part) + o_at + col) = b;
    } else {
      *reinterpret_cast<f32x4*>(O_part + o_at + col) = v;
    }
  }
}

template <int HR, int RG, int GRID>
hipError_t go(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
              float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  if (ph == PREPARE) return ensure_dynamic_lds(reinterpret_cast<const void*>(fwd_small_kernel<HR, RG, GRID>), lds_bytes(RG, padded_head(HR)));
  const dim3 grid(xcd_grid(d.heads / g.group * g.parts, (GRID ? g.b.side : 1) * g.group * ((d.nq + 32 * RG - 1) / (32 * RG))));
  A2D_LAUNCH((fwd_small_kernel<HR, RG, GRID>), grid, dim3(64 * WAVES), lds_bytes(RG, padded_head(HR)), s, d, g, (const bf16_t*)Q,
             (const bf16_t*)K, (const bf16_t*)V, O_part, m, l, in);
  return hipGetLastError();
}
template <int RG, int GRID>
hipError_t go_h(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  switch (d.hdim) {
    case 128: return go<128, RG, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s);
    case 96: return go<96, RG, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s);
    case 80: return go<80, RG, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s);
    default: return go<64, RG, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s);
  }
}
template <int RG>
hipError_t go_rows(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                   float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  return g.b.side == 0 ? go_h<RG, 0>(ph, d, g, Q, K, V, O_part, m, l, in, s)
         : g.b.cyclic  ? go_h<RG, 2>(ph, d, g, Q, K, V, O_part, m, l, in, s)
                       : go_h<RG, 1>(ph, d, g, Q, K, V, O_part, m, l, in, s);
}

}  // namespace

hipError_t launch_fwd_small(Phase ph, int rows, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                            const void* V, float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  return rows == 64 ? go_rows<2>(ph, d, g, Q, K, V, O_part, m, l, in, s) : go_rows<1>(ph, d, g, Q, K, V, O_part, m, l, in, s);
}

}  // namespace a2d
