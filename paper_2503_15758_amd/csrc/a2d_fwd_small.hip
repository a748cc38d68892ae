// bf16 MFMA forward tile kernel for short calls: the contractions of a2d_fwd_mfma.hip, 32 or 64 query rows per workgroup.
//
// A call of few query rows leaves most of the chip without work when its blocks are 128 rows, and sharing their
// walks between workgroups costs partial results in memory and a launch that merges them.  Here the eight
// wavefronts of a workgroup hold the SAME 32 rows and take every eighth slab of 32 keys; their (N, m, l) are
// merged through LDS at the end.  Nothing is shared during the walk of 32 rows, so there is no barrier in it: each wavefront
// stages its slabs in a piece of LDS of its own.  (K read straight into the A operands, a lane a row, goes 32 lines at a
// time through an L1 that eight wavefronts share: 13.5 us became 16.4 at 8 x 1024 x 1024, H = 128.)
// What bounds it: launch, argument and first-load latencies below two rounds of slabs; then what a compute unit reads
// from L2, 128 KiB a round at H = 128 (1.65 us; its MFMAs take 0.45), since every 32 rows read all keys they see.  For
// short calls that is cheaper than partial results and a second launch, for long ones not (see plan_fwd_mfma).
// Where 32-row blocks no longer run at once, 64 rows in four lanes of two wavefronts that stage their slabs together read half
// as much and need a barrier a round (1.37 us for 128 keys): H = 128 16 x 1024 x 1024 22.4 -> 18.7 us, 8 x 2048 x 2048 36.3 ->
// 29.2, 16 x 1500 x 1500 causal 32.1 -> 24.9; H = 64 32 x 512 x 512 11.6 -> 8.9.
// Measured, against the best of the other forms: H = 128 2 x 512 x 512 causal 15.4 -> 9.3 us, 8 x 1024 x 1024 23.0 -> 12.8,
// 4 x 2048 x 2048 26.5 -> 20; H = 64 2 x 512 x 512 10.8 -> 6.3, 8 x 1024 x 1024 16.6 -> 8.6.
#include "a2d_mfma.hpp"

namespace a2d {
namespace {

using namespace mfma;

constexpr int SB = 32, WAVES = 8;                  // keys of a slab, wavefronts
// LDS: eight { K slab, V slab } (rows as in a2d_fwd_mfma.hip) | m, l of every wavefront's rows
constexpr int KLD = 272, VLD = 320, V_AT = SB * KLD, SLAB_BYTES = SB * (KLD + VLD);
constexpr int STAT = WAVES * SLAB_BYTES;
constexpr int LDS_BYTES = STAT + 2 * WAVES * SB * 4;
constexpr float kRescaleThreshold = 8.0f;          // log2 units
static_assert(WAVES * 16 * 1024 <= STAT, "the pieces of four column tiles must fit the slabs");

// RG: groups of 32 rows.  1: eight key lanes, each wavefront its own slab.  2: 64 rows and four lanes of two wavefronts that
// stage a slab together, two buffers each: half the reads from L2, a barrier a round.
// (GRID, arguments and outputs as of fwd_mfma_kernel)
template <int HR, int RG, int GRID>
__global__ __launch_bounds__(64 * WAVES, 1) void fwd_small_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, float* O_part, float* m_out, float* l_out, FwdInput in) {
  constexpr int HD = padded_head(HR), H = HR, KS = (HR + 15) / 16, CT = HD / 32;
  constexpr bool PLAIN = GRID == 0, CYCLIC = GRID == 2;
  warm_arguments<9 * 8>();
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  constexpr int LANES = WAVES / RG, BM = 32 * RG;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kl = wave / RG, rg = wave % RG;        // key lane, row group
  const int half = lane >> 5, l32 = lane & 31;

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

  // ---- Q^T fragments; rows beyond nq re-read the last row
  const int q_row = w0 + l32, q_ld = min(q_row, d.nq - 1);
  bf16x8 qf[KS];
  {
    const bf16_t* qp = Q + (int64_t)q_ld * d.lq.row + 8 * half;
#pragma unroll
    for (int x = 0; x < KS; ++x) qf[x] = *reinterpret_cast<const bf16x8*>(qp + 16 * x);
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
  int nfull = 0, nvis = 0, my_vis = 0;             // keys of the current sub-block that all rows see, some row, the lane's
  auto enter_segment = [&]() {
    nfull = vis_count(min(w0, d.nq - 1));
    if (RG > 1) nvis = vis_count(min(w0 + 31, d.nq - 1));
    my_vis = vis_count(q_ld);
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

  // ---- staging: a lane moves one 16-byte chunk of ST_N rows (64 columns: eight lanes a row, else sixteen; chunks past
  // the head size: its last one once more, into columns whose results are not stored).  Rows beyond the sub-block
  // re-read its last one.
  constexpr int CHUNKS = HD == 64 ? 8 : 16, ST_ROWS = 64 / CHUNKS, ST_N = SB / ST_ROWS / RG;
  const unsigned k_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lk.row * 2);
  const unsigned v_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lv.row * 2);
  const unsigned k_col_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.k * 2)) : k_row_bytes;
  const unsigned v_col_bytes = CYCLIC ? __builtin_amdgcn_readfirstlane((unsigned)(g.b.v * 2)) : v_row_bytes;
  const int st_row = lane / CHUNKS + rg * (SB / RG), st_chunk = lane % CHUNKS;
  u32x4 kreg[ST_N], vreg[ST_N];
  auto load = [&](int s, int j) {
    if (CYCLIC) start = s;
    const gptr_t ka = uniform_gptr(reinterpret_cast<const char*>(K) + (start * k_col_bytes + (unsigned)(j * SB) * k_row_bytes));
    const gptr_t va = uniform_gptr(reinterpret_cast<const char*>(V) + (start * v_col_bytes + (unsigned)(j * SB) * v_row_bytes));
    const int chunk = min(st_chunk, H / 8 - 1);
#pragma unroll
    for (int p = 0; p < ST_N; ++p)
      kreg[p] = gload_b128(ka, __umul24((unsigned)min(st_row + ST_ROWS * p, rows - 1 - j * SB), k_row_bytes) + 16 * chunk);
#pragma unroll
    for (int p = 0; p < ST_N; ++p)
      vreg[p] = gload_b128(va, __umul24((unsigned)min(st_row + ST_ROWS * p, rows - 1 - j * SB), v_row_bytes) + 16 * chunk);
  };
  const unsigned slab = lds_base + kl * RG * SLAB_BYTES;     // (RG > 1: the first of two)
  const unsigned k_wr = slab + st_row * KLD + 16 * st_chunk, v_wr = slab + V_AT + st_row * VLD + 16 * st_chunk;
  auto store = [&](unsigned buf) {
#pragma unroll
    for (int p = 0; p < ST_N; ++p)
      *reinterpret_cast<__attribute__((address_space(3))) u32x4*>((uintptr_t)(k_wr + buf + ST_ROWS * p * KLD)) = kreg[p];
#pragma unroll
    for (int p = 0; p < ST_N; ++p)
      *reinterpret_cast<__attribute__((address_space(3))) u32x4*>((uintptr_t)(v_wr + buf + ST_ROWS * p * VLD)) = vreg[p];
  };
  const int g16 = lane >> 4, j16 = lane & 15;
  const unsigned k_rd = slab + l32 * KLD + 16 * half;
  const unsigned v_rd = slab + V_AT + (4 * (g16 >> 1) + (j16 >> 2)) * VLD + (16 * (g16 & 1) + 4 * (j16 & 3)) * 2;

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
    load(sb, j);
    enter_segment();
  }

  f32x16 o[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) o[t] = zero16();
  float m_lane = -INFINITY, m_ref = -INFINITY, l_run = 0.f;
  if (!GRID && g.acc && part == 0 && kl == 0) {
    // the first wavefront continues the stored partial (rows past nq: the last row's, never stored)
    const int64_t row = (int64_t)head * d.nq + q_ld;
    m_lane = m_ref = in.m[row] / d.scale;
    l_run = half == 0 ? in.l[row] : 0.f;
    const float* np = in.N + row * H + 4 * half;
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (32 * t + 8 * q + 4 * half >= H) continue;
        const f32x4 v = *reinterpret_cast<const f32x4*>(np + 32 * t + 8 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[t][4 * q + e] = v[e];
      }
  }

  auto compute = [&](unsigned buf) {
    const unsigned k_at = k_rd + buf, v_at = v_rd + buf;
    const int k0 = j * SB + (CYCLIC && sb > shift_from);
    if (RG > 1 && k0 >= nvis) return;
    f32x16 s = zero16();
#pragma unroll
    for (int x = 0; x < KS; ++x) s = mma(lds_load_b128(k_at + 32 * x), qf[x], s);
    if (k0 + SB > nfull) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (k0 + 8 * (r >> 2) + 4 * half + (r & 3) >= my_vis) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    m_lane = fmaxf(m_lane, mx);
    if (__builtin_amdgcn_ballot_w64((m_lane - m_ref) * c > kRescaleThreshold) != 0) {
      asm volatile("" ::: "memory");               // (a real branch, as in fwd_block)
      const float m_row = fmaxf(m_lane, __shfl_xor(m_lane, 32, 64));
      const float m_use = (m_row == -INFINITY) ? 0.f : m_row;
      const float alpha = fast_exp2((m_ref - m_use) * c);
      m_ref = m_row;
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
    }
    const float mc = (m_ref == -INFINITY) ? 0.f : m_ref * c;
    float psum = 0.f;
    bf16x8 pb[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = fast_exp2(fmaf(s[r], c, -mc));
      psum += p;
      pb[r >> 3][r & 7] = (bf16_t)p;
    }
    l_run += psum;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        const unsigned at = v_at + 16 * u * VLD + 64 * t;
        o[t] = mma(lds_load_tr(at, at + 8 * VLD), pb[u], o[t]);
      }
  };
  if constexpr (RG == 1) {
    while (sb < segs) {
      int nsb = sb, nj = j, nn = n;
      advance(stride, nsb, nj, nn);
      store(0);
      if (nsb < segs) load(nsb, nj);               // the next slab
      compute(0);
      if (!CYCLIC && nsb != sb && nsb < segs) enter_segment();
      sb = nsb; j = nj; n = nn;
    }
  } else {
    if (sb < segs) store(0);
    __syncthreads();
    unsigned buf = 0;
    for (int r = 0; r < rounds; ++r) {
      int nsb = sb, nj = j, nn = n;
      advance(stride, nsb, nj, nn);
      const bool more = nsb < segs;
      if (more) load(nsb, nj);
      if (sb < segs) compute(buf);
      if (more) store(SLAB_BYTES - buf);
      __syncthreads();
      if (!CYCLIC && more && nsb != sb) enter_segment();
      sb = nsb; j = nj; n = nn;
      buf = SLAB_BYTES - buf;
    }
  }

  // ---- the wavefronts' (N, m, l) become one, as partials of one query block do (Alg. 2)
  const float m_row = fmaxf(m_lane, __shfl_xor(m_lane, 32, 64));
  const float f = (m_row == -INFINITY) ? 0.f : fast_exp2((m_ref - m_row) * c);
  const float l_row = (l_run + __shfl_xor(l_run, 32, 64)) * f;
  float* const xm = reinterpret_cast<float*>(lds + STAT) + rg * 32 + l32;
  float* const xl = xm + WAVES * 32;
  if (half == 0) {
    xm[kl * BM] = m_row;
    xl[kl * BM] = l_row;
  }
  __syncthreads();
  float mk[LANES], lk[LANES], m_new = -INFINITY;
#pragma unroll
  for (int k = 0; k < LANES; ++k) {
    mk[k] = xm[k * BM];
    lk[k] = xl[k * BM];
    m_new = fmaxf(m_new, mk[k]);
  }
  const float m_use = m_new == -INFINITY ? 0.f : m_new;      // (2^-inf = 0 for the wavefronts that saw nothing)
  float l_tot = 0.f;
#pragma unroll
  for (int k = 0; k < LANES; ++k) l_tot += lk[k] * fast_exp2((mk[k] - m_use) * c);
  const float a = f * fast_exp2((m_row - m_use) * c);
  const bool norm = g.norm != 0, ok = q_row < d.nq;
  const int64_t row = GRID && norm ? (int64_t)head * g.b.side * d.nq + grid_token(g.b, d.nq, row_blk, q_row)
                                   : (int64_t)head * d.nq + q_row;
  const int64_t o_at = GRID && norm ? head * d.lo.head + row_blk * g.b.o + q_row * d.lo.row : row * H;
  if (kl == 0 && half == 0 && ok) {
    if (norm) m_out[row] = l_tot > 0.f ? m_new * d.scale + logf(l_tot) : -INFINITY;
    else {
      m_out[row] = m_new * d.scale;                // -inf stays -inf (scale > 0)
      l_out[row] = l_tot;
    }
  }
  // Every wavefront leaves its pieces of four columns, [wavefront][piece][lane], and adds up and stores 16 / LANES of its
  // row group's.
  f32x4* const x = reinterpret_cast<f32x4*>(lds);
  const float fn = l_tot > 0.f ? 1.0f / l_tot : 0.f;
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      x[(wave * 16 + t * 4 + q) * 64 + lane] = f32x4{o[t][4 * q] * a, o[t][4 * q + 1] * a, o[t][4 * q + 2] * a, o[t][4 * q + 3] * a};
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16 / LANES; ++i) {
    const int piece = kl + LANES * i, col = 32 * (piece >> 2) + 8 * (piece & 3) + 4 * half;
    if (piece >= 4 * CT || col >= H || !ok) continue;
    f32x4 v = x[(rg * 16 + piece) * 64 + lane];
#pragma unroll
    for (int k = 1; k < LANES; ++k) {
      const f32x4 w = x[((k * RG + rg) * 16 + piece) * 64 + lane];
      v[0] += w[0]; v[1] += w[1]; v[2] += w[2]; v[3] += w[3];
    }
    if (norm) {
      bf16x4 b;
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = (bf16_t)(v[e] * fn);
      *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(O_part) + o_at + col) = b;
    } else {
      *reinterpret_cast<f32x4*>(O_part + o_at + col) = v;
    }
  }
}

template <int HR, int RG, int GRID>
hipError_t go(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
              float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  if (ph == PREPARE) return ensure_dynamic_lds(reinterpret_cast<const void*>(fwd_small_kernel<HR, RG, GRID>), LDS_BYTES);
  const dim3 grid(xcd_grid(d.heads / g.group * g.parts, (GRID ? g.b.side : 1) * g.group * ((d.nq + 32 * RG - 1) / (32 * RG))));
  A2D_LAUNCH((fwd_small_kernel<HR, RG, GRID>), grid, dim3(64 * WAVES), LDS_BYTES, s, d, g, (const bf16_t*)Q,
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
