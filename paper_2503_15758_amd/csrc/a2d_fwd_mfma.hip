// bf16 MFMA forward tile kernel for H = 128, 96, 80 and 64 (Sec. 3.1, Eq. (3), evaluated block by
// block with the recurrence of Sec. 2.2).
//
// Work split: one workgroup = 8 wavefronts = 256 query rows of one head; each
// wavefront owns 32 query rows for the whole kernel and walks the key blocks
// (64 keys per step) that the workgroup stages through LDS.  (Tiles with too few
// query blocks for that take 128-row workgroups: see the kernel's template parameters.)
//
// Both contractions are issued TRANSPOSED so that no cross-lane data movement is
// needed between them (v_mfma_f32_16x16x32_bf16, D = A * B, A: 16 x 32, B: 32 x 16):
//   S^T = K * Q^T : A = K fragment (LDS, 128-bit reads), B = Q^T fragment (registers,
//                   loaded once).  In D a lane holds 4 keys of ONE query column per tile, so
//                   row max / row sum are in-lane reductions; the four lanes of a row
//                   (16 apart) are combined only when needed.
//   O^T += V^T * P^T : B = P^T is the D layout of two tiles of S^T (the contraction index
//                   may be permuted freely as long as A uses the same permutation),
//                   A = V^T fragment read from the row-major V tile with the LDS
//                   transpose read ds_read_b64_tr_b16.
// Large tiles are held by the chip's power (1.4 kW at 1.8-1.9 GHz), so it is the energy of a flop that counts: an MFMA of
// 16 x 16 x 32 moves half the accumulators per flop of one of 32 x 32 x 16 (787 -> 763 us at 96 x 4096 x 4096, H = 128).
// LDS: K and V tiles double-buffered, loaded straight into LDS (dma_b128) in blocks whose chunks are placed so that the
// 128-bit K reads and the transposing V reads are bank-conflict free (Blocks16).  Through registers, written to
// LDS by all wavefronts in front of a step's barrier, tiles cost a step 5-10 %.  The two together, H = 128: 96 x 4096 x 4096
// 780 -> 725 us (1137 TFLOP/s), causal 444 -> 410, 8 x 16384 x 16384 1034 -> 940, 16 x 2048 x 2048 41.9 -> 39.5; 64 x 4096 x 4096, H =
// 96 / 80 / 64 425 / 398 / 343 -> 389 / 370 / 312.  One workgroup of eight wavefronts has a compute unit with two wavefronts
// per SIMD, so one's MFMAs overlap the other's softmax arithmetic, and every staged K / V tile serves all eight (two
// workgroups of four would stage each tile twice).  The mask is a branch around its selects inside the one copy of the
// block: with a copy of its own per kind of block the compiler moved the accumulators between registers.
//
// The two wavefronts of a SIMD (w and w + 4) start a step with the scores, so that both want the matrix unit, then both the vector
// ALU.  PHASED (H = 128) keeps them in opposite phases: in the interval between two barriers one goes through the MFMAs of a step (scores of block
// t + 1, products of block t) and then the softmax of block t + 1, the other through the softmax of block t and then the same MFMAs.  In turn on one
// GPU, 96 x 4096 x 4096 / 32 x 16384 x 16384: 6.6 / 7.3 % fewer cycles (matrix unit busy 52 -> 56 / 56 -> 61 % of them) at a 3.5 / 2.4 % lower clock
// (the same power), 852 -> 824 / 3670 -> 3490 us.  From both, a step takes 3285 cycles (3550 in order) and a workgroup 25000 besides; what bounds a
// step is that an MFMA of 16 cycles leaves the other wavefront two vector instructions, not three, so that the 128 MFMAs and two softmaxes take 2730 at
// the least (both measured side by side).  Peaky logits, whose rows move their references often, lengthen the softmax alone: 8 x 16384 x 16384, sigma 4
// 2 % fewer cycles, and shorter walks are slower than in order (plan_fwd_mfma).
// Rescaling is lazy: a row's exponent reference m_ref follows its running maximum
// only when a score exceeds it by more than 2^8 (in the exponent's units) - a rare,
// wave-uniform branch, and the only place where the lanes of a row talk to each
// other.  Each lane tracks the true maximum of its own scores; at the end they
// are combined and N, l are brought to the true row maximum, so (N, m, l) leave the
// kernel exactly as Eq. (3) defines them.
#include "a2d_mfma.hpp"

namespace a2d {
namespace {

using namespace mfma;

constexpr int BN = 64;             // keys per step
__host__ __device__ constexpr int buf_bytes(int hd) { return 2 * BN * 2 * hd; }   // { K tile, V tile }, in blocks
__host__ __device__ constexpr int lds_bytes(int hd) { return 2 * buf_bytes(hd); }          // of a key lane
// of a launch: 16 rows of every wavefront come in (accumulating calls) and go out at a time
__host__ __device__ constexpr int fwd_lds(int waves, int hd, int kl) {
  const int tiles = kl * lds_bytes(hd), rows = waves / kl * acc_area(hd / 16);
  return tiles > rows ? tiles : rows;
}
// log2 units.  (Peaky rows move their references often: at 32, 8 x 16384 x 16384, sigma 4 917 -> 874 us.  But a probability of 1, which the
// maximum has where its row's reference has just moved, is rounded to itself, and such rows consist of little else: their results
// were ten times as far off, 5e-4 of O instead of 3e-5.)
constexpr float kRescaleThreshold = 8.0f;
// The plan's costs in us, of tiles (the fit below) and of calls over a grid, whose walks of every length make them wait for each
// other.  Grids: a fit to 2000 of 1 to 280 heads, 8 to 2048 rows a column, 1 to 8 columns, both layouts, causal and not: 1.2 % off the
// best form and parts in the mean, 2.2 % with the costs of earlier kernels.  Of 3000 others of 1 to 16 heads 232 go out otherwise, 1.07
// times as fast in the mean (9 heads, 544 x 4 tokens, H = 80, causal 31.5 -> 22.2 us, from two key lanes and parts to 64 rows; a seventh
// of them slower by 3 % or more, at worst 10/5 heads, 1095 x 3, H = 80 64.4 -> 72.8).  Three values: H = 64 / 80, 96 / 128.
struct FwdCosts {
  double step[3];                     // a 64-key step of a 256-row workgroup; ...
  double lanes, alone, pair[3];       // ... as multiples of it, one of 128 rows in two key lanes, in four wavefronts, in two such side by side
  double fixed, lanes_more, alone_more;   // the rest of a workgroup of 256 rows, and what the others' takes beyond
  double big_more;                    // of 256 rows
  double big_store, lanes_store;      // more of a chip with several turns, H = 128
  double pair_fixed, pair_store;      // of a pair, where pairs follow one another; by H / 128
  double round32[3], fixed32[3];      // a round of 256 keys of 32 rows, of 128 keys of 64 rows
  double round64[3], fixed64[3];
  double merge, merge_few;            // a merge of parts: of forms of many rows, of few
  double tail;
};
constexpr FwdCosts kFwdCosts[2] = {
    {{1.099, 1.449, 1.586}, 1.13, 0.657, {0.994, 1.04, 1.086}, 3.899, 0.549, 0.64, 0, 4.97, 1.82, 1.67, 4.83,
     {0.907, 1.211, 1.609}, {3.5, 3.39, 2.95}, {0.891, 1.288, 1.398}, {3.85, 3.78, 4.22}, 4.42, 4.65, 0.46},
    {{1.314, 1.34, 1.62}, 1.138, 0.707, {1.033, 1.033, 1.033}, 4.06, 1.15, 0.19, 1.77, 0, 0, 0, 0,
     {1.015, 1.119, 1.405}, {3.13, 3.84, 3.97}, {0.888, 1.125, 1.315}, {4.48, 4.18, 4.66}, 3.55, 4.66, 0.141}};

template <int HR>
struct FwdState {
  f32x4 o[HR / 16][2];   // column tiles x the wavefront's two tiles of 16 query rows
  // of the lane's row in each tile:
  float m_lane[2];       // true running max of this lane's raw dot products
  float m_ref[2];        // reference the exponentials are taken against (raw units, same in the four lanes of a row)
  float l_run[2];        // this lane's share of the row sum, relative to m_ref
};

// A 64-key block for one wavefront, in three pieces; at: its buffer's offset from the addresses in rd.  S^T in tiles of 16 keys (k) x 16
// queries (q): lane = query, registers = keys 16 k + 4 grp + 0..3; the registers of two key tiles are the eight contraction indices of a
// lane in O^T += V^T P^T.
// Fragments of K and V go through rings four deep: each is requested four slots of two MFMAs before its use (the scheduling fences
// keep the compiler from sinking the requests back to their uses), the first ones before the piece that uses them.
using Scores = f32x4[4][2];
using Ring = bf16x8[4];
template <int HR, int I>                           // slot I of the scores: key tile I & 3, slice I >> 2 of H, both query tiles
__device__ __forceinline__ void fwd_key(Ring& kr, const Blocks16& rd, unsigned at) {
  kr[I & 3] = lds_load_b128(rd.nat + at + ((I & 3) * (padded_head(HR) / 32) + (I >> 2)) * BLOCK);
}
template <int HR, int I>                           // step I of the products: 32-key group I / HT, column tile I % HT
__device__ __forceinline__ void fwd_value(Ring& vr, const Blocks16& rd, unsigned at) {
  constexpr int KS = padded_head(HR) / 32, HT = HR / 16, K_BYTES = buf_bytes(padded_head(HR)) / 2;
  const unsigned a = (I % HT & 1 ? rd.tr_o : rd.tr_e) + at + K_BYTES + ((I / HT) * 2 * KS + (I % HT >> 1)) * BLOCK;
  vr[I & 3] = lds_load_tr(a, a + KS * BLOCK);
}
template <int HR>
__device__ __forceinline__ void fwd_first_keys(Ring& kr, const Blocks16& rd, unsigned at) {
  static_for<0, 4>([&](auto I) { fwd_key<HR, decltype(I)::value>(kr, rd, at); });
  __builtin_amdgcn_sched_barrier(0);
}
template <int HR>
__device__ __forceinline__ void fwd_first_values(Ring& vr, const Blocks16& rd, unsigned at) {
  static_for<0, 4>([&](auto I) { fwd_value<HR, decltype(I)::value>(vr, rd, at); });
  __builtin_amdgcn_sched_barrier(0);
}

template <int HR>
__device__ __forceinline__ void fwd_scores(Scores& s, Ring& kr, const bf16x8 (&qf)[padded_head(HR) / 32][2], const Blocks16& rd, unsigned at) {
  constexpr int KS = padded_head(HR) / 32;
#pragma unroll
  for (int k = 0; k < 4; ++k) s[k][0] = s[k][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  static_for<0, 4 * KS>([&](auto I) {
    constexpr int i = decltype(I)::value;
#pragma unroll
    for (int q = 0; q < 2; ++q) s[i & 3][q] = mma16(kr[i & 3], qf[i >> 2][q], s[i & 3][q]);
    if constexpr (i + 4 < 4 * KS) fwd_key<HR, i + 4>(kr, rd, at);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// masked: some of the wavefront's rows do not see all of the block's keys
// (values: called in front of the exponentials)
template <int HR, class F>
__device__ __forceinline__ void fwd_softmax(FwdState<HR>& st, Scores& s, bf16x8 (&pb)[2][2], bool masked, int k0,
                                            const int (&my_vis)[2], int grp, float c, F&& values) {
  constexpr int HT = HR / 16;
  if (A2D_SELDOM(masked)) {
    asm volatile("" ::: "memory");   // keep this a branch
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + 16 * (r >> 2) + 4 * grp + (r & 3);
        // (a select: of stores under conditions that imply each other the compiler made a chain that keeps all of them in scalar
        // registers, 1 to 4 % of a walk of few steps: gathered 15/5 x 3479 x 148, H = 64 14.1 -> 13.3 us, 60 x 3832 x 133, H = 128 78.7 -> 75.3)
        s[r >> 2][q][r & 3] = key >= my_vis[q] ? -INFINITY : s[r >> 2][q][r & 3];
      }
  }
  bool grow = false;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float mx = st.m_lane[q];
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r >> 2][q][r & 3]);
    st.m_lane[q] = mx;
    // (m_lane - m_ref) is +inf on the first visible block, NaN (-> false) while nothing is visible
    grow |= (mx - st.m_ref[q]) * c > kRescaleThreshold;
  }
  if (A2D_SELDOM(__builtin_amdgcn_ballot_w64(grow) != 0)) {
    asm volatile("" ::: "memory");   // keep this a real (rarely taken) branch: no if-conversion
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float m_row = row_max(st.m_lane[q]);
      const float m_use = (m_row == -INFINITY) ? 0.f : m_row;
      const float alpha = fast_exp2((st.m_ref[q] - m_use) * c);    // m_ref = -inf gives 0
      st.m_ref[q] = m_row;
      st.l_run[q] *= alpha;
#pragma unroll
      for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) st.o[t][q][r] *= alpha;
    }
  }
  values();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float mc = (st.m_ref[q] == -INFINITY) ? 0.f : st.m_ref[q] * c;
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = fast_exp2(fmaf(s[r >> 2][q][r & 3], c, -mc));
      psum += p;
      pb[r >> 3][q][r & 7] = (bf16_t)p;
    }
    st.l_run[q] += psum;
  }
  __builtin_amdgcn_sched_barrier(0);
}

// O^T += V^T P^T
template <int HR>
__device__ __forceinline__ void fwd_products(FwdState<HR>& st, const bf16x8 (&pb)[2][2], Ring& vr, const Blocks16& rd, unsigned at) {
  constexpr int HT = HR / 16;
  static_for<0, 2 * HT>([&](auto I) {
    constexpr int i = decltype(I)::value;
#pragma unroll
    for (int q = 0; q < 2; ++q) st.o[i % HT][q] = mma16(vr[i & 3], pb[i / HT][q], st.o[i % HT][q]);
    if constexpr (i + 4 < 2 * HT) fwd_value<HR, i + 4>(vr, rd, at);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// the three in order
template <int HR>
__device__ __forceinline__ void fwd_block(FwdState<HR>& st, const bf16x8 (&qf)[padded_head(HR) / 32][2], const Blocks16& rd, unsigned at,
                                          bool masked, int k0, const int (&my_vis)[2], int grp, float c) {
  Scores s;
  Ring kr, vr;
  bf16x8 pb[2][2];
  fwd_first_keys<HR>(kr, rd, at);
  fwd_scores<HR>(s, kr, qf, rd, at);
  fwd_softmax<HR>(st, s, pb, masked, k0, my_vis, grp, c, [&]() { fwd_first_values<HR>(vr, rd, at); });
  fwd_products<HR>(st, pb, vr, rd, at);
}

// WAVES wavefronts per workgroup, in KL key lanes of WAVES / KL wavefronts (32 query rows each):
//   <8, 1>  256 rows: one workgroup fills a compute unit;
//   <4, 1>  128 rows, two workgroups per compute unit: when there are too few 256-row blocks to
//           give every compute unit one;
//   <8, 2>  128 rows walked by two key lanes: when even the 128-row blocks come to at most one per
//           compute unit, so that a SIMD still holds two wavefronts.  The lanes take alternate key
//           blocks of the walk, each staging its own tiles into its own pair of LDS buffers, and
//           their (N, m, l) are merged through LDS at the end exactly as two partials of one
//           query block are (Alg. 2).
// PHASED: see above; of two key lanes one is behind the other.
// HR: head size = row length in memory (64, 80, 96 or 128); the LDS tiles and fragments are laid out
// for the padded head size HD = padded_head(HR) (64, 96 or 128).
// (O_part, m_out and l_out are not __restrict__: an accumulating call's `in` is the same memory)
// GRID: all query blocks of an emulated grid (g.b; 1: contiguous blocks, 2: cyclic ones).  A workgroup walks the
// tiles of its whole grid row, so that AttnFix over the row happens in its registers, and writes rows of O and lse of
// the sequence (or, of a split walk, a partial of them: [part][row block][head][row]).  The tiles of a row of
// contiguous blocks are one run of keys.  Of cyclic ones, block j of every column comes before block j + 1 of any:
// the workgroups of a head, which see different numbers of keys, then read the same part of the sequence at a time.
template <int WAVES, int HR, int KL, int GRID, bool PHASED>
__global__ __launch_bounds__(64 * WAVES, 8 / WAVES) void fwd_mfma_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, float* O_part, float* m_out, float* l_out, FwdInput in) {
  constexpr int RW = WAVES / KL;          // wavefronts of one key lane
  constexpr int BM = 32 * RW;             // query rows per workgroup
  constexpr int kThreads = 64 * RW;       // threads of one key lane (they stage its tiles)
  constexpr int HD = padded_head(HR), H = HR;
  constexpr int KS = HD / 32, HT = HR / 16, BUF_BYTES = buf_bytes(HD);
  constexpr int kLdsBytes = lds_bytes(HD);
  if constexpr (GRID) warm_arguments<9 * 8>();
  extern __shared__ __attribute__((aligned(16))) char lds_all[];
  // per key lane: [buf]{ K tile, V tile }
  const int kl = KL == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads);   // key lane of this wavefront
  char* const lds = lds_all + kl * kLdsBytes;
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

  const int nqb = (d.nq + BM - 1) / BM;
  // (the query blocks of the query heads that share a key/value head are placed as one unit)
  int unit, blk;
  const int by_size = GRID ? d.causal : g.by_size;
  if (!xcd_map(blockIdx.x, d.heads / g.group * g.parts, (GRID ? g.b.side : 1) * g.group * nqb, by_size != 0, unit, blk,
               kXcdCus * 8 / WAVES)) return;
  // (unit = part `part` of the walks over one key/value head; blocks numbered by size first when the
  // workgroups are ordered by size)
  const Split up = split_by(unit, g.parts);
  const int kvh = up.q, part = up.r;
  const Split in_group = query_head(blk, g.group, nqb, GRID || by_size);
  const int head = kvh * g.group + in_group.r;
  blk = in_group.q;
  const GridBlock gb = GRID ? grid_block(g.b, nqb, blk) : GridBlock{0, blk};
  const int row_blk = gb.r;                             // of the grid
  blk = gb.blk;
  // heavy (late) query blocks first: under a causal mask they walk more key blocks
  const int q0 = (nqb - 1 - blk) * BM;
  const int tid = (int)threadIdx.x - kl * kThreads;     // within the key lane
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int grp = lane >> 4;
  Q += (int64_t)head * d.lq.head + (GRID ? row_blk * g.b.q : 0);
  K += (int64_t)kvh * d.lk.head;
  V += (int64_t)kvh * d.lv.head;
  if (!GRID || !g.norm) {
    const int64_t slot = ((int64_t)part * (GRID ? g.b.side : 1) + row_blk) * d.heads * d.nq;
    O_part += slot * HR;
    m_out += slot;
    l_out += slot;
  }

  // ---- Q^T fragments: lane holds query row (lane & 15) of two tiles, h = 32*step + 8*grp + 0..7.
  // Rows beyond nq re-read the last row (their results are never stored); columns past the head size are zero.
  const int q_row = q0 + wave * 32 + (lane & 15);       // of the first tile
  bf16x8 qf[KS][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bf16_t* qp = Q + (int64_t)min(q_row + 16 * q, d.nq - 1) * d.lq.row;
#pragma unroll
    for (int x = 0; x < KS; ++x) {
      const int at = 32 * x + 8 * grp;
      qf[x][q] = *reinterpret_cast<const bf16x8*>(qp + min(at, H - 8));
      if (32 * x + 32 > H && at >= H) qf[x][q] = bf16x8{};
    }
  }
  FwdState<HR> st;
#pragma unroll
  for (int t = 0; t < HT; ++t) st.o[t][0] = st.o[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  st.l_run[0] = st.l_run[1] = 0.f;
  const float c = d.scale * kLog2e;
  float m_in[2] = {-INFINITY, -INFINITY};
  if (!GRID && g.acc && part == 0) {
    // (key lane 0 of the first part continues the stored partial; the barriers are the whole workgroup's)
    // Continue from the (N, m, l) of `in`: N into the accumulators (same
    // element mapping as the epilogue's stores), m as the exponent reference, l into one of the four
    // lanes of the row.  A lane's share of N is scattered 16-byte pieces of its rows, so the
    // rows come in through LDS: each wavefront reads 16 of its rows at a time with whole-row
    // coalesced loads into a private, padded LDS area and the lanes pick their pieces.
    constexpr int ALD = HD * 4 + 16;                          // padded row stride, bytes
    static_assert(16 * ALD * RW <= fwd_lds(WAVES, HD, KL), "accumulator staging must fit the launch's LDS");
    char* area = lds_all + wave * 16 * ALD;
    const int64_t wrow0 = (int64_t)head * d.nq + q0 + wave * 32;   // first row of the wavefront
    const int64_t last_row = (int64_t)head * d.nq + d.nq - 1;
    // (a lane whose 16-byte piece lies past the row's end re-reads its last piece and stores zeros, or nothing)
    const int col = 4 * (lane & 31), col_ld = min(col, H - 4);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if (KL == 1 || kl == 0) {
        u32x4 t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {                        // two whole rows per load instruction
          const int64_t r = wrow0 + 16 * pass + 2 * i + (lane >> 5);
          t[i] = *reinterpret_cast<const u32x4*>(in.N + (r < last_row ? r : last_row) * H + col_ld);
        }
        if (HD == 128 || col < HD) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            *reinterpret_cast<u32x4*>(area + (2 * i + (lane >> 5)) * ALD + 4 * col) = H == HD || col < H ? t[i] : u32x4{0, 0, 0, 0};
        }
      }
      __syncthreads();
      if (kl == 0) {
        const char* mine = area + (lane & 15) * ALD + 16 * grp;
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) st.o[ht][pass] = *reinterpret_cast<const f32x4*>(mine + 16 * ht * 4);
      }
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (kl != 0) {
        // the other key lane starts from nothing
      } else if (q_row + 16 * q < d.nq) {
        const int64_t row = (int64_t)head * d.nq + q_row + 16 * q;
        m_in[q] = in.m[row];
        st.l_run[q] = grp == 0 ? in.l[row] : 0.f;
      } else {
#pragma unroll
        for (int t = 0; t < HT; ++t) st.o[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};     // rows beyond nq: nothing to continue
      }
    }
  }

  // ---- visibility, per key/value sub-block s: query i sees the first vis_count(i, s) keys of it
  // (key kk of the sub-block iff kk <= i + rel[s])
  auto vis_count = [&](int i, int s) -> int {
    // (cyclic: of a column up to the row block's own; of the others one less, see `shift`)
    if (GRID == 1) return d.causal ? row_blk * d.nq + i + 1 : g.b.side * d.nkv;
    if (GRID == 2) return d.causal ? i + 1 : d.nkv;
    if (!d.causal) return g.seg[s].rows;
    const int64_t v = (int64_t)i + g.seg[s].rel + 1;
    return v <= 0 ? 0 : (v < g.seg[s].rows ? (int)v : g.seg[s].rows);
  };
  const int blk_last = min(q0 + BM, d.nq) - 1;
  const int w_first = min(q0 + wave * 32, d.nq - 1);
  const int w_last = min(q0 + wave * 32 + 31, d.nq - 1);
  // key blocks of sub-block s that some row of the workgroup sees; the walk over (sub-block, block)
  auto seg_blocks = [&](int s) { return (vis_count(blk_last, s) + BN - 1) / BN; };
  int nvis_wave = 0, nfull_wave = 0, my_vis[2] = {0, 0};   // of the current sub-block
  auto enter_segment = [&](int s) {
    nvis_wave = vis_count(w_last, s);        // keys any row of the wave sees
    nfull_wave = vis_count(w_first, s);      // keys every row of the wave sees
#pragma unroll
    for (int q = 0; q < 2; ++q) my_vis[q] = vis_count(min(q_row + 16 * q, d.nq - 1), s);
  };


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
  // (which: bit 0 K, bit 1 V, of those that this wavefront loads)
  auto load_tile = [&](int which, int seg_start, int seg_rows, int j, int boff) {
    const int r = min(ld_row, seg_rows - 1 - j * BN);
#pragma unroll
    for (int x = 0; x < LD_N; ++x) {
      if (which != 3 && !(which >> (ld_first + x) & 1)) continue;
      const gptr_t base = uniform_gptr(ld_base[x] + (seg_start * ld_col_bytes[x] + (unsigned)(j * BN) * ld_row_bytes[x]));
      dma_blocks<KS, H>(lds_base + boff + (4 * (ld_first + x) + ld_tile) * KS * BLOCK, base,
                        __umul24(r, ld_row_bytes[x]) + 16 * ld_chunk, ld_chunk);
    }
  };
  if constexpr (H != HD) {
    // the K tiles' columns past the head size are zero for good (those of V are not read)
    for (int i = tid; i < 2 * BN * (HD - H) / 8; i += kThreads) {
      const int row = i % BN, x = i / BN, buf = x / ((HD - H) / 8), ch = H % 32 / 8 + x % ((HD - H) / 8);
      *reinterpret_cast<u32x4*>(lds + buf * BUF_BYTES + ((row >> 4) * KS + H / 32) * BLOCK + (row & 15) * 64 +
                                16 * (ch ^ block_swap((row & 15) >> 2))) = u32x4{0, 0, 0, 0};
    }
  }
  Blocks16 rd;                                    // fragment reads, buffer 0
  rd.init(lane, lds_base);

  // Walk over the entries (sub-block, key block): lane part * KL + kl of parts * KL takes every
  // (parts * KL)-th entry.  The sub-block table lives in kernel-argument memory, and scalar loads
  // share a wait counter with the LDS reads in flight, so it is only touched when a walk moves to
  // another sub-block; in between its values sit in registers.
  // An entry is (sub-block sb, block j of its nblk); sb == segs: past the end.
  // (cyclic grids: block j of all columns first, see above)
  constexpr bool PLAIN = GRID == 0, CYCLIC = GRID == 2;
  const int stride = KL * g.parts, segs = PLAIN ? g.n : CYCLIC ? __builtin_amdgcn_readfirstlane(g.b.side) : 1;
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
      while (A2D_SELDOM(j >= nblk)) {
        if (sb >= segs) break;
        j -= nblk;
        open_segment(sb + 1, sb, nblk);
      }
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
  int nx_sb = sb, nx_j = j, nx_nblk = nblk;        // the next entry (PHASED)
  int nx_start = 0, nx_rows = 0;                   // start / rows of its sub-block
  auto step_next = [&](int& n_sb, int& n_j, int& n_nblk, int& start, int& rows) {
    const int old = n_sb;
    advance(stride, n_sb, n_j, n_nblk);
    if (CYCLIC) start = n_sb;
    else if (A2D_SELDOM(n_sb != old && n_sb < segs)) { start = seg_start(n_sb); rows = seg_rows(n_sb); }
  };
  if (sb < segs) {
    enter_segment(sb);
    nx_start = seg_start(sb); nx_rows = seg_rows(sb);
    load_tile(3, nx_start, nx_rows, j, 0);
    if constexpr (PHASED) {
      step_next(nx_sb, nx_j, nx_nblk, nx_start, nx_rows);
      if (nx_sb < segs) load_tile(1, nx_start, nx_rows, nx_j, BUF_BYTES);
    }
  }
  // (one wait for the Q rows and the first tiles: the latencies overlap)
  wait_vmem_all();
#pragma unroll
  for (int q = 0; q < 2; ++q) st.m_lane[q] = st.m_ref[q] = m_in[q] / d.scale;      // -inf stays -inf
  __syncthreads();

  int boff = 0;
  if constexpr (PHASED) {
    Scores s;
    Ring kr, vr;
    bf16x8 pb[2][2];
    int k0 = 0;
    bool seen = false, masked = false;
    auto look_at = [&](int sb, int j) {
      k0 = j * BN + (CYCLIC && sb > shift_from);               // local to the sub-block
      seen = sb < segs && k0 < nvis_wave;
      masked = k0 + BN > nfull_wave;
    };
    // Interval t lies between the barriers t and t + 1.  In it wavefronts that are `behind` do the softmax of block t and then
    // the MFMAs - scores of block t + 1, products of block t -, the others these MFMAs and then the softmax of block t + 1: one sequence
    // for both, with the barrier at another place.  Requested right behind barrier t, used from barrier t + 1 on: K of block t + 2 into the
    // buffer of block t (its scores were made in the interval before), V of block t + 1 into that of block t - 1.
    // (Fragments requested earlier - the first of V in front of the exponentials or of the scores, the products in front of the
    // scores - cost 1-3 %: the wavefront that waits for them leaves the other one the vector ALU.)
    const bool behind = KL == 2 ? kl == 1 : wave >= 4;
    look_at(sb, j);
    if (seen) {
      fwd_first_keys<HR>(kr, rd, 0);
      fwd_scores<HR>(s, kr, qf, rd, 0);
    }
    if (behind) __syncthreads();
    while ((KL == 1 ? sb : lead_sb) < segs) {
      int n2_sb = nx_sb, n2_j = nx_j, n2_nblk = nx_nblk, n2_start = nx_start, n2_rows = nx_rows;
      if (nx_sb < segs) step_next(n2_sb, n2_j, n2_nblk, n2_start, n2_rows);
      auto request = [&]() {
        if (A2D_OFTEN(n2_sb < segs)) load_tile(1, n2_start, n2_rows, n2_j, boff);
        if (A2D_OFTEN(nx_sb < segs)) load_tile(2, nx_start, nx_rows, nx_j, BUF_BYTES - boff);
      };
      if (behind) request();                       // (the others: behind the barrier below)
      const bool mine = seen;
      if (mine)
        fwd_softmax<HR>(st, s, pb, masked, k0, my_vis, grp, c, []() {});
      if (!behind) {
        wait_vmem_all();
        __syncthreads();
        request();
      }
      if (!CYCLIC && A2D_SELDOM(nx_sb != sb && nx_sb < segs)) enter_segment(nx_sb);
      __builtin_amdgcn_s_setprio(0);               // (the softmax first, where both want to issue)
      look_at(nx_sb, nx_j);
      if (seen) {
        fwd_first_keys<HR>(kr, rd, BUF_BYTES - boff);
        fwd_scores<HR>(s, kr, qf, rd, BUF_BYTES - boff);
      }
      if (mine) {
        fwd_first_values<HR>(vr, rd, boff);
        fwd_products<HR>(st, pb, vr, rd, boff);
      }
      __builtin_amdgcn_s_setprio(1);
      if (behind) {
        wait_vmem_all();
        __syncthreads();
      }
      if (KL > 1) advance(stride, lead_sb, lead_j, lead_nblk);
      sb = nx_sb;
      nx_sb = n2_sb; nx_j = n2_j; nx_nblk = n2_nblk; nx_start = n2_start; nx_rows = n2_rows;
      boff = BUF_BYTES - boff;
    }
    if (!behind) __syncthreads();                  // (as many barriers for all)
    __builtin_amdgcn_s_setprio(0);
  } else {
    // (the next entry is found in the step that requests it: found a step ahead, the loop is 2 % slower - 4 x 14885 x 4812, H = 64, causal, two
    // blocks 90.6 -> 92.7 us, 9 x 16075 x 321 53.4 -> 54.6)
    while ((KL == 1 ? sb : lead_sb) < segs) {
      int nsb = sb, nj = j, nnblk = nblk;
      advance(stride, nsb, nj, nnblk);
      const bool more = nsb < segs;
      if (CYCLIC) nx_start = nsb;
      else if (A2D_SELDOM(more && nsb != sb)) { nx_start = seg_start(nsb); nx_rows = seg_rows(nsb); }
      if (A2D_OFTEN(more)) load_tile(3, nx_start, nx_rows, nj, BUF_BYTES - boff);
      const int k0 = j * BN + (CYCLIC && sb > shift_from);     // local to the sub-block
      if ((KL == 1 || sb < segs) && k0 < nvis_wave) fwd_block<HR>(st, qf, rd, boff, k0 + BN > nfull_wave, k0, my_vis, grp, c);
      wait_vmem_all();
      __syncthreads();
      if (!CYCLIC && A2D_SELDOM(more && nsb != sb)) enter_segment(nsb);
      if (KL > 1) advance(stride, lead_sb, lead_j, lead_nblk);
      sb = nsb; j = nj; nblk = nnblk;
      boff = BUF_BYTES - boff;
    }
  }

  // ---- epilogue: bring N and l to the true row maximum, store N, m (scaled units), l
  float m_row[2], f[2], l_tot[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    m_row[q] = row_max(st.m_lane[q]);
    f[q] = (m_row[q] == -INFINITY) ? 0.f : fast_exp2((st.m_ref[q] - m_row[q]) * c);
    l_tot[q] = row_sum(st.l_run[q]) * f[q];
  }
  if constexpr (KL == 2) {
    // Key lane 1 hands its (N, m, l) to lane 0 through LDS (the tiles are no longer read: every
    // wavefront has passed the walk's last barrier), which merges the two as Alg. 2 does.
    // Layout: [row wavefront][value index][lane], one float each, so every access is conflict free.
    constexpr int NV = HT * 8 + 4;
    static_assert(RW * NV * 256 <= KL * kLdsBytes, "the exchange area must fit the tile buffers");
    float* xch = reinterpret_cast<float*>(lds_all) + wave * NV * 64 + lane;
    if (kl == 1) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int t = 0; t < HT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) xch[(8 * t + 4 * q + r) * 64] = st.o[t][q][r] * f[q];
        xch[(HT * 8 + 2 * q) * 64] = m_row[q];
        xch[(HT * 8 + 2 * q + 1) * 64] = l_tot[q];
      }
    }
    __syncthreads();
    if (kl == 1) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float m1 = xch[(HT * 8 + 2 * q) * 64], l1 = xch[(HT * 8 + 2 * q + 1) * 64];
      const float m_new = fmaxf(m_row[q], m1);
      const float a0 = (m_row[q] == -INFINITY) ? 0.f : f[q] * fast_exp2((m_row[q] - m_new) * c);
      const float a1 = (m1 == -INFINITY) ? 0.f : fast_exp2((m1 - m_new) * c);
#pragma unroll
      for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) st.o[t][q][r] = st.o[t][q][r] * a0 + xch[(8 * t + 4 * q + r) * 64] * a1;
      l_tot[q] = (m_row[q] == -INFINITY ? 0.f : l_tot[q] * fast_exp2((m_row[q] - m_new) * c)) + l1 * a1;
      m_row[q] = m_new;
      f[q] = 1.f;
    }
  }
  // (KL = 2: inside what this wavefront has read of the exchange)
  char* const area = lds_all + wave * (KL == 2 ? (HT * 8 + 4) * 256 : acc_area(HT));
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int first = q0 + wave * 32 + 16 * q, r = first + (lane & 15);
    const bool stat = grp == 0 && r < d.nq;
    if (g.norm) {
      // normalised partial: O' = N / l rounded to bf16, lse' = m + ln l (Sec. 3.2, footnote)
      // (GRID: the row of O and lse itself)
      const int64_t row = GRID ? (int64_t)head * g.b.side * d.nq + grid_token(g.b, d.nq, row_blk, r) : (int64_t)head * d.nq + r;
      const int64_t o_at = GRID ? head * d.lo.head + row_blk * g.b.o + first * d.lo.row : ((int64_t)head * d.nq + first) * H;
      const float fn = l_tot[q] > 0.f ? f[q] / l_tot[q] : 0.f;
      store_acc16(reinterpret_cast<bf16_t*>(O_part) + o_at, GRID ? d.lo.row : H, d.nq - first, area, st.o, q, lane, fn);
      if (stat) m_out[row] = l_tot[q] > 0.f ? m_row[q] * d.scale + logf(l_tot[q]) : -INFINITY;
    } else {
      const int64_t row = (int64_t)head * d.nq + first;
      store_acc16(O_part + row * H, H, d.nq - first, area, st.o, q, lane, f[q]);
      if (stat) {
        m_out[row + (lane & 15)] = m_row[q] * d.scale;      // -inf stays -inf (scale > 0)
        l_out[row + (lane & 15)] = l_tot[q];
      }
    }
  }
}

}  // namespace

namespace {
template <int WAVES, int HR, int KL, int GRID, bool PHASED = false>
hipError_t fwd_launch(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                      float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  constexpr int bytes = fwd_lds(WAVES, padded_head(HR), KL), BM = 32 * WAVES / KL;
  if (ph == PREPARE)
    return ensure_dynamic_lds(reinterpret_cast<const void*>(fwd_mfma_kernel<WAVES, HR, KL, GRID, PHASED>), bytes);
  dim3 grid(xcd_grid(d.heads / g.group * g.parts, (GRID ? g.b.side : 1) * g.group * ((d.nq + BM - 1) / BM))), block(64 * WAVES);
  A2D_LAUNCH((fwd_mfma_kernel<WAVES, HR, KL, GRID, PHASED>), grid, block, bytes, s, d, g, (const bf16_t*)Q,
                     (const bf16_t*)K, (const bf16_t*)V, O_part, m, l, in);
  return hipGetLastError();
}
enum { FWD_BIG = 0, FWD_LANES = 1, FWD_PAIRS = 2, FWD_32 = 3, FWD_64 = 4 };   // <8, HR, 1>, <8, HR, 2>, <4, HR, 1>; fwd_small_kernel
}  // namespace

namespace {
template <int GRID>
hipError_t fwd_form(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                    float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
#define A2D_FWD(HR)                                                                            \
  return g.form == FWD_BIG     ? fwd_launch<8, HR, 1, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s) \
         : g.form == FWD_LANES ? fwd_launch<8, HR, 2, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s) \
                               : fwd_launch<4, HR, 1, GRID>(ph, d, g, Q, K, V, O_part, m, l, in, s)
  if (d.hdim == 128 && g.phased)
    return g.form == FWD_BIG ? fwd_launch<8, 128, 1, GRID, true>(ph, d, g, Q, K, V, O_part, m, l, in, s)
                             : fwd_launch<8, 128, 2, GRID, true>(ph, d, g, Q, K, V, O_part, m, l, in, s);
  if (d.hdim == 128) { A2D_FWD(128); }
  if (d.hdim == 96) { A2D_FWD(96); }
  if (d.hdim == 80) { A2D_FWD(80); }
  A2D_FWD(64);
#undef A2D_FWD
}
}  // namespace

// Shape and parts.  Five shapes: 256-row workgroups, one per compute unit; 128-row workgroups whose two
// key lanes walk alternate key blocks, one per compute unit; 128-row workgroups of four wavefronts, two
// per compute unit (each K / V tile is staged twice, but there is no merge of lanes and the last turn
// is finer); 64- and 32-row workgroups whose four or eight key lanes share the walk (a2d_fwd_small.hip; a step is a round
// of 128 or 256 keys).  By model, with parts > 1 where the blocks leave compute units idle and the walk is long.  The costs of tiles
// are a fit to 2700 of 1 to 96 heads, 32 to 16384 rows and keys, H = 64 to 128, a fifth of them with peaky logits (which rescale
// oftener), each in the five forms and up to nine numbers of parts, on three sets of inputs in turn (on one set, which stays in the caches,
// the forms that read more come out too well): 0.7 % off the best of them in the mean, 2.0 % with the costs fitted to earlier kernels
// (tiles that became slower count double in the fit).  Of 6000 other tiles 740 go out otherwise than before, 1.09 times as fast in
// the mean (84/21 x 12746 x 306, H = 64 204 -> 139 us, from 256 rows to pairs; an eighth of them slower by 3 % or more, at worst 4/1 x
// 10485 x 2347, H = 128, causal 62 -> 78).  32 rows are taken up to about 256 such blocks, 64 rows up to 256 of theirs, under a
// causal mask up to 512, with walks of 16 rounds at the most.  Two at a time side by side cost more power than one of 256 rows, so
// that at H = 128 large tiles stay there (96 x 4096 x 4096 720 us against 743, causal 400 / 406; H = 64 64 x 4096 x 4096 304 / 290).
void plan_fwd_mfma(const a2d_tile_desc& d, SegList* g, int cus, int cap) {
  const int64_t heads = (int64_t)d.heads * (g->b.side ? g->b.side : 1);
  double most = (double)visible_keys(d, *g, d.nq - 1) / BN + 0.2, mean = most;
  double seen[8];
  if (g->b.side) {                                             // (the rows of a whole sequence see half of it in the mean)
    most = (double)g->b.side * ((d.nkv + BN - 1) / BN) + 0.2;
    mean = d.causal ? 0.5 * most + 0.5 * (g->b.cyclic ? g->b.side : 1) : most;
    for (int i = 0; i < 8; ++i) seen[i] = (d.causal ? (15 - 2 * i) / 16.0 : 1.0) * most * BN;
  } else if (g->by_size) {
    mean = mean_visible_keys(d, *g, seen) / BN + 0.2;
  }
  const double* const sorted = mean < most ? seen : nullptr;
  const int h = d.hdim > 96 ? 2 : d.hdim > 64 ? 1 : 0;
  const FwdCosts& c = kFwdCosts[g->b.side > 0];
  const double step = c.step[h];
  const double part_us = (double)heads * d.nq * (d.hdim + 2) * 8 / 4.5e6;      // written and read back at 4.5 TB/s
  const int64_t b256 = heads * ((d.nq + 255) / 256), b128 = heads * ((d.nq + 127) / 128), b64 = heads * ((d.nq + 63) / 64), b32 = heads * ((d.nq + 31) / 32);
  // (plain calls write fp32 partials, 128 KiB a workgroup of 256 rows at H = 128: those that start and end together store
  // at the rate of the memory, two side by side on a compute unit one under the other's walk.  29 x 4679 x 359, H = 96: 49 us
  // in 256-row workgroups, 42 in pairs.  The walks of a causal grid are of every length down to a few steps, so that the last ones end
  // nearly together; those of 32 and 64 rows wait for each other's loads all the same: 7 heads, 5166 tokens on 3 x 3, H = 128, cyclic
  // 101 us with 0.1, 82 in pairs)
  const double store = g->b.side ? 0 : d.hdim / 128.0, big = c.fixed + c.big_more;
  const double big_fix = big + (b256 > cus ? c.big_store * store : 0), lanes_fix = c.fixed + c.lanes_more + (b128 > cus ? c.lanes_store * store : 0);
  const double pair_fix = store > 0 && b128 > 2 * cus ? c.pair_fixed + c.pair_store * store : c.fixed + c.alone_more;
  const WalkModel m[5] = {{b256, cus, mean, most, step, big_fix, 0, 0, nullptr, 0, c.tail},
                          {b128, cus, mean / 2, most / 2, step * c.lanes, lanes_fix, 0, 0, nullptr, 0, c.tail},
                          {b128, cus, mean, most, step * c.alone, c.fixed, step * c.pair[h], pair_fix, nullptr, 0, c.tail},
                          {b32, cus, mean / 4, most / 4, c.round32[h], c.fixed32[h], 0, 0, sorted, 0.25 / BN, 0.5, true},
                          {b64, cus, mean / 2, most / 2, c.round64[h], c.fixed64[h], 0, 0, sorted, 0.5 / BN, 0.5, true, true}};
  double least = 0;
  for (int f = 0; f < 5; ++f) {
    double t;
    const int z = best_parts(m[f], cap, f >= FWD_32 ? c.merge_few : c.merge, part_us, &t);
    if (f == 0 || t < (g->form == 0 ? 0.98 : 1.0) * least) { least = t; g->form = f; g->parts = z; }
  }
  // Opposite phases (PHASED), walks in order / in phases, us: 96 x 4096 x 4096, unmasked and then causal 1161 -> 1131, 21 x 2194 x 5272
  // 132.9 -> 124.8, 16/2 x 2416 x 3675 94.6 -> 89.1, 16 x 2048 x 2048 38.2 -> 37.6, 40/8 x 1300 gathered 71.2 -> 68.0.  They begin and end
  // with half a step that nothing stands beside, so that walks of a few steps lose: 9 x 2616 x 288 19.9 -> 20.9, 19 x 2218 x 213,
  // causal 14.8 -> 15.3, 9/3 x 4618 x 796 34.0 -> 34.6; from some 14 steps on they win.  32 drawn walks of that kind, unit-scale logits: 0.97 of the time
  // in order in the mean (0.93 to 1.01).  Not so with peaky ones (sigma 4, which no size tells): 1.02 (0.99 to 1.05), 16 x 2048 x 2048 41.8 -> 42.9,
  // and the same only from some hundred steps on.  Below H = 128, where a step's softmax is as long as its MFMAs, they lose oftener than they win:
  // 72/9 x 2302 x 7437, H = 96 487 -> 469, but 39 x 9559 x 1886, H = 80 916 -> 957, 9 x 4032 x 1332, H = 64 28.5 -> 31.4.
  constexpr double kPhasedSteps = 14;
  g->phased = d.hdim == 128 && g->form <= FWD_LANES && mean >= kPhasedSteps * g->parts * (g->form == FWD_LANES ? 2 : 1);
}

hipError_t launch_fwd_mfma(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                           const void* V, float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  if (g.form >= FWD_32) return launch_fwd_small(ph, g.form == FWD_64 ? 64 : 32, d, g, Q, K, V, O_part, m, l, in, s);
  return g.b.side == 0 ? fwd_form<0>(ph, d, g, Q, K, V, O_part, m, l, in, s)
         : g.b.cyclic  ? fwd_form<2>(ph, d, g, Q, K, V, O_part, m, l, in, s)
                       : fwd_form<1>(ph, d, g, Q, K, V, O_part, m, l, in, s);
}

}  // namespace a2d
