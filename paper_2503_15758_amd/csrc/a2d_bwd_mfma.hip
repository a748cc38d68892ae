// bf16 MFMA backward tile kernels for H = 128, 96, 80 and 64: the per-tile gradient call of Alg. 3
// line 3 with P = exp(S - lse) rebuilt from the FINAL log-sum-exp of the query block,
//   dV = P^T dO,  dP = dO V^T,  dS = P o (dP - delta),  dQ = scale dS K,  dK = scale dS^T Q.
//
// Two kinds of workgroups, so that every output has exactly one writer and no atomics are needed
// (bitwise reproducible results), in launches of their own here and in one launch in a2d_bwd_one.hip:
//   bwd_dkdv_kernel  owns key rows.  Workgroup = 8 wavefronts = 128 keys: four PAIRS of
//                    wavefronts (w, w + 4; both on SIMD w), 32 keys per pair.  The "score"
//                    wave of a pair holds the K^T fragments and the dV^T accumulators and
//                    computes S = Q K^T, P, dV^T += dO^T P; the "gradient" wave holds the V^T
//                    fragments and the dK^T accumulators and computes dP = dO V^T,
//                    dS = P o (dP - delta), dK^T += Q^T dS, with P handed over in fp32
//                    through LDS.  That halves the accumulators per wavefront (64 registers),
//                    so two wavefronts fit on a SIMD and one's exponentials overlap the
//                    other's MFMAs (a single wavefront cannot overlap the two).  The query
//                    blocks are walked 32 rows per step, staged through LDS together with dO,
//                    lse and delta; the gradient waves run one step behind the score waves, so
//                    one barrier per step is the only synchronisation.  S and dP leave a lane
//                    holding ONE key column, so P and dS feed the second contractions directly
//                    as B operands; dO^T / Q^T come from the LDS transpose read.
//                    Tiles with many keys take bwd_dkdv_wide_kernel (a2d_bwd_wide.hip) instead: 256 keys
//                    per workgroup, every wavefront doing all four contractions for 32 of them.
//   bwd_dq_kernel    owns query rows.  Workgroup = 8 wavefronts = 256 queries (32 per
//                    wavefront, Q and dO fragments in registers), two wavefronts per
//                    SIMD; walks the key blocks, 64 keys per step.  S^T = K Q^T
//                    and dP^T = V dO^T leave a lane holding ONE query column;
//                    dQ^T += K^T dS^T with K^T from the LDS transpose read.  Runs first and
//                    computes delta = rowsum(dO o O) of its rows for both kernels.  (Its body is dq_rows, a2d_bwd_dq.hpp;
//                    that of bwd_dkdv_kernel dkdv_pairs, a2d_bwd_pairs.hpp.)
//   bwd_dq_ds_kernel owns query rows like bwd_dq_kernel, but reads dS from a workspace the
//                    dK/dV kernel filled (its WRITE_DS variant) and only contracts it with K, so that S
//                    and dP are computed once (5 contractions for 5 counted ones instead of 7): large
//                    tiles of H = 128, where the caller allows it.
// Tiles that are read both ways (natural and transposed fragments) live in LDS in the blocks of a2d_mfma.hpp (Blocks16), those of
// bwd_dkdv_kernel in its "dual" layout: every fragment address is a per-lane base plus an immediate.
#include <type_traits>

#include "a2d_bwd_dq.hpp"
#include "a2d_bwd_pairs.hpp"

namespace a2d {
namespace {

using namespace mfma;

template <int HR, bool GROUPED, bool WRITE_DS, bool PLAIN = false>
__global__ __launch_bounds__(DK_THREADS) void bwd_dkdv_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO, const float* __restrict__ lse,
    const float* __restrict__ delta, float* __restrict__ dK, float* __restrict__ dV,
    bf16_t* __restrict__ dS) {
  warm_arguments<9 * 8>();
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  dkdv_pairs<HR, GROUPED, WRITE_DS, PLAIN, 0, false>(blockIdx.x, lds, d, g, g.parts, Q, K, V, nullptr, dO, lse, delta, dK, dV, dS);
}

template <int WAVES, int HR, int KL>
__global__ __launch_bounds__(64 * WAVES, 8 / WAVES) void bwd_dq_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, const bf16_t* __restrict__ O, const bf16_t* __restrict__ dO,
    const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dQ) {
  warm_arguments<8 * 8>();
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  dq_rows<WAVES, HR, KL, 0>(blockIdx.x, lds, d, g, g.parts, Q, K, V, O, dO, lse, delta, dQ);
}

// ---------------------------------------------------------------------- dQ from a stored dS
// Contraction-only dQ kernel: dQ^T += K^T dS^T with dS read back from the workspace the dK/dV
// kernel filled (layout at ds_row_tiles above).  Workgroup = WAVES wavefronts of 32 query rows;
// 64 keys per step: the K tile and every wavefront's own 4 KiB tile of dS come straight into LDS, in three stages
// where one workgroup has the compute unit (requests run two steps ahead), else two, and are read with the transposing
// loads.  The stream is HBM-bound: 2 bytes per score.  The sub-blocks of a gathered tile must start at multiples of 64
// keys, so that a 64-key block never straddles two of them.
constexpr int DSQ_RING = 4;
__host__ __device__ constexpr int dsq_stages(int waves, int kl) { return waves == 8 && kl == 1 ? 3 : 2; }
__host__ __device__ constexpr int dsq_stage(int rw, int hd) { return BKS * 2 * hd + rw * DS_TILE_BYTES; }   // { K tile, dS tiles }
__host__ __device__ constexpr int dsq_lds(int waves, int hd, int kl) { return kl * dsq_stages(waves, kl) * dsq_stage(waves / kl, hd); }
// A piece's granules (rows 4 g + 0..3 and 16 + 4 g + 0..3 of a key, 16 bytes) in LDS, and what a transposing read takes of them:
// 8 bytes a lane, of four g of eight keys at a time.  It meets every bank once with the keys of g = 2, 3 moved
// and the other half taken where g is odd, so that tile u of the results is made of the rows 16 (u ^ (g & 1)) + 4 g + 0..3.  With the
// granules in the order of memory and one half for all a bank was met four times (36 % of the kernel's LDS cycles at 96 x 4096 x 4096,
// now none; the time is the memory's: 2108 -> 2095 us for the whole call).
__host__ __device__ constexpr int dsq_granule(int g, int key) { return 16 * g + (key ^ (g >> 1 ? 12 : 0)); }
__host__ __device__ constexpr int dsq_at(int lane) {        // of tile 0 (of tile 1: ^ 8)
  return 16 * dsq_granule(lane & 3, 4 * (lane >> 4) + ((lane & 15) >> 2)) + 8 * (lane & 1);
}
__host__ __device__ constexpr int dsq_row(int u, int j) { return 16 * (u ^ (j >> 2 & 1)) + j; }
constexpr bool dsq_banks_once() {
  for (int first = 0; first < 64; first += 32) {             // half a wavefront's 8 bytes a lane are the 64 banks' width
    unsigned banks = 0;
    for (int l = first; l < first + 32; ++l) banks |= 1u << (dsq_at(l) / 8 % 32);
    if (banks != ~0u) return false;
  }
  return true;
}
static_assert(dsq_banks_once(), "the reads of dS meet a bank more than once");
template <int HD>
struct DsqCtx {
  f32x4 dq[HD / 16][2]; // column tiles x the wavefront's two tiles of 16 query rows (dsq_row)
  unsigned kt_e, kt_o;  // transposed fragments of the K tile of the current stage (Blocks16), ...
  unsigned ds[2];       // ... of the dS tile
  int my_vis[2];        // number of leading keys of the current sub-block this lane's query rows see
  int grp;
};

// one 32-key piece (T = 0, 1) of the step; key0 = its first key, local to its sub-block.  masked: some of the rows do not see
// all of its keys.
template <int T, int HD>
__device__ __forceinline__ void dsq_piece(DsqCtx<HD>& cx, int key0, bool masked) {
  constexpr int HT = HD / 16, KS = HD / 32;
  bf16x8 kt[DSQ_RING], dsb[2];
  auto ld = [&](auto I) {
    constexpr int i = decltype(I)::value;
    const unsigned at = (i & 1 ? cx.kt_o : cx.kt_e) + (T * 2 * KS + (i >> 1)) * BLOCK;
    kt[i % DSQ_RING] = lds_load_tr(at, at + KS * BLOCK);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int u = 0; u < 2; ++u) dsb[u] = lds_load_tr(cx.ds[u] + T * 2048, cx.ds[u] + T * 2048 + 1024);
  static_for<0, (DSQ_RING < HT ? DSQ_RING : HT)>(ld);
  if (A2D_SELDOM(masked)) {
    asm volatile("" ::: "memory");                 // keep this a branch
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      u32x4 w = __builtin_bit_cast(u32x4, dsb[u]);
      // element e of the fragment <-> key key0 + 16 (e >> 2) + 4 grp + (e & 3); two per word
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int k = key0 + 16 * (x >> 1) + 4 * cx.grp + 2 * (x & 1);
        const unsigned keep = (k < cx.my_vis[u] ? 0x0000FFFFu : 0u) | (k + 1 < cx.my_vis[u] ? 0xFFFF0000u : 0u);
        w[x] &= keep;
      }
      dsb[u] = __builtin_bit_cast(bf16x8, w);
    }
  }
  static_for<0, HT>([&](auto I) {
    constexpr int i = decltype(I)::value;
#pragma unroll
    for (int u = 0; u < 2; ++u) cx.dq[i][u] = mma16(kt[i % DSQ_RING], dsb[u], cx.dq[i][u]);
    if constexpr (i + DSQ_RING < HT) ld(std::integral_constant<int, i + DSQ_RING>{});
  });
}

// KL key lanes of WAVES / KL wavefronts: with KL = 2 a 128-row workgroup of eight wavefronts walks
// the key blocks in two lanes (alternate blocks, own K buffers) whose dQ sums are added through LDS
// at the end - for tiles with at most one 128-row block per compute unit, so that a SIMD still
// holds two wavefronts and twice the dS requests are in flight.
template <int WAVES, int HR, int KL>
__global__ __launch_bounds__(64 * WAVES, 8 / WAVES) void bwd_dq_ds_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ K, const bf16_t* __restrict__ dS,
    float* __restrict__ dQ) {
  warm_arguments<3 * 8>();
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];
  constexpr int RW = WAVES / KL;                       // wavefronts of one key lane
  constexpr int DQ_ROWS = 32 * RW, DQ_THREADS = 64 * RW;   // rows of the workgroup, threads of one key lane
  constexpr int HD = padded_head(HR), H = HR, HT = HD / 16, KS = HD / 32;
  constexpr int ST = dsq_stages(WAVES, KL), STAGE = dsq_stage(RW, HD), K_TILE = BKS * 2 * HD;
  const int kl = KL == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / DQ_THREADS);
  char* const lds = lds_all + kl * (ST * STAGE);
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int nqb = (d.nq + DQ_ROWS - 1) / DQ_ROWS;
  // placement as in bwd_dq_kernel (grouped heads: the query heads of a key/value head share an XCD)
  int unit, blk;
  if (!xcd_map(blockIdx.x, d.heads / g.group * g.parts, g.group * nqb, g.by_size != 0, unit, blk)) return;
  const int kvh = unit / g.parts, part = unit - kvh * g.parts;
  const int head = kvh * g.group + (g.by_size ? blk % g.group : blk / nqb);
  blk = g.by_size ? blk / g.group : blk % nqb;
  const int q0 = (nqb - 1 - blk) * DQ_ROWS;            // heavy blocks first under a causal mask
  const int tid = (int)threadIdx.x - kl * DQ_THREADS;  // within the key lane
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  K += (int64_t)kvh * d.lk.head;

  DsqCtx<HD> cx;
  cx.grp = lane >> 4;
  const int w_row = q0 + wave * 32;                    // the wavefront's first row
#pragma unroll
  for (int t = 0; t < HT; ++t) cx.dq[t][0] = cx.dq[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  Blocks16 at;
  at.init(lane, lds_base);
  cx.kt_e = at.tr_e;
  cx.kt_o = at.tr_o;
  cx.ds[0] = lds_base + K_TILE + wave * DS_TILE_BYTES + dsq_at(lane);
  cx.ds[1] = cx.ds[0] ^ 8;

  // this wavefront's row tile of dS (a wavefront past the last row reads the last tile; its
  // results are never stored)
  const int n_rt = ds_row_tiles(d.nq), n_kb = ds_key_blocks(d.nkv);
  const int rt = min((q0 + wave * 32) / 32, n_rt - 1);
  const gptr_t ds_base = uniform_gptr(reinterpret_cast<const char*>(dS) +
                                      head * ds_head_bytes(d.nq, d.nkv) +
                                      (int64_t)rt * n_kb * DS_TILE_BYTES);

  // visibility per key/value sub-block s: query i sees the first vis_count(i, s) keys of it
  auto vis_count = [&](int i, int s) -> int {
    if (!d.causal) return g.seg[s].rows;
    const int64_t v = (int64_t)i + g.seg[s].rel + 1;
    return v <= 0 ? 0 : (v < g.seg[s].rows ? (int)v : g.seg[s].rows);
  };
  const int blk_last = min(q0 + DQ_ROWS, d.nq) - 1;
  const int w_first = min(q0 + wave * 32, d.nq - 1);
  const int w_last = min(q0 + wave * 32 + 31, d.nq - 1);
  auto seg_blocks = [&](int s) { return (vis_count(blk_last, s) + BKS - 1) / BKS; };
  int count = 0;                                   // 64-key blocks the workgroup walks
  for (int s = 0; s < g.n; ++s) count += seg_blocks(s);

  // Walk over the visible blocks, as global block numbers (start of the sub-block / 64 + block
  // inside it): lane part * KL + kl of parts * KL takes every (parts * KL)-th.  The fetch walker runs
  // ahead of the compute walker; once it has run out it keeps returning its last block (loads stay
  // unconditional).
  const int stride = KL * g.parts;
  int f_sb = -1, f_j = 0, f_nblk = 0, f_id = 0;
  auto fetch_by = [&](int by) {
    int sb = f_sb, j = f_j + by, nblk = f_nblk;
    while (j >= nblk) {
      j -= nblk;
      nblk = 0;
      do { ++sb; } while (sb < g.n && (nblk = seg_blocks(sb)) == 0);
      if (sb >= g.n) return;
    }
    f_id = g.seg[sb].start / BKS + j;
    f_sb = sb; f_j = j; f_nblk = nblk;
  };
  int c_sb = -1, c_j = 0, c_nblk = 0;              // compute walker: sub-block, block inside it
  int nvis_wave = 0, nfull_wave = 0;
  auto compute_by = [&](int by) {
    c_j += by;
    while (c_j >= c_nblk) {
      c_j -= c_nblk;
      c_nblk = 0;
      do { ++c_sb; } while (c_sb < g.n && (c_nblk = seg_blocks(c_sb)) == 0);
      if (c_sb >= g.n) {                           // past the last block: nothing to compute
        c_sb = g.n - 1; c_j = 0; c_nblk = 0;
        nvis_wave = 0;
        return;
      }
      nvis_wave = vis_count(w_last, c_sb);
      nfull_wave = vis_count(w_first, c_sb);
      for (int u = 0; u < 2; ++u) cx.my_vis[u] = vis_count(min(w_row + dsq_row(u, lane & 15), d.nq - 1), c_sb);
    }
  };

  // ---- staging, straight into LDS: a wavefront's own tile of dS, and its share of the K tile - half a row tile of eight
  // wavefronts, a whole one of four.  Rows past the end re-read the last key.
  static_assert(H == 128, "K blocks are dealt out whole");
  constexpr int K_N = 4 * KS / RW, LOADS = K_N + 4;
  const int ld_tile = wave & 3, ld_sl = RW == 8 ? (wave >> 2) * K_N : 0;
  const int ld_chunk = (lane & 3) ^ block_swap(lane >> 4);
  const char* const k_base = reinterpret_cast<const char*>(K) + 64 * ld_sl;
  const unsigned k_row_bytes = __builtin_amdgcn_readfirstlane((unsigned)d.lk.row * 2);
  auto load = [&](int id, unsigned stage) {        // block id into the stage at `stage`
    const int r = min(16 * ld_tile + (lane >> 2), d.nkv - 1 - id * BKS);
    const gptr_t kb = uniform_gptr(k_base + (uint64_t)(unsigned)(id * BKS) * k_row_bytes);
    dma_blocks<K_N, H>(stage + (ld_tile * KS + ld_sl) * BLOCK, kb, __umul24(r, k_row_bytes) + 16 * ld_chunk, ld_chunk);
    const gptr_t from = ds_base + (unsigned)id * DS_TILE_BYTES;
    // (dS is read once: kept from displacing the K tiles in L2)
    static_for<0, 4>([&](auto I) {
      constexpr int off = 1024 * decltype(I)::value;
      dma_b128<off, true>(stage + K_TILE + wave * DS_TILE_BYTES + off, from, dsq_granule(lane >> 4, lane & 15) * 16);
    });
  };

  // (KL = 2: inside what this wavefront has read of the exchange)
  char* const area = lds_all + wave * (KL == 2 ? HT * 8 * 256 : acc_area(HT));
  auto store_rows = [&](float mul, bool add) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      store_acc16(dQ + (((int64_t)part * d.heads + head) * d.nq + w_row) * H, H, d.nq - w_row, area, cx.dq, u, lane, mul, add,
                  [u](int r) { return dsq_row(u, r); });
  };
  count = count > part * KL ? count - part * KL : 0;           // from this part's first block on
  if (count == 0) {                                // no visible key: dQ share is zero
    if (!g.acc && kl == 0) store_rows(0.f, false);
    return;
  }
  // (the first block is block 0; a lane without one re-reads the last block it passed)
  fetch_by(0);
  fetch_by(part * KL);
  if (KL > 1) fetch_by(kl);
  load(f_id, lds_base);
  if (ST == 3) {
    fetch_by(stride);
    load(f_id, lds_base + STAGE);
  }
  compute_by(part * KL + kl);
  wait_vmem<(ST - 2) * LOADS>();                   // (block 0 has arrived)
  __syncthreads();

  // iteration t: block t + ST - 1 is requested into the stage of block t - 1, block t is computed, block t + 1 has arrived.
  // (blocks past the last find nvis_wave = 0)
  unsigned cur = 0;
  for (int t = 0; t < (count + stride - 1) / stride; ++t) {
    fetch_by(stride);
    load(f_id, lds_base + (cur == 0 ? (ST - 1) * STAGE : cur - STAGE));
    const int k0 = c_j * BKS;                      // local to the sub-block
    if (k0 < nvis_wave) dsq_piece<0>(cx, k0, k0 + 32 > nfull_wave);
    if (k0 + 32 < nvis_wave) dsq_piece<1>(cx, k0 + 32, k0 + 64 > nfull_wave);
    const int go = cur == (ST - 1) * STAGE ? -(ST - 1) * STAGE : STAGE;
    cx.kt_e += go; cx.kt_o += go; cx.ds[0] += go; cx.ds[1] += go;
    cur += go;
    compute_by(stride);
    wait_vmem<(ST - 2) * LOADS>();
    __syncthreads();
  }
  wait_vmem_all();                                 // (requests past the last block, of every wavefront, before LDS is used otherwise or left)
  __syncthreads();
  if constexpr (KL == 2) {
    // lane 1 hands its sums to lane 0 through LDS (the K tiles are no longer read: every wavefront
    // has passed the walk's last barrier); layout [row wavefront][value][lane]: conflict free
    static_assert(RW * HT * 8 * 256 <= dsq_lds(WAVES, HD, KL), "the exchange area must fit the stages");
    __syncthreads();
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
  store_rows(d.scale, g.acc != 0);
}

}  // namespace

bool bwd_mfma_supported(const a2d_tile_desc& d) {
  return d.dtype == A2D_BF16 && (d.hdim == 128 || d.hdim == 96 || d.hdim == 80 || d.hdim == 64);
}

// Bytes of the dS workspace of a tile (0 when the hand-over does not apply: a sub-block that does
// not start at a multiple of 64 keys, or 4 GiB or more per key/value head).  Below H = 128 it is not used
// (plan_bwd_mfma); its size is part of the interface, so that callers' sizes hold whatever the plan does.
size_t bwd_ds_bytes(const a2d_tile_desc& d, const SegList& g) {
  if (!bwd_mfma_supported(d)) return 0;
  for (int s = 0; s < g.n; ++s)
    if (g.seg[s].start % 64 != 0) return 0;
  const size_t per_head = ds_head_bytes(d.nq, d.nkv);
  if (per_head * (size_t)g.group >= ((size_t)1 << 32)) return 0;   // 32-bit offsets inside a key/value head's share
  return per_head * (size_t)d.heads;
}

namespace {
enum { DQ_BIG = 0, DQ_LANES = 1, DQ_PAIRS = 2 };   // <8, HR, 1>, <8, HR, 2>, <4, HR, 1>

template <int HR>
hipError_t bwd_launch_ds(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                         const void* V, const void* dO, const float* lse, const float* delta, float* dQ, float* dK,
                         float* dV, void* ds_ws, const BwdParts& parts, hipStream_t s) {
  constexpr int HD = padded_head(HR);
  const bool grouped = g.group > 1;
  hipError_t e = hipSuccess;
  SegList gk = g, gq = g;
  gk.parts = parts.kv;
  gq.parts = parts.q;
  if (parts.q > 1) gq.acc = 0;                         // (the sum over the parts adds)
  const bool big = parts.form == DQ_BIG, lanes = parts.form == DQ_LANES;
  if (ph == PREPARE) {
    e = parts.wide ? launch_dkdv_wide(ph, d, gk, Q, K, V, dO, lse, delta, dK, dV, ds_ws, s)
        : ensure_dynamic_lds(grouped ? reinterpret_cast<const void*>(bwd_dkdv_kernel<HR, true, true>)
                                   : reinterpret_cast<const void*>(bwd_dkdv_kernel<HR, false, true>), DK_LDS);
    if (e != hipSuccess) return e;
    return lanes ? ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dq_ds_kernel<8, HR, 2>), dsq_lds(8, HD, 2))
           : big ? ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dq_ds_kernel<8, HR, 1>), dsq_lds(8, HD, 1))
                 : ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dq_ds_kernel<4, HR, 1>), dsq_lds(4, HD, 1));
  }
  dim3 grid_kv(xcd_grid(d.heads / g.group * parts.kv, (d.nkv + DK_KEYS - 1) / DK_KEYS));
  const int dq_rows = big ? 256 : 128;
  dim3 grid_q(xcd_grid(d.heads / g.group * parts.q, g.group * ((d.nq + dq_rows - 1) / dq_rows)));
  if (parts.wide)
    e = launch_dkdv_wide(ph, d, gk, Q, K, V, dO, lse, delta, dK, dV, ds_ws, s);
  else if (grouped)
    A2D_LAUNCH((bwd_dkdv_kernel<HR, true, true>), grid_kv, dim3(DK_THREADS), DK_LDS, s, d, gk,
                       (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, lse, delta, dK, dV,
                       (bf16_t*)ds_ws);
  else
    A2D_LAUNCH((bwd_dkdv_kernel<HR, false, true>), grid_kv, dim3(DK_THREADS), DK_LDS, s, d, gk,
                       (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, lse, delta, dK, dV,
                       (bf16_t*)ds_ws);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (big)
    A2D_LAUNCH((bwd_dq_ds_kernel<8, HR, 1>), grid_q, dim3(512), dsq_lds(8, HD, 1), s, d, gq, (const bf16_t*)K,
                       (const bf16_t*)ds_ws, dQ);
  else if (lanes)
    A2D_LAUNCH((bwd_dq_ds_kernel<8, HR, 2>), grid_q, dim3(512), dsq_lds(8, HD, 2), s, d, gq, (const bf16_t*)K,
                       (const bf16_t*)ds_ws, dQ);
  else
    A2D_LAUNCH((bwd_dq_ds_kernel<4, HR, 1>), grid_q, dim3(256), dsq_lds(4, HD, 1), s, d, gq, (const bf16_t*)K,
                       (const bf16_t*)ds_ws, dQ);
  return hipGetLastError();
}

template <int HR>
hipError_t bwd_launch_hd(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                         const void* V, const void* O, const void* dO, const float* lse, float* delta, float* dQ, float* dK,
                         float* dV, void* ds_ws, const BwdParts& parts, hipStream_t s) {
  if constexpr (HR == 128)                             // (dS is kept at H = 128 only, see plan_bwd_mfma)
    if (ds_ws) return bwd_launch_ds<HR>(ph, d, g, Q, K, V, dO, lse, delta, dQ, dK, dV, ds_ws, parts, s);
  constexpr int DQ_LDS = dq_launch_lds(padded_head(HR), 1), DQ_LDS2 = dq_launch_lds(padded_head(HR), 2), DQ_LDS4 = dq_lds(padded_head(HR));
  const bool grouped = g.group > 1;
  // Q and dO in the plain layout: the variant with compile-time staging offsets
  const bool plain = d.lq.row == HR && d.ldo.row == HR && d.lq.head == (int64_t)d.nq * HR && d.ldo.head == d.lq.head;
  SegList gk = g, gq = g;
  gk.parts = parts.kv;
  gq.parts = parts.q;
  if (parts.q > 1) gq.acc = 0;                         // (the sum over the parts adds)
  const bool big = parts.form == DQ_BIG, lanes = parts.form == DQ_LANES;
  hipError_t e = hipSuccess;
  if (ph == PREPARE) {
    const void* dkdv = plain ? (grouped ? reinterpret_cast<const void*>(bwd_dkdv_kernel<HR, true, false, true>)
                                        : reinterpret_cast<const void*>(bwd_dkdv_kernel<HR, false, false, true>))
                             : (grouped ? reinterpret_cast<const void*>(bwd_dkdv_kernel<HR, true, false, false>)
                                        : reinterpret_cast<const void*>(bwd_dkdv_kernel<HR, false, false, false>));
    e = parts.wide ? launch_dkdv_wide(ph, d, gk, Q, K, V, dO, lse, delta, dK, dV, nullptr, s) : ensure_dynamic_lds(dkdv, DK_LDS);
    if (e != hipSuccess) return e;
    return lanes ? ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dq_kernel<8, HR, 2>), DQ_LDS2)
           : big ? ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dq_kernel<8, HR, 1>), DQ_LDS)
                 : ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dq_kernel<4, HR, 1>), DQ_LDS4);
  }
  dim3 grid_kv(xcd_grid(d.heads / g.group * parts.kv, (d.nkv + DK_KEYS - 1) / DK_KEYS));
  const int dq_rows = big ? 256 : 128;
  dim3 grid_q(xcd_grid(d.heads / g.group * parts.q, g.group * ((d.nq + dq_rows - 1) / dq_rows)));
  if (big)
    A2D_LAUNCH((bwd_dq_kernel<8, HR, 1>), grid_q, dim3(512), DQ_LDS, s, d, gq, (const bf16_t*)Q,
                       (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, (const bf16_t*)dO, lse, delta, dQ);
  else if (lanes)
    A2D_LAUNCH((bwd_dq_kernel<8, HR, 2>), grid_q, dim3(512), DQ_LDS2, s, d, gq, (const bf16_t*)Q,
                       (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, (const bf16_t*)dO, lse, delta, dQ);
  else
    A2D_LAUNCH((bwd_dq_kernel<4, HR, 1>), grid_q, dim3(256), DQ_LDS4, s, d, gq, (const bf16_t*)Q,
                       (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, (const bf16_t*)dO, lse, delta, dQ);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
#define A2D_DKDV(GR, PL)                                                                                          \
  A2D_LAUNCH((bwd_dkdv_kernel<HR, GR, false, PL>), grid_kv, dim3(DK_THREADS), DK_LDS, s, d, gk, (const bf16_t*)Q, \
                     (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, lse, delta, dK, dV, (bf16_t*)nullptr)
  if (parts.wide) return launch_dkdv_wide(ph, d, gk, Q, K, V, dO, lse, delta, dK, dV, nullptr, s);
  if (grouped && plain) A2D_DKDV(true, true);
  else if (grouped) A2D_DKDV(true, false);
  else if (plain) A2D_DKDV(false, true);
  else A2D_DKDV(false, false);
#undef A2D_DKDV
  return hipGetLastError();
}
}  // namespace

// How a backward goes out (steps in microseconds; H = 64, 96, 128):
//   - in one launch, recomputing (a2d_bwd_one.hip), for whole grids, and where its workgroups come to at most six turns of the
//     chip and no engine's share comes out badly: against dQ and dK/dV one after the other 0.6 of the time at a few
//     workgroups, 0.8-0.95 at one to three turns, the same at four (1 x 161 x 308 20 -> 11 us, 16 x 1024 x 1024 74 -> 50,
//     16 x 2048 x 2048 144 -> 130; from some ten turns on 1 % slower).  The second kind does not fill what the first leaves of
//     its last turn where the shader engines are dealt unlike numbers of the long walks (dealt_time): 72/18 heads x 651 x 861,
//     H = 64 88 us in one launch, 77 in two; 6 x 9048 x 1290, H = 128 197 / 174; 51 x 2015 x 438, H = 64 96 / 88; 9 x 563 x
//     2404, H = 80 50 / 43.  kOneUs is fitted to 770 drawn shapes of up to six turns, and favours one launch a little: where the
//     walks are even the choice is 0.1 % off the better one in the mean (one launch always: 0.4 %, 23 % at worst).  Of uneven
//     walks 3 % of the shapes would be 3-9 % faster in two and neither model tells which (84 x 1117 x 2587, H = 96, causal
//     167 / 154): 0.3 % in the mean.
//   - with dS kept, where the caller allows it and the model says so: at H = 128 only.  Below, recomputing S and dP costs
//     less than writing and reading dS (64 x 4096 x 4096 H = 64 1044 against 1157 us, H = 80 1268 / 1320, 16 x 2048 x 2048
//     H = 64 79 / 103; of 262 drawn shapes of H = 64 to 96 15 % in the mean, 14 of them 2-11 % slower: 36 x 1413 x 2468, H = 96
//     221 / 199).  At H = 128, beyond six turns, it is
//     always taken: 74 drawn shapes 1.03 times as fast in the mean, 96 x 4096 x 4096 2151 -> 2056 us, causal 1201 -> 1158, 64 x 4096 x
//     4096 1424 -> 1355; ten of them slower, by 2 % in the mean but for 40/10 x 9013 x 522, 378 -> 429.  A whole step of 96 x 4096 x
//     4096 tiles, forward and merges included, gains less, 5.71 -> 5.68 ms: the forward runs cooler behind a backward that recomputes.
//     Up to six turns by the model (16 x 2048 x 2048, one turn, 138 us kept, 130 in one launch).
//   - else dQ, recomputing, then dK/dV.
// Parts of the dK/dV and dQ walks where their row blocks leave compute units idle, and the dQ kernels' workgroup
// shape, as in plan_fwd_mfma; measured over 30 unmasked shapes (1 x 300 x 8000 to 32 x 2000 x 2700) and 44 causal ones.
// Half as many workgroups of 256 keys pay from the point where those of 128 no longer run at once.  The choice for
// dK/dV does not depend on `ds`, so that the two dQ paths give the same dK, dV.
BwdParts plan_bwd_mfma(const a2d_tile_desc& d, const SegList& g, bool ds, int cus, int cap_kv, int cap_q) {
  constexpr double kKvUs[3] = {0.75, 0.85, 1.0}, kWideUs[3] = {1.0, 1.2, 1.5};
  constexpr double kDqUs[3] = {1.6, 1.75, 2.1};
  constexpr double kOneUs[3] = {1.03, 1.0, 0.85};      // two launches' modelled time over that of one which takes as long
  const int hx = d.hdim > 96 ? 2 : d.hdim > 64 ? 1 : 0, kv_heads = d.heads / g.group, side = g.b.side ? g.b.side : 1;
  // (a grid's walks are `side` times as long; under the mask of every length down to a few steps)
  const bool grid = g.b.side > 0, uneven = grid ? d.causal != 0 : g.by_size != 0;
  double of_rows[8];                                   // keys that rows see
  const double seen = mean_visible_keys(d, g, of_rows);
  const double rows = (double)g.group * side * ((d.nq + BQ - 1) / BQ);
  const double kv_mean = !uneven ? rows : grid ? 0.5 * rows + side : rows * seen / d.nkv + 1;
  const double most = grid ? (double)side * ((d.nkv + BKS - 1) / BKS) + 0.2 : (double)visible_keys(d, g, d.nq - 1) / BKS + 0.2;
  const double mean = !uneven ? most : grid ? 0.5 * most + 0.5 * (g.b.cyclic ? side : 1) : seen / BKS + 0.2;
  const double kv_part_us = (double)kv_heads * d.nkv * d.hdim * 16 / 4.5e6;
  const auto walk = [&](int w) {                       // 128 keys per workgroup, 256
    const int keys = w ? 256 : DK_KEYS;
    return WalkModel{(int64_t)kv_heads * ((d.nkv + keys - 1) / keys), cus, kv_mean, rows, (w ? kWideUs : kKvUs)[hx],
                     w ? 10.0 : 8.0, 0, 0, nullptr, 0};
  };
  const double* sorted = g.by_size ? of_rows : nullptr;
  const double fixed = 7.0;
  const int64_t heads = d.heads, b256 = heads * ((d.nq + 255) / 256), b128 = heads * ((d.nq + 127) / 128);
  const double part_us = (double)heads * d.nq * d.hdim * 8 / 4.5e6;
  // (dS comes at the rate of the memory: a full chip's steps take longer)
  const auto full = [&](int64_t n) { return n < cus ? (double)n / cus : 1.0; };
  const auto rows_of = [&](bool from_ds, BwdParts* p) {    // shape and parts of the dQ launch; its time
    const double step = from_ds ? 0.7 + 0.9 * full(b256) : kDqUs[hx];
    const WalkModel q[3] = {{b256, cus, mean, most, step, fixed, 0, 0, sorted, 1.0 / BKS},
                            {b128, cus, mean / 2, most / 2, step * 1.2, fixed + 0.5, 0, 0, sorted, 0.5 / BKS},
                            {b128, cus, mean, most, step * 0.74, fixed, step, fixed + 0.5, nullptr, 0}};
    double least = 0;
    for (int f = 0; f < 3; ++f) {
      double t;
      const int z = best_parts(q[f], cap_q, p->kv > 1 ? 1.0 : 4.0, part_us, &t);   // (one launch sums both)
      if (f == 0 || t < (p->form == 0 ? 0.98 : 1.0) * least) { least = t; p->form = f; p->q = z; }
    }
    return least;
  };

  const int64_t wgs = (int64_t)side * (kv_heads * (int64_t)((d.nkv + 255) / 256) + d.heads * (int64_t)((d.nq + 255) / 256));
  const bool few = wgs <= 6 * (int64_t)cus;
  BwdParts one = {}, plan = {};                        // recomputing, in one launch ...
  double one_us = 0, dealt_us = 0;
  if (grid || few) {
    const BwdWalks w = {kv_mean < rows ? kv_mean : rows, rows, mean < most ? mean : most, most, uneven};
    one_us = plan_bwd_one(d, g, w, cus, cap_kv, cap_q, &one, &dealt_us);
    if (grid || one.small) return one;
  }
  double kv_us[2];                                     // ... or dQ, then dK/dV
  int kv_parts[2];
  for (int w = 0; w < 2; ++w) kv_parts[w] = best_parts(walk(w), cap_kv, 4.0, kv_part_us, &kv_us[w]);
  plan.wide = kv_us[1] < kv_us[0] && d.scale > 1e-30f;     // (it takes lse / scale, which has to stay finite)
  plan.kv = kv_parts[plan.wide];
  double plan_us = kv_us[plan.wide];
  plan_us = (plan_us + rows_of(false, &plan)) / kOneUs[hx];
  if (few && dealt_us <= plan_us) {
    plan = one;
    plan_us = one_us;
  }
  if (!ds || d.hdim != 128) return plan;
  BwdParts kept = {};
  kept.wide = plan.wide;
  kept.kv = plan.kv;
  kept.keep_ds = 1;
  const double dq_us = rows_of(true, &kept);
  if (!few) return kept;
  WalkModel kv = walk(kept.wide);                      // (a full chip clocks lower, most so beside the dS stores)
  const double f = full(kv.blocks * kept.kv);
  kv.step = kept.wide ? 1.3 + 0.8 * f * f : 1.1;
  kv.tail = 0.3;
  const double kept_us = 8.0 + walk_time(kv, kept.kv) + (kept.kv > 1 ? 4.0 + kept.kv * kv_part_us : 0) + dq_us;
  return plan_us * (wgs >= cus ? 1.08 : 1.0) <= kept_us ? plan : kept;
}

// ds_ws != NULL: a workspace of bwd_ds_bytes(d, g) bytes; the dK/dV kernel leaves dS there and the
// dQ kernel is the contraction-only one; `delta` holds rowsum(dO o O) then.  Otherwise the dQ kernel
// runs first and computes delta from O for itself and the dK/dV kernel (a launch less).
hipError_t launch_bwd_mfma(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                           const void* V, const void* O, const void* dO, const float* lse, float* delta, float* dQ,
                           float* dK, float* dV, void* ds_ws, const BwdParts& parts, hipStream_t s) {
  if (parts.one) return launch_bwd_one(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
  if (d.hdim == 128) return bwd_launch_hd<128>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, ds_ws, parts, s);
  if (d.hdim == 96) return bwd_launch_hd<96>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, ds_ws, parts, s);
  if (d.hdim == 80) return bwd_launch_hd<80>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, ds_ws, parts, s);
  return bwd_launch_hd<64>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, ds_ws, parts, s);
}

}  // namespace a2d
