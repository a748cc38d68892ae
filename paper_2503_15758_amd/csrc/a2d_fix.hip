// AttnFix (Alg. 2) folded over k partials + normalisation (Alg. 1 line 6), and the
// plain-sum merge of gradient partials (Alg. 3 lines 4-5).  Both are pure
// streaming kernels bound by HBM bandwidth: every input byte is read once with
// 128-bit loads, all k loads of a thread are issued before the first use (those of more than 16 partials one behind the other).
#include <type_traits>

#include "a2d_common.hpp"

namespace a2d {
namespace {

// Each thread handles CPT 16-byte column groups and issues the loads of all of them (CPT * k
// 128-bit loads) before the first use: the amount of data in flight per thread, not the
// arithmetic, decides how close these kernels get to the HBM rate.
// (read once: non-temporal loads measured 8-10 % faster than plain ones here)
#define A2D_LD(p) __builtin_nontemporal_load(p)
// How many groups a thread has, and how the results are stored, for `groups` column groups (weights: AttnFix, which holds m and l besides N;
// half: AttnFix of normalised bf16 partials, groups of 8 bytes).  Few groups come to as many workgroups as they can, many have the loads of two or
// four in flight; in between lies what was measured, on three sets of inputs in turn.  One / two / four groups, us for rows x H, the better way
// to store:
//   AttnFix k = 2, 63709 x 96 12.4 / 11.9 / 11.8, 266808 x 64 32.8 / 31.9 / 32.7; k = 4, 17278 x 96 6.9 / 7.1 / 7.4, 19386 x 128
//   8.7 / 8.4 / 9.4, 32768 x 128 15.1 / 14.2 / 13.9, 51946 x 128 22.2 / 21.6 / 21.0, 65536 x 128 27.1 / 26.2 / 26.3; k = 6, 15593 x 64 5.9 / 5.9 / 6.7,
//   39088 x 64 12.9 / 11.9 / 13.5, 60062 x 96 27.8 / 27.4 / 26.7; k = 8, 12366 x 96 8.6 / 9.2 / 11.1, 15492 x 128 13.6 / 12.4 / 13.1, 104325 x 96
//   58.7 / 56.7 / 57.2; k = 16, 8355 x 80 9.3 / 10.7 / 11.4, 29059 x 64 23.5 / 22.1 / 25.9, 39760 x 96 48.6 / 46.9 / 51.5;
//   sums of 2 to 4 one; k = 6, 15990 x 96 7.5 / 7.1 / 7.7, 30774 x 64 9.6 / 9.1 / 8.8, 48288 x 80 19.0 / 19.6 / 18.6; k = 8, 12493 x 128 10.1 / 10.4 / 9.6,
//   62396 x 96 36.8 / 37.1 / 35.4; k = 16, 12573 x 64 10.3 / 9.6 / 9.6, 16622 x 128 24.5 / 24.8 / 27.3, 31214 x 128 46.7 / 47.0 / 42.6;
//   half k = 2, 358276 x 64 26.4 / 24.7 / 24.0, k = 4, 59542 x 80 10.8 / 10.0 / 10.8, k = 8, 51209 x 96 17.1 / 17.4 / 18.0, k = 16, 30544 x 64 13.2 /
//   13.4 / 14.5, 52452 x 96 31.3 / 31.5 / 32.9.
// through, plain / written through: sum k = 3, 5385 x 64 2.2 / 2.1; AttnFix k = 6, 28217 x 64 8.9 / 9.3, k = 8, 35492 x 64 14.4 / 15.0,
// k = 4, 12322 x 128 6.2 / 6.4, 92778 x 96 32.3 / 30.2; sum k = 8, 13455 x 128 9.9 / 10.6, 266664 x 64 100.7 / 98.7.
// Against kernels of one to four groups by the number of partials alone, plain stores and loads under conditions: 430 merges, 1.06 to 1.28
// times as fast in the mean of a set; of those between 2^17.5 and 2^20 groups a tenth are 1 to 5 % slower, at worst 9 % (sum of 16, 6168 x 128).
struct Way {
  int cpt;
  bool through;
};
constexpr int64_t kGroups = 1 << 14;               // (64 workgroups of one group a thread)
constexpr Way way_of(int kmax, bool weights, bool half, int64_t groups) {
  const int64_t n = groups / kGroups;
  int cpt = 1;
  if (half) cpt = n < 32 || kmax == 1 || kmax > 16 ? 1 : kmax == 2 && n >= 128 ? 4 : 2;
  else if (weights && kmax == 2) cpt = n < 32 ? 1 : 2;
  else if (weights && (kmax == 3 || kmax == 4)) cpt = n < 24 ? 1 : n >= (kmax == 3 ? 64 : 50) && n < 128 ? 4 : 2;
  else if (weights && kmax > 4) cpt = n < (kmax == 16 ? 11 : 20) || kmax > 16 ? 1 : kmax == 6 && n >= 52 ? 4 : 2;
  else if (kmax == 16) cpt = n < 11 ? 1 : n < 40 ? 2 : 4;
  else if (kmax > 4) cpt = n < 24 || kmax > 16 ? 1 : 4;
  const int through = cpt == 1 || (kmax == 16 && !weights) ? 32 : !weights || half ? 48 : kmax <= 4 ? 128 : kmax == 6 ? 96 : 48;
  const int plain = kmax == 3 || (kmax == 4 && !weights) ? 16 : 11;
  return {cpt, kmax <= 2 || n < plain || n >= through};
}

// Which column groups a thread owns: its wavefront owns CPT * 64 CONSECUTIVE groups and lane l takes
// the groups l, l + 64, ... of that run, so that every load instruction of a wavefront reads 1 KiB
// in one piece and its CPT loads of one partial read CPT KiB in one piece.  (Measured on MI355X: a
// read stream made of such per-wavefront runs of 4-16 KiB reaches 6.8-7.0 TB/s, the same bytes
// requested one grid-sized stride apart 5.3-6.4 TB/s.)
// A workgroup's groups are [first, first + rest); everything of a thread is numbered from `first` on, in 32 bits, and goes
// through buffer descriptors of the workgroup's own share: no 64-bit arithmetic in a lane, and the loads past
// the end give zeros without a branch (a sum of 8 partials, 96 x 4096 rows of 128: 283 -> 277 us).
template <int CPT>
struct Share {
  int64_t first;
  unsigned rest;
  // (from: the first group of the launch, see launch_slices)
  __device__ __forceinline__ Share(int64_t from, int64_t total) {
    first = from + (int64_t)blockIdx.x * (256 * CPT);
    rest = (unsigned)min(total - first, (int64_t)(256 * CPT));
  }
  __device__ __forceinline__ unsigned at(int c) const { return (threadIdx.x >> 6) * (CPT * 64) + c * 64 + (threadIdx.x & 63); }
};
enum { NT = 2, THROUGH = 16 };                     // cache policies of the buffer instructions: read once; straight on to memory
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, int64_t bytes_before, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(static_cast<const char*>(p)) + bytes_before, 0, bytes, 0x00020000);
}
__device__ __forceinline__ void load(float& v, __amdgpu_buffer_rsrc_t b, unsigned i) {
  v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, i * 4, 0, 0));
}
__device__ __forceinline__ void load(f32x4& v, __amdgpu_buffer_rsrc_t b, unsigned i) {
  v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, i * 16, 0, NT));
}
__device__ __forceinline__ void load(bf16x4& v, __amdgpu_buffer_rsrc_t b, unsigned i) {
  v = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(b, i * 8, 0, NT));
}
// Partial x of k: v[c] = elements at[c] of the `n` from p + before on; zeros past them and of an absent partial.
// Up to four partials there is a kernel for each number; of more, absent ones have no size: no branch around them, so that the pointers of
// all come in together (us, with branches / without: AttnFix 8 x 96 x 4096 297 / 292, 16 x 16 x 8000 171 / 169, sum 2 x 53212 x 64 7.0 / 6.5).
// BRANCH, sums of three and four: with one, which makes a thread read a pointer, request its 16 bytes, and then read the next pointer.  The
// requests, spread out like that, suit partials that lie a power of two apart, whose same places meet the same channels (4 x 16 x 1024 x 128
// 7.1 / 7.4, 4 x 16 x 2048 13.0 / 13.5, 3 x 16 x 1024 5.8 / 6.1); others are the same from 2^18 groups on and 2 to 4 % slower below.
template <bool BRANCH, int KMAX, int CPT, typename T>
__device__ __forceinline__ void load_partial(T (&v)[CPT][KMAX], int x, int k, const T* p, int64_t before, unsigned n, const unsigned (&at)[CPT]) {
  if (BRANCH && x >= k) {                          // (never taken: k is KMAX here)
#pragma unroll
    for (int c = 0; c < CPT; ++c) v[c][x] = T{};
    return;
  }
  const auto b = buffer(p, before * (int)sizeof(T), KMAX <= 4 || x < k ? n * (unsigned)sizeof(T) : 0);
#pragma unroll
  for (int c = 0; c < CPT; ++c) load(v[c][x], b, at[c]);
}
__device__ __forceinline__ void store_out4(float* O, int64_t off, f32x4 v) {
  *reinterpret_cast<f32x4*>(O + off) = v;
}
__device__ __forceinline__ void store_out4(bf16_t* O, int64_t off, f32x4 v) {
  bf16x4 b;
  b[0] = (bf16_t)v[0]; b[1] = (bf16_t)v[1]; b[2] = (bf16_t)v[2]; b[3] = (bf16_t)v[3];
  *reinterpret_cast<bf16x4*>(O + off) = b;
}

// Where column group i of the share goes: plain, or row r of head h (nq rows per head) at h * head + r * row elements.
// Results of small and of large merges are written through: at 96 x 4096 rows of 128 and 8 partials the reads alone take 230 us, a seventeenth as many bytes
// of results another 50, as lines that the stream of reads drives out of the L2s one by one; sent on at once (device
// scope) 277 -> 265, non-temporal 275, collected in LDS and stored in longer runs 270 to 305; fp32 results 254 -> 248, non-temporal 269.
template <typename OutT>
struct Results {
  OutT* O;
  const OutMap& om;
  __amdgpu_buffer_rsrc_t b;
  int64_t first, h0, r0;                           // the share's first group; strided: head and row in it of the share's first row
  int hv;
  template <int CPT>
  __device__ __forceinline__ Results(OutT* o, const OutMap& m, const Share<CPT>& sh, int64_t row0, int h) : O(o), om(m), first(sh.first), hv(h) {
    b = buffer(O, first * 4 * sizeof(OutT), sh.rest * 4 * sizeof(OutT));
    h0 = om.plain ? 0 : row0 / om.nq;
    r0 = om.plain ? 0 : row0 - h0 * om.nq;
  }
  // (row, col: its row, counted from the share's first one, and its place in it)
  template <int POLICY>
  __device__ __forceinline__ void store_plain(unsigned i, f32x4 v) const {
    if constexpr (sizeof(OutT) == 4) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, i * 16, 0, POLICY);
    } else {
      bf16x4 o;
      o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), b, i * 8, 0, POLICY);
    }
  }
  __device__ __forceinline__ void store(unsigned i, unsigned row, unsigned col, f32x4 v) const {
    if (om.plain == OutMap::PLAIN_THROUGH) {
      store_plain<THROUGH>(i, v);
    } else if (om.plain) {
      store_plain<0>(i, v);
    } else {
      const unsigned r = (unsigned)r0 + row, h = r / (unsigned)om.nq;
      store_out4(O, (h0 + h) * om.head + (int64_t)(r - h * (unsigned)om.nq) * om.row + col * 4, v);
    }
  }
};

// A column group = 4 consecutive columns of one row; hv = H / 4 groups per row.
// KMAX is the unroll bound (k <= KMAX; k itself up to four).
// TRIPLE: the merge alone (Alg. 2 over k inputs): the result stays an unnormalised partial
// (N, m, l) - O receives N in fp32, lse receives m, l_out receives l.
template <typename OutT, int KMAX, int CPT, bool TRIPLE = false>
__global__ __launch_bounds__(256) void fix_kernel(FixPtrs p, int k, int64_t from, int64_t rows, int hv, OutMap om,
                                                  OutT* __restrict__ O, float* __restrict__ lse,
                                                  float* __restrict__ l_out) {
  const Share<CPT> sh(from, rows * hv);
  unsigned at[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) at[c] = sh.at(c);
  int64_t row0;
  unsigned rem, row[CPT];                          // (rows counted from row0)
  f32x4 n[CPT][KMAX];
  float mk[CPT][KMAX], lk[CPT][KMAX];
  const auto rows_of = [&]() {                     // (some hundred instructions: behind the large requests, 8 x 96 x 4096 300 -> 292 us)
    row0 = sh.first / hv;
    rem = (unsigned)(sh.first - row0 * hv);
#pragma unroll
    for (int c = 0; c < CPT; ++c) row[c] = (rem + at[c]) / (unsigned)hv;
  };
  if constexpr (KMAX > 16) {
    // (more descriptors than scalar registers: plain pointers and one row a lane.  The split walk of 1 x 128 x 16384, whose
    // merge is 16 workgroups, 16.8 -> 15.4 us)
    static_assert(CPT == 1, "");
    const int64_t idx = sh.first + at[0], r = idx / hv;
#pragma unroll
    for (int x = 0; x < KMAX; ++x) {
      if (x < k && idx < rows * hv) {
        n[0][x] = A2D_LD(reinterpret_cast<const f32x4*>(p.o[x]) + idx);
        mk[0][x] = p.m[x][r];
        lk[0][x] = p.l[x][r];
      } else {
        n[0][x] = f32x4{0.f, 0.f, 0.f, 0.f};
        mk[0][x] = -INFINITY;
        lk[0][x] = 0.f;
      }
    }
    row0 = r;                                      // (the lane's own row)
    row[0] = 0;
    rem = (unsigned)(idx - r * hv) - at[0];
  } else {
#pragma unroll
    for (int x = 0; x < KMAX; ++x) load_partial<false>(n, x, k, reinterpret_cast<const f32x4*>(p.o[x]), sh.first, sh.rest, at);
    __builtin_amdgcn_sched_barrier(0);
    rows_of();
    const unsigned stat = (unsigned)min(rows - row0, (int64_t)(256 * CPT));
#pragma unroll
    for (int x = 0; x < KMAX; ++x) {
      load_partial<false>(mk, x, k, p.m[x], row0, stat, row);
      load_partial<false>(lk, x, k, p.l[x], row0, stat, row);
    }
#pragma unroll
    for (int x = 0; x < KMAX; ++x)
#pragma unroll
      for (int c = 0; c < CPT; ++c)
        if (KMAX > 4 && x >= k) mk[c][x] = -INFINITY;
  }
  const Results<OutT> out(O, om, sh, row0, hv);
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const unsigned i = at[c], col = rem + i - row[c] * (unsigned)hv;
    if (i >= sh.rest) continue;
    float M = -INFINITY;
#pragma unroll
    for (int x = 0; x < KMAX; ++x) M = fmaxf(M, mk[c][x]);
    float D = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < KMAX; ++x) {
      // weight of partial x: exp(m_x - M); an empty partial (m = -inf) weighs 0
      const float w = (mk[c][x] == -INFINITY) ? 0.f : fast_exp2((mk[c][x] - M) * kLog2e);
      D = fmaf(w, lk[c][x], D);
      acc[0] = fmaf(w, n[c][x][0], acc[0]);
      acc[1] = fmaf(w, n[c][x][1], acc[1]);
      acc[2] = fmaf(w, n[c][x][2], acc[2]);
      acc[3] = fmaf(w, n[c][x][3], acc[3]);
    }
    if constexpr (TRIPLE) {
      if (col == 0) {                              // (first: behind the other store the wait for l would be one for it too)
        lse[row0 + row[c]] = M;
        l_out[row0 + row[c]] = D;
      }
      out.store(i, row[c], col, acc);
    } else {
      const float inv = (D > 0.f) ? 1.0f / D : 0.f;
      acc[0] *= inv; acc[1] *= inv; acc[2] *= inv; acc[3] *= inv;
      out.store(i, row[c], col, acc);
      if (col == 0) lse[row0 + row[c]] = (D > 0.f) ? M + logf(D) : -INFINITY;
    }
  }
}

template <typename OutT, int KMAX, int CPT>
__global__ __launch_bounds__(256) void sum_kernel(SumPtrs p, int k, int64_t from, int64_t n4, int hv, OutMap om,
                                                  OutT* __restrict__ out) {
  const Share<CPT> sh(from, n4);
  unsigned at[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) at[c] = sh.at(c);
  f32x4 v[CPT][KMAX];
#pragma unroll
  for (int x = 0; x < KMAX; ++x) {
    load_partial<KMAX == 3 || KMAX == 4>(v, x, k, reinterpret_cast<const f32x4*>(p.p[x]), sh.first, sh.rest, at);
  }
  const int64_t row0 = om.plain ? 0 : sh.first / hv;           // (plain results need no rows)
  const unsigned rem = om.plain ? 0 : (unsigned)(sh.first - row0 * hv);
  const Results<OutT> res(out, om, sh, row0, hv);
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const unsigned i = at[c], row = om.plain ? 0 : (rem + i) / (unsigned)hv;
    if (i >= sh.rest) continue;
    // left-to-right sum over the partials (absent ones hold zeros)
    f32x4 acc = v[c][0];
#pragma unroll
    for (int x = 1; x < KMAX; ++x) {
      acc[0] += v[c][x][0]; acc[1] += v[c][x][1]; acc[2] += v[c][x][2]; acc[3] += v[c][x][3];
    }
    res.store(i, row, rem + i - row * (unsigned)hv, acc);
  }
}

// Merge of k NORMALISED partials: L = log sum_k exp(lse_k), O = sum_k exp(lse_k - L) O'_k.  A
// column group = 4 consecutive columns of one row, as in fix_kernel; InT is the partials' dtype.
template <typename InT, typename OutT, int KMAX, int CPT>
__global__ __launch_bounds__(256) void fix_norm_kernel(NormPtrs p, int k, int64_t from, int64_t rows, int hv, OutMap om,
                                                       OutT* __restrict__ O, float* __restrict__ lse) {
  const Share<CPT> sh(from, rows * hv);
  unsigned at[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) at[c] = sh.at(c);
  typedef InT in4 __attribute__((ext_vector_type(4)));
  in4 n[CPT][KMAX];
  float lk[CPT][KMAX];
#pragma unroll
  for (int x = 0; x < KMAX; ++x) {
    load_partial<false>(n, x, k, reinterpret_cast<const in4*>(p.o[x]), sh.first, sh.rest, at);
  }
  const int64_t row0 = sh.first / hv;
  const unsigned rem = (unsigned)(sh.first - row0 * hv), stat = (unsigned)min(rows - row0, (int64_t)(256 * CPT));
  unsigned row[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) row[c] = (rem + at[c]) / (unsigned)hv;
#pragma unroll
  for (int x = 0; x < KMAX; ++x) {
    load_partial<false>(lk, x, k, p.lse[x], row0, stat, row);
  }
#pragma unroll
  for (int x = 0; x < KMAX; ++x)
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (KMAX > 4 && x >= k) lk[c][x] = -INFINITY;
  const Results<OutT> out(O, om, sh, row0, hv);
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const unsigned i = at[c], col = rem + i - row[c] * (unsigned)hv;
    if (i >= sh.rest) continue;
    float M = -INFINITY;
#pragma unroll
    for (int x = 0; x < KMAX; ++x) M = fmaxf(M, lk[c][x]);
    float D = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < KMAX; ++x) {
      // weight of partial x relative to the largest lse; an empty partial (lse = -inf) weighs 0
      const float w = (lk[c][x] == -INFINITY) ? 0.f : fast_exp2((lk[c][x] - M) * kLog2e);
      D += w;
      acc[0] = fmaf(w, to_f32(n[c][x][0]), acc[0]);
      acc[1] = fmaf(w, to_f32(n[c][x][1]), acc[1]);
      acc[2] = fmaf(w, to_f32(n[c][x][2]), acc[2]);
      acc[3] = fmaf(w, to_f32(n[c][x][3]), acc[3]);
    }
    const float inv = (D > 0.f) ? 1.0f / D : 0.f;
    acc[0] *= inv; acc[1] *= inv; acc[2] *= inv; acc[3] *= inv;
    out.store(i, row[c], col, acc);
    if (col == 0) lse[row0 + row[c]] = (D > 0.f) ? M + logf(D) : -INFINITY;
  }
}

// ---- the merges of a whole emulated grid whose walks were split, one launch for all its blocks.  Same
// arithmetic and order of sums as above; where a block's rows go follows from GridMap.
// (Everything but the partials' addresses fits 32 bits: the launcher checks it.)
struct GridRow {
  int b, h, i;                                     // block, head, row inside the block
  __device__ __forceinline__ GridRow(const GridMap& g, unsigned row) {
    const unsigned hb = row / (unsigned)g.rows;
    i = row - hb * g.rows;
    b = hb / (unsigned)g.heads;
    h = hb - b * g.heads;
  }
  // inside the head's sequence
  __device__ __forceinline__ int token(const GridMap& g) const { return g.cyclic ? i * g.side + b : b * g.rows + i; }
};

template <typename OutT, int KMAX>
__global__ __launch_bounds__(256) void fix_grid_kernel(FixPtrs p, GridMap g, int hv, a2d_layout lo,
                                                       OutT* __restrict__ O, float* __restrict__ lse) {
  const unsigned idx = blockIdx.x * 256 + threadIdx.x;
  const unsigned row = idx / (unsigned)hv, col = idx - row * hv;
  if (row >= (unsigned)(g.side * g.heads * g.rows)) return;
  const GridRow gr(g, row);
  f32x4 n[KMAX];
  float mk[KMAX], lk[KMAX];
#pragma unroll
  for (int x = 0; x < KMAX; ++x) {
    if (x < g.parts) {
      n[x] = A2D_LD(reinterpret_cast<const f32x4*>(p.o[x]) + idx);
      mk[x] = p.m[x][row];
      lk[x] = p.l[x][row];
    } else {
      n[x] = f32x4{0.f, 0.f, 0.f, 0.f};
      mk[x] = -INFINITY;
      lk[x] = 0.f;
    }
  }
  float M = -INFINITY;
#pragma unroll
  for (int x = 0; x < KMAX; ++x) M = fmaxf(M, mk[x]);
  float D = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int x = 0; x < KMAX; ++x) {
    const float w = (mk[x] == -INFINITY) ? 0.f : fast_exp2((mk[x] - M) * kLog2e);
    D = fmaf(w, lk[x], D);
    acc[0] = fmaf(w, n[x][0], acc[0]);
    acc[1] = fmaf(w, n[x][1], acc[1]);
    acc[2] = fmaf(w, n[x][2], acc[2]);
    acc[3] = fmaf(w, n[x][3], acc[3]);
  }
  const float inv = (D > 0.f) ? 1.0f / D : 0.f;
  acc[0] *= inv; acc[1] *= inv; acc[2] *= inv; acc[3] *= inv;
  const int t = gr.token(g);
  store_out4(O, gr.h * lo.head + t * lo.row + col * 4, acc);
  if (col == 0) lse[(int64_t)gr.h * g.side * g.rows + t] = (D > 0.f) ? M + logf(D) : -INFINITY;
}

struct SumSets {
  SumSet s[3];
};
template <typename OutT, int KMAX>
__global__ __launch_bounds__(256) void sum_grid_kernel(SumSets a, int hv) {
  const SumSet& s = a.s[blockIdx.y];
  const GridMap& g = s.gm;
  const unsigned idx = blockIdx.x * 256 + threadIdx.x;
  const unsigned row = idx / (unsigned)hv, col = idx - row * hv;
  if (row >= (unsigned)(g.side * g.heads * g.rows)) return;
  const GridRow gr(g, row);
  f32x4 v[KMAX];
#pragma unroll
  for (int x = 0; x < KMAX; ++x) {
    if (x < g.parts) v[x] = A2D_LD(reinterpret_cast<const f32x4*>(s.p.p[x]) + idx);
    else v[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 acc = v[0];
#pragma unroll
  for (int x = 1; x < KMAX; ++x) {
    acc[0] += v[x][0]; acc[1] += v[x][1]; acc[2] += v[x][2]; acc[3] += v[x][3];
  }
  store_out4(static_cast<OutT*>(s.out), gr.h * s.lo.head + gr.token(g) * s.lo.row + col * 4, acc);
}

// The partial results of a split walk, which lie one behind the other: out (+)= sum over the parts,
// in their order.  Small data that the kernel before it left in L2: one 16-byte group per thread, four
// loads in flight.  blockIdx.y picks the set.
struct PartSets {
  PartSet s[3];
};
__global__ __launch_bounds__(256) void sum_parts_kernel(PartSets a) {
  const PartSet& s = a.s[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, n4 = s.n / 4;
  if (i >= n4) return;
  const f32x4* p = reinterpret_cast<const f32x4*>(s.p) + i;
  f32x4* out = reinterpret_cast<f32x4*>(s.out) + i;
  f32x4 acc = s.add ? *out : f32x4{0.f, 0.f, 0.f, 0.f};
  int z = 0;
  for (; z + 4 <= s.k; z += 4) {
    f32x4 v[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] = p[(z + x) * n4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      acc[0] += v[x][0]; acc[1] += v[x][1]; acc[2] += v[x][2]; acc[3] += v[x][3];
    }
  }
  for (; z < s.k; ++z) {
    const f32x4 v = p[z * n4];
    acc[0] += v[0]; acc[1] += v[1]; acc[2] += v[2]; acc[3] += v[3];
  }
  *out = acc;
}

// (go(std::integral_constant<int, CPT>, first group, grid): launches)
// HIP launches no 2^32 threads and more at a time: merges of more groups than that go out in slices of 2^31 threads.
constexpr int64_t kSliceBlocks = (int64_t)1 << 23;
template <int CPT, class F>
void launch_slices(int64_t groups, F&& go) {
  constexpr int64_t share = 256 * CPT;
  for (int64_t from = 0; from < groups; from += kSliceBlocks * share) {
    const int64_t blocks = (groups - from + share - 1) / share;
    go(std::integral_constant<int, CPT>{}, from, dim3((unsigned)(blocks < kSliceBlocks ? blocks : kSliceBlocks)));
  }
}
constexpr bool occurs(int kmax, bool weights, bool half, int cpt) {        // (the rule changes last at 128 kGroups)
  for (int n = 0; n <= 128; ++n)
    if (way_of(kmax, weights, half, n * kGroups).cpt == cpt) return true;
  return false;
}
template <int KMAX, bool WEIGHTS, bool HALF, class F>
void with_chunks(int64_t groups, OutMap om, F&& go) {
  const Way w = way_of(KMAX, WEIGHTS, HALF, groups);
  if (om.plain && w.through) om.plain = OutMap::PLAIN_THROUGH;
  const auto of = [&](auto C, int64_t from, dim3 grid) { go(C, from, grid, om); };
  if constexpr (occurs(KMAX, WEIGHTS, HALF, 2)) {
    if (w.cpt == 2) return launch_slices<2>(groups, of);
  }
  if constexpr (occurs(KMAX, WEIGHTS, HALF, 4)) {
    if (w.cpt == 4) return launch_slices<4>(groups, of);
  }
  launch_slices<1>(groups, of);
}

template <typename OutT, int KMAX, bool TRIPLE = false>
void fix_launch(int k, int64_t rows, int hv, const FixPtrs& p, const OutMap& om, OutT* O, float* lse, float* l_out,
                hipStream_t s) {
  with_chunks<KMAX, true, false>(rows * hv, om, [&](auto C, int64_t from, dim3 grid, const OutMap& map) {
    constexpr int CPT = decltype(C)::value;
    A2D_LAUNCH((fix_kernel<OutT, KMAX, CPT, TRIPLE>), grid, dim3(256), 0, s, p, k, from, rows, hv, map, O, lse, l_out);
  });
}

template <typename OutT, int KMAX>
void sum_launch(int k, int64_t n4, int hv, const SumPtrs& p, const OutMap& om, OutT* out, hipStream_t s) {
  with_chunks<KMAX, false, false>(n4, om, [&](auto C, int64_t from, dim3 grid, const OutMap& map) {
    constexpr int CPT = decltype(C)::value;
    A2D_LAUNCH((sum_kernel<OutT, KMAX, CPT>), grid, dim3(256), 0, s, p, k, from, n4, hv, map, out);
  });
}

template <typename OutT, bool TRIPLE = false>
hipError_t fix_dispatch(int k, int64_t rows, int hdim, const FixPtrs& p, const OutMap& om, OutT* O, float* lse,
                        float* l_out, hipStream_t s) {
  const int hv = hdim / 4;
  if (k <= 1) fix_launch<OutT, 1, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else if (k <= 2) fix_launch<OutT, 2, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else if (k <= 3) fix_launch<OutT, 3, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else if (k <= 4) fix_launch<OutT, 4, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else if (k <= 6) fix_launch<OutT, 6, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else if (k <= 8) fix_launch<OutT, 8, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else if (k <= 16) fix_launch<OutT, 16, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  else fix_launch<OutT, 32, TRIPLE>(k, rows, hv, p, om, O, lse, l_out, s);
  return hipGetLastError();
}

template <typename OutT>
hipError_t sum_dispatch(int k, int64_t n, int hv, const SumPtrs& p, const OutMap& om, OutT* out, hipStream_t s) {
  const int64_t n4 = n / 4;
  if (k <= 1) sum_launch<OutT, 1>(k, n4, hv, p, om, out, s);
  else if (k <= 2) sum_launch<OutT, 2>(k, n4, hv, p, om, out, s);
  else if (k <= 3) sum_launch<OutT, 3>(k, n4, hv, p, om, out, s);
  else if (k <= 4) sum_launch<OutT, 4>(k, n4, hv, p, om, out, s);
  else if (k <= 6) sum_launch<OutT, 6>(k, n4, hv, p, om, out, s);
  else if (k <= 8) sum_launch<OutT, 8>(k, n4, hv, p, om, out, s);
  else if (k <= 16) sum_launch<OutT, 16>(k, n4, hv, p, om, out, s);
  else sum_launch<OutT, 32>(k, n4, hv, p, om, out, s);
  return hipGetLastError();
}


template <typename InT, typename OutT, int KMAX>
void fix_norm_launch(int k, int64_t rows, int hv, const NormPtrs& p, const OutMap& om, OutT* O, float* lse, hipStream_t s) {
  with_chunks<KMAX, true, sizeof(InT) == 2>(rows * hv, om, [&](auto C, int64_t from, dim3 grid, const OutMap& map) {
    constexpr int CPT = decltype(C)::value;
    A2D_LAUNCH((fix_norm_kernel<InT, OutT, KMAX, CPT>), grid, dim3(256), 0, s, p, k, from, rows, hv, map, O, lse);
  });
}

template <typename InT, typename OutT>
hipError_t fix_norm_dispatch(int k, int64_t rows, int hdim, const NormPtrs& p, const OutMap& om, OutT* O, float* lse,
                             hipStream_t s) {
  const int hv = hdim / 4;
  if (k <= 1) fix_norm_launch<InT, OutT, 1>(k, rows, hv, p, om, O, lse, s);
  else if (k <= 2) fix_norm_launch<InT, OutT, 2>(k, rows, hv, p, om, O, lse, s);
  else if (k <= 3) fix_norm_launch<InT, OutT, 3>(k, rows, hv, p, om, O, lse, s);
  else if (k <= 4) fix_norm_launch<InT, OutT, 4>(k, rows, hv, p, om, O, lse, s);
  else if (k <= 6) fix_norm_launch<InT, OutT, 6>(k, rows, hv, p, om, O, lse, s);
  else if (k <= 8) fix_norm_launch<InT, OutT, 8>(k, rows, hv, p, om, O, lse, s);
  else if (k <= 16) fix_norm_launch<InT, OutT, 16>(k, rows, hv, p, om, O, lse, s);
  else fix_norm_launch<InT, OutT, 32>(k, rows, hv, p, om, O, lse, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fix_norm(int k, int64_t rows, int hdim, int in_dtype, int out_dtype, const NormPtrs& p,
                           const OutMap& om, void* O, float* lse, hipStream_t s) {
  if (in_dtype == A2D_BF16) {
    if (out_dtype == A2D_BF16) return fix_norm_dispatch<bf16_t, bf16_t>(k, rows, hdim, p, om, (bf16_t*)O, lse, s);
    return fix_norm_dispatch<bf16_t, float>(k, rows, hdim, p, om, (float*)O, lse, s);
  }
  if (out_dtype == A2D_BF16) return fix_norm_dispatch<float, bf16_t>(k, rows, hdim, p, om, (bf16_t*)O, lse, s);
  return fix_norm_dispatch<float, float>(k, rows, hdim, p, om, (float*)O, lse, s);
}

hipError_t launch_fix(int k, int64_t rows, int hdim, int out_dtype, const FixPtrs& p, const OutMap& om, void* O,
                      float* lse, hipStream_t s) {
  if (out_dtype == A2D_BF16) return fix_dispatch<bf16_t>(k, rows, hdim, p, om, (bf16_t*)O, lse, nullptr, s);
  return fix_dispatch<float>(k, rows, hdim, p, om, (float*)O, lse, nullptr, s);
}

namespace {
template <typename OutT>
void fix_grid_dispatch(const GridMap& gm, int hv, const FixPtrs& p, const a2d_layout& lo, OutT* O, float* lse,
                       hipStream_t s) {
  const dim3 grid((unsigned)(((int64_t)gm.side * gm.heads * gm.rows * hv + 255) / 256)), block(256);
  const int k = gm.parts;
#define A2D_GO(KMAX) A2D_LAUNCH((fix_grid_kernel<OutT, KMAX>), grid, block, 0, s, p, gm, hv, lo, O, lse)
  if (k <= 2) A2D_GO(2);
  else if (k <= 4) A2D_GO(4);
  else if (k <= 8) A2D_GO(8);
  else if (k <= 16) A2D_GO(16);
  else A2D_GO(32);
#undef A2D_GO
}
template <typename OutT>
void sum_grid_dispatch(int nsets, const SumSets& a, int hv, int64_t blocks, hipStream_t s) {
  const dim3 grid((unsigned)blocks, nsets), block(256);
  int k = 0;
  for (int x = 0; x < nsets; ++x) k = a.s[x].gm.parts > k ? a.s[x].gm.parts : k;
#define A2D_GO(KMAX) A2D_LAUNCH((sum_grid_kernel<OutT, KMAX>), grid, block, 0, s, a, hv)
  if (k <= 2) A2D_GO(2);
  else if (k <= 4) A2D_GO(4);
  else if (k <= 8) A2D_GO(8);
  else if (k <= 16) A2D_GO(16);
  else A2D_GO(32);
#undef A2D_GO
}
}  // namespace

hipError_t launch_fix_grid(const GridMap& gm, int hdim, int out_dtype, const FixPtrs& p, const a2d_layout& lo, void* O,
                           float* lse, hipStream_t s) {
  if (out_dtype == A2D_BF16) fix_grid_dispatch<bf16_t>(gm, hdim / 4, p, lo, (bf16_t*)O, lse, s);
  else fix_grid_dispatch<float>(gm, hdim / 4, p, lo, (float*)O, lse, s);
  return hipGetLastError();
}

hipError_t launch_sum_grid(int nsets, const SumSet* sets, int hdim, int out_dtype, hipStream_t s) {
  SumSets a;
  int64_t most = 0;
  for (int x = 0; x < 3; ++x) {
    a.s[x] = sets[x < nsets ? x : 0];
    const int64_t n = (int64_t)a.s[x].gm.side * a.s[x].gm.heads * a.s[x].gm.rows * (hdim / 4);
    if (n > most) most = n;
  }
  if (out_dtype == A2D_BF16) sum_grid_dispatch<bf16_t>(nsets, a, hdim / 4, (most + 255) / 256, s);
  else sum_grid_dispatch<float>(nsets, a, hdim / 4, (most + 255) / 256, s);
  return hipGetLastError();
}

hipError_t launch_sum_parts(int nsets, const PartSet* sets, hipStream_t s) {
  PartSets a;
  int64_t most = 0;
  for (int x = 0; x < 3; ++x) {
    a.s[x] = sets[x < nsets ? x : 0];
    if (a.s[x].n > most) most = a.s[x].n;
  }
  A2D_LAUNCH(sum_parts_kernel, dim3((unsigned)((most / 4 + 255) / 256), nsets), dim3(256), 0, s, a);
  return hipGetLastError();
}

// the merge alone: k partials in, one unnormalised partial (N, m, l) out
hipError_t launch_attnfix(int k, int64_t rows, int hdim, const FixPtrs& p, float* N, float* m, float* l,
                          hipStream_t s) {
  return fix_dispatch<float, true>(k, rows, hdim, p, plain_out(), N, m, l, s);
}

// hv = column groups per row (only used when the output is not plain)
hipError_t launch_fix_bwd(int k, int64_t n, int hv, int out_dtype, const SumPtrs& p, const OutMap& om, void* out,
                          hipStream_t s) {
  if (out_dtype == A2D_BF16) return sum_dispatch<bf16_t>(k, n, hv, p, om, (bf16_t*)out, s);
  return sum_dispatch<float>(k, n, hv, p, om, (float*)out, s);
}

}  // namespace a2d
