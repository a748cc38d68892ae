// fp32 tile kernels on the fp32 matrix units: forward (Sec. 3.1, Eq. (3), block by block with the
// recurrence of Sec. 2.2) and the per-tile gradient call of Alg. 3 line 3, for H = 64, 80, 96, 128.
// fp32 throughout: v_mfma_f32_16x16x4_f32 multiplies and accumulates in fp32 (2048 flop in 32 cycles
// of a SIMD, 157 TFLOP/s over the chip - twice what unpacked vector FMAs reach).
//
// What bounds them: the fp32 MFMA rate where there are many rows (84 % of it at 16 x 4096 x 4096, H = 128, in both passes); at
// 16 x 700 x 900 prologues, merges and uneven walks of a few steps (58 %).  A step of 16 keys (queries)
// against 16 rows is H / 4 MFMAs of 32 cycles per contraction, on 8 KiB of operands at H = 128.
//   - The backward's dQ and dK/dV workgroups go out in one launch, so that the end of the one kind overlaps the start of
//     the other (two launches, dQ leaving delta for dK/dV: 2 x 128 x 128, H = 64 13.4 -> 7.1 us; 16 x 700 x 900, H = 96,
//     causal 109 -> 100).
//   - Operands of a step pass through a tile in LDS that is the wavefront's own (no barriers): a contraction over H needs
//     lane = row, and loading that from memory is 64 separate accesses per instruction, which kept the matrix units
//     half idle (16 heads x 1024 x 1024, H = 96: 6.4e7 cache accesses for 1.2 GB, 50 % MFMA busy).
//   - The forward's K tile goes straight into LDS, the next block's as soon as the scores are there, and V by columns into registers as
//     soon as the products are through.  With K one block ahead in registers and V requested at the start of its own step, two workgroups
//     shared a compute unit; without these 20 to 32 registers three to four of 16 rows do.  us, before -> now: 16 x 1024 x 1024,
//     H = 128 / 96 / 80 / 64 81.8 / 63.3 / 52.1 / 43.4 -> 75.3 / 59.0 / 49.8 / 41.5 (114 TFLOP/s, 73 % of the peak, at H = 128), 12 x 1024 x 600, H = 128
//     42.4 -> 38.0, 8 x 500 x 1000, H = 80 19.0 -> 17.4, 3 x 600 x 1000, H = 64 13.5 -> 11.7, 16 x 700 x 900, H = 96, causal 31.9 -> 30.5;
//     22 shapes 1.06 times as fast in the mean, 180 drawn ones 1.05, none more than 1 % slower.
//   - The backward loads its tiles straight into LDS, each as soon as the last read of the one before is through: V behind dP, K
//     behind half of dQ; Q behind half of dK, dO behind most of dV.  By way of registers, one step ahead, the rows of Q, dO and O took
//     96 of them at H = 128 and left room for two workgroups a compute unit; now three fit up to H = 96 (at H = 96 where delta is read),
//     whose prologues, exponentials and waits are covered by the others' MFMAs.  us, before -> now: H = 96 16 x 1024 x 1024
//     213 -> 187, 16 x 700 x 900 150 -> 129, causal 99.6 -> 92, 16 x 256 x 256 20.8 -> 18.3; H = 128 12 x 300 x 300 causal 31.2 -> 25,
//     16 x 4096 x 4096 3841 -> 3648; H = 64 2 x 128 x 128 7.0 -> 6.8; 170 shapes of 32 to 2500 rows 1.09 times as fast in the mean,
//     at worst 8 x 256 x 900, H = 80, 29.5 -> 31: long dQ walks with two neighbours, in parts 27.5 (plan_bwd_f32).  (The same stream of
//     MFMAs with staging through registers gave nothing: it is the third workgroup and the registers that do.)
//   - A wavefront owns 16 * RT rows and walks blocks of 16 keys (queries); the KL wavefronts of a
//     workgroup own the SAME rows and take every KL-th block of the walk ("key lanes"), because fp32
//     tiles are small: it is the walk that has to be spread over the SIMDs.  Their results are
//     merged at the end through LDS, by halves, in a fixed order (bitwise reproducible).
//   - MFMA layout (A: 16 x 4, B: 4 x 16, D: 16 x 16): lane = row of A / column of B (lane & 15), the
//     lane's group g = lane >> 4 is the contraction index; D: lane = column, register r = row
//     4 g + r.  As in the bf16 kernels the score contraction is issued transposed, so that a lane
//     holds 4 keys (4 g + r) of ONE query, and its D is the B operand of the next contraction: step r
//     contracts the keys r, 4 + r, 8 + r, 12 + r.
//   - Contractions over H read rows "naturally": lane (row l15, group g) reads the 16 bytes
//     16 y + 4 g .. + 3 of its row, which serve four MFMAs (the contraction index may be permuted as
//     long as both operands use the same permutation).
//   - Contractions over rows need the transposed operand (lane = column): lane l15 loads 16 bytes of
//     row 4 g + r, columns 64 G + 4 l15 + t, and MFMA t of the group takes one of the four, i.e. row
//     i of its result is column 64 G + 4 i + t.  A lane then holds 16 consecutive columns of the
//     result (64 G + 16 g + 4 r + t), stored as four 16-byte pieces.  (H = 96 and 80 end in a group of
//     32 or 16 columns with 8- or 4-byte pieces: Cols<H> below.)
// Measured against the vector-ALU kernels of a2d_generic.hip: 16 heads x 700 x 900, H = 96, causal,
// backward call 1034 -> 92 us; 2 heads x 128 x 128, H = 64, forward 29 -> 5.0 us; 16 heads x 4096 x 4096, H = 128: forward
// 1.04 ms (132 TFLOP/s, 84 % of the fp32 matrix peak), backward 3.65 ms (132 TFLOP/s executed).
#include <cmath>

#include "a2d_mfma.hpp"

namespace a2d {
namespace {

using mfma::gptr_t;
using mfma::row_max;
using mfma::row_sum;
using mfma::static_for;
using mfma::uniform_gptr;
using mfma::xcd_grid;
using mfma::xcd_map;

constexpr int BLK = 16;                      // rows of one step of a walk
constexpr int KL = 4;                        // key lanes (wavefronts) of a workgroup
constexpr float kRescaleThreshold = 8.0f;    // log2 units (lazy rescaling, as in the bf16 forward)

__device__ __forceinline__ f32x4 mma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
template <typename T>
__device__ __forceinline__ T gload(gptr_t base, unsigned byte_off) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(base + byte_off);
}

// Natural rows: H / 16 pieces of 16 bytes per lane
template <int H>
struct Nat {
  f32x4 v[H / 16];
  __device__ __forceinline__ void load(gptr_t base, unsigned row, unsigned row_bytes, int g4) {
    const unsigned off = __umul24(row, row_bytes) + 16 * g4;
#pragma unroll
    for (int y = 0; y < H / 16; ++y) v[y] = gload<f32x4>(base, off + 64 * y);
  }
};

// Column groups of a row for the transposed operand: H / 64 groups of 64 columns (4 per lane) and a
// rest of 32 (2 per lane) or 16 (1 per lane); T = tile index 0 .. H / 16 - 1
template <int H>
struct Cols {
  static constexpr int N4 = H / 64, REST = H % 64;
  f32x4 a[N4];
  f32x4 b;                                   // 1, 2 of it used when there is a rest
  __device__ __forceinline__ void load(gptr_t base, unsigned row, unsigned row_bytes, int l15) {
    const unsigned off = __umul24(row, row_bytes);
#pragma unroll
    for (int G = 0; G < N4; ++G) a[G] = gload<f32x4>(base, off + 256 * G + 16 * l15);
    if constexpr (REST == 32) {
      const f32x2 w = gload<f32x2>(base, off + 256 * N4 + 8 * l15);
      b[0] = w[0]; b[1] = w[1];
    }
    if constexpr (REST == 16) b[0] = gload<float>(base, off + 256 * N4 + 4 * l15);
  }
  template <int T>
  __device__ __forceinline__ float get() const {
    if constexpr (T < 4 * N4) return a[T / 4][T % 4]; else return b[T - 4 * N4];
  }
};

typedef __attribute__((address_space(3))) char* lds_t;
template <typename T>
__device__ __forceinline__ T lload(lds_t p) { return *reinterpret_cast<__attribute__((address_space(3))) T*>(p); }
template <typename T>
__device__ __forceinline__ void lstore(lds_t p, T v) { *reinterpret_cast<__attribute__((address_space(3))) T*>(p) = v; }

// A wavefront's tile of 16 rows that is loaded straight into LDS (see mfma::Blocks16: here a block is 16 rows x 16 columns).
// Blocks lie 64 bytes more than their size apart, so that the columns' reads, which take 64 bytes of four blocks at a time,
// meet every bank once too.  (Not so those of the last 32 columns at H = 96, which meet half of the banks twice, and of the last 16 at
// H = 80, a quarter four times: 10 % of the kernel's LDS cycles at H = 96.)
template <int H>
struct Blocks {
  static constexpr int N = H / 16, N4 = Cols<H>::N4, REST = Cols<H>::REST, STRIDE = mfma::BLOCK + 64, BYTES = N * STRIDE;
  lds_t base, nat, col, rest;                // + this lane's place for natural rows, for columns (row 4 g), for the last ones
  __device__ __forceinline__ void init(lds_t b, int l15, int g4) {
    const int swap = mfma::block_swap(g4);
    base = b;
    nat = b + l15 * 64 + 16 * (g4 ^ mfma::block_swap(l15 >> 2));
    col = b + (l15 >> 2) * STRIDE + 256 * g4 + 16 * ((l15 & 3) ^ swap);
    rest = b + 4 * N4 * STRIDE + 256 * g4 +
           (REST == 32 ? (l15 >> 3) * STRIDE + 16 * ((l15 >> 1 & 3) ^ swap) + 8 * (l15 & 1) : 16 * ((l15 >> 2) ^ swap) + 4 * (l15 & 3));
  }
  // lane i's row i >> 2 of the tile is at byte `off` of from; + chunk(i)
  static __device__ __forceinline__ unsigned chunk(int lane) { return 16 * ((lane & 3) ^ mfma::block_swap(lane >> 4)); }
  __device__ __forceinline__ void load(gptr_t from, unsigned off) const {
    static_for<0, N>([&](auto Y) {
      constexpr int y = decltype(Y)::value;
      mfma::dma_b128<64 * y>((unsigned)(uintptr_t)base + y * STRIDE, from, off);
    });
  }
  __device__ __forceinline__ f32x4 row(int y) const { return lload<f32x4>(nat + y * STRIDE); }
  // what this lane has loaded
  __device__ __forceinline__ f32x4 own(int y, int lane) const { return lload<f32x4>(base + y * STRIDE + 16 * lane); }
  __device__ __forceinline__ void cols(Cols<H>& c, int r) const {
#pragma unroll
    for (int G = 0; G < N4; ++G) c.a[G] = lload<f32x4>(col + 64 * r + 4 * G * STRIDE);
    if constexpr (REST == 32) {
      const f32x2 w = lload<f32x2>(rest + 64 * r);
      c.b[0] = w[0]; c.b[1] = w[1];
    }
    if constexpr (REST == 16) c.b[0] = lload<float>(rest + 64 * r);
  }
};
// before a load into a tile that has been read
__device__ __forceinline__ void reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// D layout of the transposed results: acc[T][r] is column col<T>(g, r) of the lane's row (l15)
template <int H>
struct Out {
  f32x4 acc[H / 16];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int t = 0; t < H / 16; ++t) acc[t] = zero4();
  }
  __device__ __forceinline__ void scale(float f) {
#pragma unroll
    for (int t = 0; t < H / 16; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[t][r] *= f;
  }
  // The 16-byte pieces of the lane's row: f(column, four places (t, r) of the accumulators)
  template <class F>
  __device__ __forceinline__ void pieces(int g4, F&& f) {
    constexpr int N4 = Cols<H>::N4, REST = Cols<H>::REST;
#pragma unroll
    for (int G = 0; G < N4; ++G)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        f(64 * G + 16 * g4 + 4 * r, [=](int e) { return 4 * G + e; }, [=](int) { return r; });
    if constexpr (REST == 32) {
#pragma unroll
      for (int r = 0; r < 4; r += 2)
        f(64 * N4 + 8 * g4 + 2 * r, [=](int e) { return 4 * N4 + (e & 1); }, [=](int e) { return r + (e >> 1); });
    }
    if constexpr (REST == 16) f(64 * N4 + 4 * g4, [=](int) { return 4 * N4; }, [=](int e) { return e; });
  }
  __device__ __forceinline__ void store(float* row, int g4, float mul, bool add = false) {
    pieces(g4, [&](int col, auto t, auto r) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[t(e)][r(e)] * mul;
      if (add) {
        const f32x4 o = *reinterpret_cast<const f32x4*>(row + col);
        v[0] += o[0]; v[1] += o[1]; v[2] += o[2]; v[3] += o[3];
      }
      *reinterpret_cast<f32x4*>(row + col) = v;
    });
  }
  __device__ __forceinline__ void load(const float* row, int g4) {
    pieces(g4, [&](int col, auto t, auto r) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(row + col);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t(e)][r(e)] = v[e];
    });
  }
  // acc += rows^T * b over the 4 rows (one per group) `c` holds
  __device__ __forceinline__ void contract(const Cols<H>& c, float b) {
    static_for<0, H / 16>([&](auto T) {
      constexpr int t = decltype(T)::value;
      acc[t] = mma4(c.template get<t>(), b, acc[t]);
    });
  }
};

// 16 x 16 results of contractions over H of a tile's rows with RT sets of rows in registers (two
// accumulators each).  The tile's pieces are requested one ahead of their use.
template <int H, int RT>
__device__ __forceinline__ void dot_rows(f32x4 (&out)[RT], const Blocks<H>& a, const Nat<H> (&b)[RT]) {
  constexpr int N = H / 16;
  f32x4 s1[RT], ring[2];
#pragma unroll
  for (int t = 0; t < RT; ++t) { out[t] = zero4(); s1[t] = zero4(); }
  ring[0] = a.row(0);
  ring[1] = a.row(1);
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, N>([&](auto Y) {
    constexpr int y = decltype(Y)::value;
    const f32x4 v = ring[y & 1];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      out[t] = mma4(v[0], b[t].v[y][0], out[t]);
      s1[t] = mma4(v[1], b[t].v[y][1], s1[t]);
      out[t] = mma4(v[2], b[t].v[y][2], out[t]);
      s1[t] = mma4(v[3], b[t].v[y][3], s1[t]);
    }
    if constexpr (y + 2 < N) ring[y & 1] = a.row(y + 2);
    __builtin_amdgcn_sched_barrier(0);
  });
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) out[t][r] += s1[t][r];
}

// The backward's two contractions over H of a step, s = rows of `a` . fa and d = rows of `b` . fb, as one stream of MFMAs: the
// tiles' pieces are requested two ahead of their use across the seam (`seam()`: before b's first), and what `between(y)` does
// behind the MFMAs of d's piece y (s is complete from y = 1 on) runs while they do.
template <int H, class S, class F>
__device__ __forceinline__ void dot_two(f32x4& s, f32x4& d, const Blocks<H>& a, const Nat<H>& fa, const Blocks<H>& b,
                                        const Nat<H>& fb, S&& seam, F&& between) {
  constexpr int N = H / 16;
  f32x4 acc[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}}, ring[2] = {a.row(0), a.row(1)};
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, 2 * N>([&](auto I) {
    constexpr int i = decltype(I)::value, of = i / N, y = i % N, next = i + 2;
    const f32x4 v = ring[i & 1];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[of][e & 1] = mma4(v[e], (of ? fb : fa).v[y][e], acc[of][e & 1]);
    if constexpr (next == N) seam();
    if constexpr (next < 2 * N) ring[i & 1] = next < N ? a.row(next) : b.row(next - N);
    if constexpr (i == N + 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = acc[0][0][r] + acc[0][1][r];
    }
    if constexpr (of == 1) between(std::integral_constant<int, y>{});
    __builtin_amdgcn_sched_barrier(0);
  });
#pragma unroll
  for (int r = 0; r < 4; ++r) d[r] = acc[1][0][r] + acc[1][1][r];
}

// Sum of N results over the KL wavefronts of the workgroup, by halves: the upper half writes, the
// lower half adds; wavefront 0 ends up with the total.  xch: KL / 2 areas of N * 64 16-byte pieces.
template <int N, class Get>
__device__ __forceinline__ void merge_lanes(f32x4* xch, int kl, int lane, Get&& get) {
#pragma unroll
  for (int half = KL / 2; half >= 1; half /= 2) {
    __syncthreads();
    if (kl >= half && kl < 2 * half) {
#pragma unroll
      for (int i = 0; i < N; ++i) xch[((kl - half) * N + i) * 64 + lane] = get(i);
    }
    __syncthreads();
    if (kl < half) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const f32x4 v = xch[(kl * N + i) * 64 + lane];
        f32x4& a = get(i);
        a[0] += v[0]; a[1] += v[1]; a[2] += v[2]; a[3] += v[3];
      }
    }
  }
}

// The walk over the 16-key blocks that some row of the workgroup sees, sub-block by sub-block; key
// lane kl takes every KL-th block.  (s == g.n: past the end)
// The current sub-block's entry is kept in registers: read from the kernel arguments in every step it
// would be scalar loads, which share a wait counter with the LDS operations in flight.
struct Walk {
  int s, j, nblk;
  int start, rows;                           // of the sub-block
  template <class SegBlocks>
  __device__ __forceinline__ void find(const SegList& g, SegBlocks&& blocks) {   // from sub-block s on
    while (s < g.n && (nblk = blocks(s)) == 0) ++s;
    if (s < g.n) { start = g.seg[s].start; rows = g.seg[s].rows; }
  }
  template <class SegBlocks>
  __device__ __forceinline__ void open(const SegList& g, SegBlocks&& blocks) {
    s = 0; j = 0; nblk = start = rows = 0;
    find(g, blocks);
  }
  template <class SegBlocks>
  __device__ __forceinline__ void advance(int by, const SegList& g, SegBlocks&& blocks) {
    j += by;
    while (s < g.n && j >= nblk) {
      j -= nblk;
      ++s;
      find(g, blocks);
    }
  }
};

// workgroup -> (head, first row, part of the walk): as in the bf16 kernels the row blocks of the query
// heads that share a key/value head are placed together, late (heavy) blocks first
__device__ __forceinline__ bool query_block(int id, const a2d_tile_desc& d, const SegList& g, int parts, int rows,
                                            int& head, int& q0, int& part) {
  const int nqb = (d.nq + rows - 1) / rows;
  int unit, blk;
  if (!xcd_map(id, d.heads / g.group * parts, g.group * nqb, g.by_size != 0, unit, blk)) return false;
  const mfma::Split up = mfma::split_by(unit, parts), in_group = mfma::query_head(blk, g.group, nqb, g.by_size != 0);
  part = up.r;
  head = up.q * g.group + in_group.r;
  q0 = (nqb - 1 - in_group.q) * rows;
  return true;
}

__device__ __forceinline__ int vis_count(const a2d_tile_desc& d, const SegList& g, int i, int s) {
  if (!d.causal) return g.seg[s].rows;
  const int64_t v = (int64_t)i + g.seg[s].rel + 1;
  return v <= 0 ? 0 : (v < g.seg[s].rows ? (int)v : g.seg[s].rows);
}

// ------------------------------------------------------------------ forward
// (O_part, m_out and l_out are not __restrict__: an accumulating call's `in` is the same memory)
// workgroups of the forward that a compute unit holds at a time, by their registers (three of 32 rows at H = 96 kept six in scratch)
constexpr int fwd_fit(int hdim, int rt) { return rt == 2 ? (hdim <= 80 ? 3 : 2) : hdim == 128 ? 3 : 4; }
template <int H, int RT>
__global__ __launch_bounds__(64 * KL) __attribute__((amdgpu_waves_per_eu(fwd_fit(H, RT)))) void fwd_f32_kernel(
    a2d_tile_desc d, SegList g, const float* __restrict__ Q, const float* __restrict__ K,
    const float* __restrict__ V, float* O_part, float* m_out, float* l_out, FwdInput in) {
  warm_arguments<6 * 8 + sizeof(FwdInput)>();
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int head, q0, part;
  if (!query_block(blockIdx.x, d, g, g.parts, BLK * RT, head, q0, part)) return;
  const int lanes = KL * g.parts;
  const int kl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l15 = lane & 15, g4 = lane >> 4;
  const int kvh = mfma::split_by(head, g.group).q;
  const gptr_t kb = uniform_gptr(K + (int64_t)kvh * d.lk.head), vb = uniform_gptr(V + (int64_t)kvh * d.lv.head);
  const gptr_t qb = uniform_gptr(Q + (int64_t)head * d.lq.head);
  const unsigned k_row = (unsigned)d.lk.row * 4, v_row = (unsigned)d.lv.row * 4;
  const float c = d.scale * kLog2e;

  Nat<H> qf[RT];
  Out<H> o[RT];
  float m_lane[RT], m_ref[RT], l_run[RT];
  int q_row[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    q_row[t] = q0 + BLK * t + l15;
    qf[t].load(qb, min(q_row[t], d.nq - 1), (unsigned)d.lq.row * 4, g4);
    o[t].zero();
    m_lane[t] = -INFINITY;
    l_run[t] = 0.f;
    if (g.acc && kl == 0 && part == 0 && q_row[t] < d.nq) {     // continue from the triple given
      const int64_t row = (int64_t)head * d.nq + q_row[t];
      o[t].load(in.N + row * H, g4);
      m_lane[t] = in.m[row] / d.scale;             // -inf stays -inf
      l_run[t] = g4 == 0 ? in.l[row] : 0.f;
    }
    m_ref[t] = m_lane[t];
  }

  const int blk_last = min(q0 + BLK * RT, d.nq) - 1;
  auto seg_blocks = [&](int s) { return (vis_count(d, g, blk_last, s) + BLK - 1) / BLK; };
  Walk w;
  w.open(g, seg_blocks);
  w.advance(part * KL + kl, g, seg_blocks);
  // K comes in through LDS, the next block's as soon as the scores are there; V by columns into registers, the next block's as
  // soon as the products are through.  (Past the walk's end a block of K is read again, which is there before the products are through,
  // and none of V, which would be waited for: 3 x 130 x 64, H = 128 5.6 -> 5.5 us, 6 x 491 x 355 11.9 -> 11.8; without that of K either the loop of
  // longer walks is 1 % slower.  In the 32-row form the scores wait for V already, since the compiler takes the second tile of Q as possibly
  // under way in every step; a loop entered and gone round behind requests alone has no such wait, and is 1 to 2 % slower at H = 64 and 80.)
  Blocks<H> kt;
  kt.init((lds_t)smem + kl * Blocks<H>::BYTES, l15, g4);
  Cols<H> vt[4];
  constexpr int V_LOADS = 4 * (Cols<H>::N4 + (Cols<H>::REST != 0));
  auto load_k = [&]() {
    kt.load(kb, __umul24((unsigned)(w.start + min(w.j * BLK + (lane >> 2), w.rows - 1)), k_row) + Blocks<H>::chunk(lane));
  };
  auto load_v = [&]() {
#pragma unroll
    for (int r = 0; r < 4; ++r) vt[r].load(vb, w.start + min(w.j * BLK + 4 * g4 + r, w.rows - 1), v_row, l15);
  };
  int vis_s = -1, my_vis[RT];                         // keys of sub-block vis_s that this lane's rows see
  if (w.s < g.n) {
    load_k();
    load_v();
  }
  while (w.s < g.n) {
    const int k0 = w.j * BLK;
    if (w.s != vis_s) {
      vis_s = w.s;
#pragma unroll
      for (int t = 0; t < RT; ++t) my_vis[t] = vis_count(d, g, min(q_row[t], d.nq - 1), w.s);
    }
    f32x4 p[RT];
    mfma::wait_dma<V_LOADS>();
    __builtin_amdgcn_sched_barrier(0);
    dot_rows<H, RT>(p, kt, qf);
    w.advance(lanes, g, seg_blocks);
    mfma::wait_vmem_all();                            // V: the products would wait for the next block's K too
    reads_done();
    load_k();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (k0 + 4 * g4 + r >= my_vis[t]) p[t][r] = -INFINITY;
        m_lane[t] = fmaxf(m_lane[t], p[t][r]);
      }
      // (m_lane - m_ref) is +inf on the first visible block, NaN (-> false) while nothing is visible
      const bool grow = (m_lane[t] - m_ref[t]) * c > kRescaleThreshold;
      if (__builtin_amdgcn_ballot_w64(grow) != 0) {
        const float m_row = row_max(m_lane[t]);
        const float alpha = m_ref[t] == -INFINITY ? 0.f : fast_exp2((m_ref[t] - m_row) * c);
        m_ref[t] = m_row;
        l_run[t] *= alpha;
        o[t].scale(alpha);
      }
      const float mr = m_ref[t] == -INFINITY ? 0.f : m_ref[t];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[t][r] = fast_exp2((p[t][r] - mr) * c);
        l_run[t] += p[t][r];
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int t = 0; t < RT; ++t) o[t].contract(vt[r], p[t][r]);
    __builtin_amdgcn_sched_barrier(0);
    if (w.s < g.n) load_v();
  }
  mfma::wait_vmem_all();                              // (the K tile's place is written over below)

  // ---- to the true row maximum over all key lanes, then the sums over the lanes
  float m_all[RT];
  float* stat = reinterpret_cast<float*>(smem);      // [kl][t][16]
#pragma unroll
  for (int t = 0; t < RT; ++t) m_all[t] = row_max(m_lane[t]);
  __syncthreads();                                   // (the tiles are written over)
#pragma unroll
  for (int t = 0; t < RT; ++t)
    if (g4 == 0) stat[(kl * RT + t) * 16 + l15] = m_all[t];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int x = 0; x < KL; ++x) m_all[t] = fmaxf(m_all[t], stat[(x * RT + t) * 16 + l15]);
  f32x4 lsum[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const float f = m_ref[t] == -INFINITY ? 0.f : fast_exp2((m_ref[t] - m_all[t]) * c);
    o[t].scale(f);
    lsum[t] = f32x4{row_sum(l_run[t]) * f, 0.f, 0.f, 0.f};
  }
  merge_lanes<RT * (H / 16 + 1)>(reinterpret_cast<f32x4*>(smem), kl, lane, [&](int i) -> f32x4& {
    return i < RT ? lsum[i] : o[(i - RT) / (H / 16)].acc[(i - RT) % (H / 16)];
  });
  if (kl != 0) return;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (q_row[t] >= d.nq) continue;
    const int64_t row = ((int64_t)part * d.heads + head) * d.nq + q_row[t];
    const float l = lsum[t][0];
    if (g.norm) {                                     // O' = N / l, lse' = m + ln l
      o[t].store(O_part + row * H, g4, l > 0.f ? 1.0f / l : 0.f);
      if (g4 == 0) m_out[row] = l > 0.f ? m_all[t] * d.scale + logf(l) : -INFINITY;
    } else {
      o[t].store(O_part + row * H, g4, 1.0f);
      if (g4 == 0) { m_out[row] = m_all[t] * d.scale; l_out[row] = l; }
    }
  }
}

// ---------------------------------------------------------------- backward: dQ (and delta)
// Owns 16 query rows per workgroup.  Also computes delta = rowsum(dO o O) of its rows (every key lane
// for itself): no separate pass over O and dO.
template <int H>
__device__ __forceinline__ void dq_rows(int id, char* const smem, const a2d_tile_desc& d, const SegList& g,
                                        const int parts, const float* __restrict__ Q, const float* __restrict__ K,
                                        const float* __restrict__ V, const float* __restrict__ O,
                                        const float* __restrict__ dO, const float* __restrict__ lse,
                                        float* __restrict__ dQ) {
  int head, q0, part;
  if (!query_block(id, d, g, parts, BLK, head, q0, part)) return;
  const int lanes = KL * parts;
  const int kl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l15 = lane & 15, g4 = lane >> 4;
  const int kvh = mfma::split_by(head, g.group).q;
  const gptr_t kb = uniform_gptr(K + (int64_t)kvh * d.lk.head), vb = uniform_gptr(V + (int64_t)kvh * d.lv.head);
  const unsigned k_row = (unsigned)d.lk.row * 4, v_row = (unsigned)d.lv.row * 4;
  const int q_row = q0 + l15, q_ld = min(q_row, d.nq - 1);

  Nat<H> qf, gf, of;
  qf.load(uniform_gptr(Q + (int64_t)head * d.lq.head), q_ld, (unsigned)d.lq.row * 4, g4);
  gf.load(uniform_gptr(dO + (int64_t)head * d.ldo.head), q_ld, (unsigned)d.ldo.row * 4, g4);
  of.load(uniform_gptr(O + (int64_t)head * d.lo.head), q_ld, (unsigned)d.lo.row * 4, g4);     // for delta only
  const float lse_i = q_row < d.nq ? lse[(int64_t)head * d.nq + q_ld] : -INFINITY;
  float del = 0.f;
#pragma unroll
  for (int y = 0; y < H / 16; ++y)
#pragma unroll
    for (int e = 0; e < 4; ++e) del = fmaf(gf.v[y][e], of.v[y][e], del);
  del = row_sum(del);

  const int blk_last = min(q0 + BLK, d.nq) - 1;
  auto seg_blocks = [&](int s) { return (vis_count(d, g, blk_last, s) + BLK - 1) / BLK; };
  Walk w;
  w.open(g, seg_blocks);
  w.advance(part * KL + kl, g, seg_blocks);
  Out<H> dq;
  dq.zero();
  Blocks<H> kt, vt;
  kt.init((lds_t)smem + 2 * kl * Blocks<H>::BYTES, l15, g4);
  vt.init((lds_t)smem + (2 * kl + 1) * Blocks<H>::BYTES, l15, g4);
  const auto load = [&](const Blocks<H>& to, gptr_t from, unsigned row_bytes) {
    to.load(from, __umul24((unsigned)(w.start + min(w.j * BLK + (lane >> 2), w.rows - 1)), row_bytes) + Blocks<H>::chunk(lane));
  };
  if (w.s < g.n) {
    load(kt, kb, k_row);
    load(vt, vb, v_row);
  }
  int vis_s = -1, my_vis = 0;                         // keys of sub-block vis_s that this lane's row sees
  Cols<H> ring[2];
  while (w.s < g.n) {
    const int k0 = w.j * BLK;
    if (w.s != vis_s) { vis_s = w.s; my_vis = vis_count(d, g, q_ld, w.s); }
    f32x4 p, ds;
    mfma::wait_dma();
    dot_two<H>(p, ds, kt, qf, vt, gf, [] {}, [&](auto Y) {
      constexpr int y = decltype(Y)::value;
      if constexpr (y == 1 || y == 2) {
#pragma unroll
        for (int r = 2 * y - 2; r < 2 * y; ++r) {
          const bool vis = lse_i != -INFINITY && k0 + 4 * g4 + r < my_vis;
          p[r] = vis ? fast_exp2(fmaf(p[r], d.scale, -lse_i) * kLog2e) : 0.f;
        }
      }
      if constexpr (y >= H / 16 - 2) kt.cols(ring[y - (H / 16 - 2)], y - (H / 16 - 2));
    });
    // the next tiles come in as soon as the pieces of these have been read: V behind dP, K behind half of the last contraction
    reads_done();
    w.advance(lanes, g, seg_blocks);
    const bool more = w.s < g.n;
    if (more) load(vt, vb, v_row);
#pragma unroll
    for (int r = 0; r < 4; ++r) ds[r] = p[r] * (ds[r] - del);
    static_for<0, 4>([&](auto R) {
      constexpr int r = decltype(R)::value;
      dq.contract(ring[r & 1], ds[r]);
      if constexpr (r < 2) kt.cols(ring[r & 1], r + 2);
      if constexpr (r == 2) {
        reads_done();
        if (more) load(kt, kb, k_row);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  merge_lanes<H / 16>(reinterpret_cast<f32x4*>(smem), kl, lane, [&](int i) -> f32x4& { return dq.acc[i]; });
  if (kl != 0) return;
  if (q_row < d.nq) {
    float* row = dQ + (((int64_t)part * d.heads + head) * d.nq + q_row) * H;
    dq.store(row, g4, d.scale, g.acc != 0);
  }
}

// ---------------------------------------------------------------- backward: dK, dV
// Owns 16 keys of a key/value head per workgroup and walks the query rows of all its group's query
// heads, 16 at a time: S = Q K^T and dP = dO V^T leave a lane holding 4 queries of ONE key.  OWN_DELTA: delta of the step's
// rows from those of O, which come in beside those of dO (lane: the same columns of the same rows); else it is read.
template <int H, bool OWN_DELTA>
__device__ __forceinline__ void dkdv_keys(int id, char* const smem, const a2d_tile_desc& d, const SegList& g,
                                          const int parts, const float* __restrict__ Q, const float* __restrict__ K,
                                          const float* __restrict__ V, const float* __restrict__ O,
                                          const float* __restrict__ dO, const float* __restrict__ lse,
                                          const float* __restrict__ delta, float* __restrict__ dK,
                                          float* __restrict__ dV) {
  int head, blk;                                      // key/value head
  if (!xcd_map(id, d.heads / g.group * parts, (d.nkv + BLK - 1) / BLK, g.by_size != 0, head, blk)) return;
  const int lanes = KL * parts;
  const mfma::Split up = mfma::split_by(head, parts);
  head = up.q;
  const int part = up.r;
  const int kl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l15 = lane & 15, g4 = lane >> 4;
  const int k0 = blk * BLK, key = k0 + l15, k_ld = min(key, d.nkv - 1);
  const gptr_t qb = uniform_gptr(Q + (int64_t)head * g.group * d.lq.head);
  const gptr_t gb = uniform_gptr(dO + (int64_t)head * g.group * d.ldo.head);
  const float* lse_b = lse + (int64_t)head * g.group * d.nq;
  const float* del_b = OWN_DELTA ? nullptr : delta + (int64_t)head * g.group * d.nq;
  const gptr_t ob = uniform_gptr(O + (int64_t)head * g.group * d.lo.head);
  const unsigned q_row = (unsigned)d.lq.row * 4, g_row = (unsigned)d.ldo.row * 4, o_row = (unsigned)d.lo.row * 4;
  const unsigned q_head = (unsigned)d.lq.head * 4, g_head = (unsigned)d.ldo.head * 4, o_head = (unsigned)d.lo.head * 4;

  Nat<H> kf, vf;
  kf.load(uniform_gptr(K + (int64_t)head * d.lk.head), k_ld, (unsigned)d.lk.row * 4, g4);
  vf.load(uniform_gptr(V + (int64_t)head * d.lv.head), k_ld, (unsigned)d.lv.row * 4, g4);

  // first query row that sees this lane's key, and the first that sees any of the block's keys
  auto first_row = [&](int s, int k) -> int {
    const int64_t f = (int64_t)(k - g.seg[s].start) - g.seg[s].rel;
    return f <= 0 ? 0 : (f >= d.nq ? d.nq : (int)f);
  };
  int my_first = 0, i_first = 0;
  if (d.causal) {
    my_first = i_first = d.nq;
    for (int s = 0; s < g.n; ++s) {
      const int a = max(k0, g.seg[s].start), b = min(k0 + BLK, g.seg[s].start + g.seg[s].rows);
      if (a < b) i_first = min(i_first, first_row(s, a));
      if (key >= g.seg[s].start && key < g.seg[s].start + g.seg[s].rows) my_first = first_row(s, key);
    }
  }
  if (key >= d.nkv) my_first = d.nq;                  // padding keys see nothing
  const int b0 = i_first / BLK, nblk = (d.nq + BLK - 1) / BLK - b0;
  const int total = nblk * g.group;                   // the group's query heads one after the other

  Out<H> dk, dv;
  dk.zero();
  dv.zero();
  Blocks<H> qt, gt;
  qt.init((lds_t)smem + 2 * kl * Blocks<H>::BYTES, l15, g4);
  gt.init((lds_t)smem + (2 * kl + 1) * Blocks<H>::BYTES, l15, g4);
  f32x4 oc[OWN_DELTA ? H / 16 : 1];                   // of the step to come: O where dO goes, and the rows' statistics
  float ln[4], dn[4];
  // position of walk step n: query head (inside the group) and first row
  const int n0 = part * KL + kl;
  int qh = 0, rb = n0;                                // of the next step to be loaded
  auto wrap = [&]() { while (rb >= nblk && qh < g.group) { rb -= nblk; ++qh; } };
  if (nblk > 0) wrap();
  auto off = [&](unsigned head_bytes, unsigned row_bytes) {
    const int ln = mfma::lane_again();
    return qh * head_bytes + __umul24((unsigned)min((b0 + rb) * BLK + (ln >> 2), d.nq - 1), row_bytes) + Blocks<H>::chunk(ln);
  };
  auto load_stats = [&]() {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const unsigned row = min((b0 + rb) * BLK + 4 * g4 + r, d.nq - 1);
      if constexpr (!OWN_DELTA) dn[r] = del_b[qh * d.nq + row];
      ln[r] = lse_b[qh * d.nq + row];
    }
    if constexpr (OWN_DELTA) {
      const unsigned at = off(o_head, o_row);
#pragma unroll
      for (int y = 0; y < H / 16; ++y) oc[y] = gload<f32x4>(ob, at + 64 * y);
    }
  };
  if (n0 < total) {
    load_stats();
    qt.load(qb, off(q_head, q_row));
    gt.load(gb, off(g_head, g_row));
  }
  Cols<H> ring[2];
  for (int n = n0; n < total; n += lanes) {
    const bool more = n + lanes < total;
    const int i0 = (b0 + rb) * BLK;
    float ls[4], de[4];
    f32x4 p, ds;
    mfma::wait_dma<H / 16>();                         // Q, and the statistics
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      ls[r] = ln[r];
      if constexpr (!OWN_DELTA) de[r] = dn[r];
    }
    f32x4 own;
    float del = 0.f;
    auto own_delta = [&](int y) {
#pragma unroll
      for (int e = 0; e < 4; ++e) del = fmaf(own[e], oc[y][e], del);
    };
    dot_two<H>(p, ds, qt, kf, gt, vf, [] { mfma::wait_dma(); }, [&](auto Y) {
      constexpr int y = decltype(Y)::value;
      if constexpr (OWN_DELTA) {                      // of row lane >> 2, a piece at a time
        if constexpr (y > 0) own_delta(y - 1);
        own = gt.own(y, mfma::lane_again());
      }
      if constexpr (y == 1 || y == 2) {
#pragma unroll
        for (int r = 2 * y - 2; r < 2 * y; ++r) {
          const int i = i0 + 4 * g4 + r;
          const bool vis = i < d.nq && i >= my_first && ls[r] != -INFINITY;
          p[r] = vis ? fast_exp2(fmaf(p[r], d.scale, -ls[r]) * kLog2e) : 0.f;
        }
      }
      if constexpr (y >= H / 16 - 2) qt.cols(ring[y - (H / 16 - 2)], y - (H / 16 - 2));
    });
    if constexpr (OWN_DELTA) {                        // the row's sum in all four of its lanes, then those of rows 4 g + r
      own_delta(H / 16 - 1);
      del += mfma::lane_swap<0xB1>(del);
      del += mfma::lane_swap<0x4E>(del);
      static_for<0, 4>([&](auto R) { de[decltype(R)::value] = mfma::lane_swap<0x150 + 4 * decltype(R)::value>(del); });
    }
    rb += lanes;
    wrap();
    if (more) load_stats();
#pragma unroll
    for (int r = 0; r < 4; ++r) ds[r] = p[r] * (ds[r] - de[r]);
    static_for<0, 8>([&](auto R) {                    // dK, dV; the next tiles as in dq_rows, Q behind most of dV
      constexpr int r = decltype(R)::value, next = r + 2;
      if constexpr (r < 4) dk.contract(ring[r & 1], ds[r]); else dv.contract(ring[r & 1], p[r - 4]);
      if constexpr (r == 2 || r == 6) {
        reads_done();
        if (more) {
          if constexpr (r == 2) qt.load(qb, off(q_head, q_row)); else gt.load(gb, off(g_head, g_row));
        }
      }
      if constexpr (next < 8) (next < 4 ? qt : gt).cols(ring[r & 1], next & 3);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  merge_lanes<H / 8>(reinterpret_cast<f32x4*>(smem), kl, lane, [&](int i) -> f32x4& {
    return i < H / 16 ? dk.acc[i] : dv.acc[i - H / 16];
  });
  if (kl != 0) return;
  if (key < d.nkv) {
    const int64_t row = ((int64_t)part * (d.heads / g.group) + head) * d.nkv + key;
    dk.store(dK + row * H, g4, d.scale);
    dv.store(dV + row * H, g4, 1.0f);
  }
}

// workgroups of the backward that a compute unit holds at a time (a wavefront of each on every SIMD)
constexpr int bwd_fit(int hdim, bool own_delta) { return hdim < 96 || (hdim == 96 && !own_delta) ? 3 : 2; }
// The two kinds of workgroups in one launch, `first` of the kind with the longer walks before the others (see
// a2d_bwd_one.hip; here always: fp32 tiles are small).
template <int H, bool OWN_DELTA>
__global__ __launch_bounds__(64 * KL) __attribute__((amdgpu_waves_per_eu(bwd_fit(H, OWN_DELTA)))) void bwd_f32_kernel(
    a2d_tile_desc d, SegList g, const float* __restrict__ Q, const float* __restrict__ K,
    const float* __restrict__ V, const float* __restrict__ O, const float* __restrict__ dO,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dQ, float* __restrict__ dK,
    float* __restrict__ dV, int first, int q_first, int parts_q) {
  warm_arguments<10 * 8 + 12>();
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int id = (int)blockIdx.x < first ? blockIdx.x : blockIdx.x - first;
  if (((int)blockIdx.x < first) == (q_first != 0)) dq_rows<H>(id, smem, d, g, parts_q, Q, K, V, O, dO, lse, dQ);
  else dkdv_keys<H, OWN_DELTA>(id, smem, d, g, g.parts, Q, K, V, O, dO, lse, delta, dK, dV);
}

// LDS of a workgroup: the wavefronts' tiles, over which their results are merged at the end
constexpr int most(int a, int b) { return a > b ? a : b; }
template <int H, int RT>
constexpr int fwd_lds() { return most(KL * Blocks<H>::BYTES, KL / 2 * RT * (H / 16 + 1) * 1024); }
template <int H>
constexpr int dq_lds() { return most(2 * KL * Blocks<H>::BYTES, KL / 2 * (H / 16) * 1024); }
template <int H>
constexpr int dkdv_lds() { return most(2 * KL * Blocks<H>::BYTES, KL / 2 * (H / 8) * 1024); }
static_assert(fwd_lds<128, 2>() <= 80 * 1024, "two workgroups of the forward per compute unit");
static_assert(most(dkdv_lds<128>(), dq_lds<128>()) * bwd_fit(128, false) <= 160 * 1024 &&
              most(dkdv_lds<96>(), dq_lds<96>()) * bwd_fit(96, false) <= 160 * 1024, "bwd_fit workgroups per compute unit");

template <int H, int RT>
hipError_t fwd_go(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                  float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  constexpr int lds = fwd_lds<H, RT>(), rows = BLK * RT;
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(fwd_f32_kernel<H, RT>), lds);
  if (e != hipSuccess) return e;
  dim3 grid(xcd_grid(d.heads / g.group * g.parts, g.group * ((d.nq + rows - 1) / rows))), block(64 * KL);
  A2D_LAUNCH((fwd_f32_kernel<H, RT>), grid, block, lds, s, d, g, (const float*)Q, (const float*)K,
             (const float*)V, O_part, m, l, in);
  return hipGetLastError();
}

enum { F32_ROWS16 = 0, F32_ROWS32 = 1 };

template <int H>
hipError_t fwd_h(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                 float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  return g.form == F32_ROWS32 ? fwd_go<H, 2>(d, g, Q, K, V, O_part, m, l, in, s)
                              : fwd_go<H, 1>(d, g, Q, K, V, O_part, m, l, in, s);
}

template <int H, bool OWN_DELTA>
hipError_t bwd_go(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                  const void* O, const void* dO, const float* lse, float* delta, float* dQ, float* dK, float* dV,
                  const BwdParts& parts, hipStream_t s) {
  SegList go = g;
  if (parts.q > 1) go.acc = 0;                       // (the sum over the parts adds)
  go.parts = parts.kv;
  constexpr int lds = most(dq_lds<H>(), dkdv_lds<H>());
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_f32_kernel<H, OWN_DELTA>), lds);
  if (e == hipSuccess && !OWN_DELTA) e = launch_delta(d, O, dO, delta, s);
  if (e != hipSuccess) return e;
  const int n_q = xcd_grid(d.heads / g.group * parts.q, g.group * ((d.nq + BLK - 1) / BLK));
  const int n_kv = xcd_grid(d.heads / g.group * parts.kv, (d.nkv + BLK - 1) / BLK);
  A2D_LAUNCH((bwd_f32_kernel<H, OWN_DELTA>), dim3(n_q + n_kv), dim3(64 * KL), lds, s, d, go, (const float*)Q,
             (const float*)K, (const float*)V, (const float*)O, (const float*)dO, lse, delta, dQ, dK, dV,
             parts.q_first ? n_q : n_kv, parts.q_first, parts.q);
  return hipGetLastError();
}
template <int H>
hipError_t bwd_h(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                 const void* O, const void* dO, const float* lse, float* delta, float* dQ, float* dK, float* dV,
                 const BwdParts& parts, hipStream_t s) {
  return parts.delta ? bwd_go<H, false>(d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s)
                     : bwd_go<H, true>(d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
}

// Numbers of parts that are tried, and what they cost beside the walks: a launch behind the tile's
constexpr int kParts[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
constexpr double kSumUs = 5.0, kPartUs = 0.2;
// H = 64, 80, 96, 128
int head_index(int hdim) { return hdim > 96 ? 3 : hdim > 80 ? 2 : hdim > 64 ? 1 : 0; }
// A workgroup of KL wavefronts that walks `steps` steps in `parts` parts, whole steps at the most, some half a step more than
// their share in the mean of an uneven walk
Kind f32_kind(int64_t blocks, double mean, double most, int parts, bool uneven, double step, double fixed) {
  const auto whole = [](double n) { return n <= 1 ? 1.0 : std::ceil(n - 1e-9); };
  const double z = (double)KL * parts, m = uneven ? mean / z + 0.4 : whole(mean / z);
  return Kind{blocks * parts, (m < 1 ? 1 : m) * step + fixed, whole(most / z) * step + fixed};
}

}  // namespace

// 32 rows per workgroup halve the operand traffic per MFMA; 16 rows when those come to fewer than
// four workgroups per compute unit
void plan_fwd_f32(const a2d_tile_desc& d, SegList* g, int cus, int cap) {
  const int64_t b32 = (int64_t)d.heads * ((d.nq + 31) / 32), b16 = (int64_t)d.heads * ((d.nq + 15) / 16);
  g->parts = 1;
  g->form = b32 >= 4 * (int64_t)cus ? F32_ROWS32 : F32_ROWS16;
  if (g->form == F32_ROWS32) return;
  // (fitted, as plan_bwd_f32, to 39 shapes of 1 x 64 x 64 to 16 x 1024 x 1024 x up to 6 (36) numbers of parts: 2 % (6 %) off the best of
  // them in the mean, where steps as long as their matrix instructions were 5 % (12 %) off - a step of a chip that is
  // not full waits for its loads.  2 x 300 x 900, H = 64 15.0 -> 10.7 us)
  constexpr double kStep[4] = {0.93, 1.11, 1.49, 1.99}, kFixed = 2.4;
  double of_rows[8];
  const double most = (double)visible_keys(d, *g, d.nq - 1) / BLK;
  const double mean = g->by_size ? mean_visible_keys(d, *g, of_rows) / BLK : most;
  const double part_us = (double)d.heads * d.nq * (d.hdim + 2) * 8 / 4.6e6;
  double whole = 0, least = 0;
  for (int z : kParts) {
    if (z > 1 && (z > cap || z > most + 1)) break;
    const Kind k = f32_kind(b16, mean, most, z, g->by_size != 0, kStep[head_index(d.hdim)], kFixed);
    const double t = one_time(k, Kind{0, 0, 0}, 2 * cus, g->by_size != 0, 0.5) + (z > 1 ? kSumUs + z * (part_us + 1.5 * kPartUs) : 0);
    if (z == 1) whole = least = t;
    else if (t < 0.85 * whole && t < least) { least = t; g->parts = z; }      // (a split has to be clearly better)
  }
}

BwdParts plan_bwd_f32(const a2d_tile_desc& d, const SegList& g, int cus, int cap_kv, int cap_q) {
  const int64_t bq = (int64_t)d.heads * ((d.nq + 15) / 16), bk = (int64_t)(d.heads / g.group) * ((d.nkv + 15) / 16);
  const double sq = (double)visible_keys(d, g, d.nq - 1) / BLK + 1, sk = (double)g.group * ((d.nq + 15) / 16);
  constexpr double kRow[4] = {0.95, 1.21, 1.87, 2.88}, kRowFixed = 3.6, kKey[4] = {1.69, 2.06, 3.05, 4.28}, kKeyFixed = 1.7;
  const int hx = head_index(d.hdim);
  const bool uneven = g.by_size != 0;
  double seen[8];
  const double q_most = (double)visible_keys(d, g, d.nq - 1) / BLK;
  const double mean = uneven ? mean_visible_keys(d, g, seen) : q_most * BLK;
  const double part_kv = (double)d.heads / g.group * d.nkv * d.hdim * 16 / 4.9e6, part_q = (double)d.heads * d.nq * d.hdim * 8 / 4.9e6;
  BwdParts p = {};
  p.kv = p.q = 1;
  // delta: from O by the dK/dV workgroups themselves; by a launch in front where these take more than some steps a compute
  // unit in all.  (own / launch, us: H = 96 12 x 700 x 900 causal 72 / 76, 16 x 700 x 900 92 / 96, 20 x 700 x 900 110 / 107, 16 x 700 x
  // 900 unmasked 137 / 129; H = 64 16 x 1024 x 1024 causal 80 / 85; H = 128 4 x 300 x 300 20 / 24.  Earliest at H = 128, where the rows
  // of O cost the registers of the next loads, then at H = 96, where they cost the third workgroup of a compute unit)
  constexpr int kDeltaSteps[4] = {140, 140, 110, 80};
  p.delta = (double)bq * mean / BLK > (double)kDeltaSteps[hx] * cus;
  // Parts, over 1040 drawn shapes of 1 to 16 heads, 64 to 1024 rows and keys, each against up to 42 of them: with slots for the workgroups
  // that fit, a third one that takes 6 % of a step and 4.6 us for the sum 4.0 % off the best in the mean, with two slots for all and
  // 5 us 4.6 %.  Of 4000 other shapes 390 go out otherwise, 1.06 times as fast in the mean, those that were whole 1.14 times (8 x
  // 256 x 900, H = 80 31.8 -> 27.5 us, 2 x 361 x 157, H = 80, causal 13.9 -> 9.1), those of more parts than before the same in the mean
  // (a third of them 3 % slower or more: 15/5 x 275 x 179, H = 64 15.4 -> 19.2).
  constexpr double kBwdSumUs = 4.6;
  const int slots = bwd_fit(d.hdim, !p.delta) * cus;
  double whole = 0, least = 0;
  for (int zk : kParts) {
    if (bq + bk > 16 * (int64_t)cus) break;          // (a chip that is full for many turns)
    if (zk > 1 && (zk > cap_kv || zk > sk)) break;
    for (int zq : kParts) {
      if (zq > 1 && (zq > cap_q || zq > sq)) break;
      const double share = (double)(bq * zq + bk * zk) / cus, third = (share < slots / cus ? share : slots / cus) - 2;
      const double busy = share > 2 ? 1.14 + 0.06 * third : share > 1.75 ? 0.57 * share : 1;
      const Kind q = f32_kind(bq, mean / BLK, q_most, zq, uneven, kRow[hx] * busy, kRowFixed);
      const Kind k = f32_kind(bk, uneven ? sk * mean / d.nkv : sk, sk, zk, uneven, kKey[hx] * busy, kKeyFixed);
      const double t = (q.most > k.most ? one_time(q, k, slots, uneven, 0.86) : one_time(k, q, slots, uneven, 0.86)) +
                       (zk > 1 || zq > 1 ? kBwdSumUs : 0) + (zk > 1 ? zk * (part_kv + kPartUs) : 0) + (zq > 1 ? zq * (part_q + kPartUs) : 0);
      if (zk == 1 && zq == 1) whole = least = t;
      else if (t < 0.87 * whole && t < least) { least = t; p.kv = zk; p.q = zq; }
    }
  }
  // the kind with the longer walks first; under a mask the longest and the shortest count alike, so that short ones come
  // last (16 x 700 x 900: dQ first 92.0 us, dK/dV first 93.2; 16 x 1024 x 1024, H = 64, causal 87 / 80)
  double lq = sq, lk = sk, of_rows[8];
  if (g.by_size) {
    mean_visible_keys(d, g, of_rows);
    const double all = (double)visible_keys(d, g, d.nq - 1);
    lq = (double)visible_keys(d, g, 0) / BLK;
    lk = 0;                                          // rows that see the last keys
    for (int i = 0; i < 8; ++i) lk += of_rows[i] >= all ? sk / 8 : 0;
  }
  p.q_first = 3 * (sq + lq) / p.q > 4 * (sk + lk) / p.kv;
  p.one = 1;
  return p;
}

hipError_t launch_fwd_f32(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                          float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s) {
  switch (d.hdim) {
    case 128: return fwd_h<128>(d, g, Q, K, V, O_part, m, l, in, s);
    case 96: return fwd_h<96>(d, g, Q, K, V, O_part, m, l, in, s);
    case 80: return fwd_h<80>(d, g, Q, K, V, O_part, m, l, in, s);
    default: return fwd_h<64>(d, g, Q, K, V, O_part, m, l, in, s);
  }
}

hipError_t launch_bwd_f32(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                          const void* O, const void* dO, const float* lse, float* delta, float* dQ, float* dK,
                          float* dV, const BwdParts& parts, hipStream_t s) {
  switch (d.hdim) {
    case 128: return bwd_h<128>(d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
    case 96: return bwd_h<96>(d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
    case 80: return bwd_h<80>(d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
    default: return bwd_h<64>(d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
  }
}

}  // namespace a2d
