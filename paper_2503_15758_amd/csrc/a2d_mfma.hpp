// Building blocks shared by the bf16 MFMA tile kernels (H = 128, 96, 80, 64): the MFMA wrapper and its
// fragment layouts, LDS fragment reads, the "dual" LDS tile layout, scalar-base global loads and
// the XCD-aware work mapping.
//
// v_mfma_f32_32x32x16_bf16, D(32x32) += A(32x16) * B(16x32):
//   A fragment: lane holds row (lane & 31), contraction indices 8*(lane>>5) + 0..7
//   B fragment: lane holds column (lane & 31), contraction indices 8*(lane>>5) + 0..7
//   D: lane holds column (lane & 31); register r is row 8*(r>>2) + 4*(lane>>5) + (r&3)
// v_mfma_f32_16x16x32_bf16, D(16x16) += A(16x32) * B(32x16):
//   A, B fragments: lane holds row / column (lane & 15), contraction indices 8*(lane>>4) + 0..7
//   D: lane holds column (lane & 15); register r is row 4*(lane>>4) + r
// All bf16 kernels but the dK/dV pairs and the backward of few rows run on the latter, which costs less power per flop (see
// a2d_bwd_wide.hpp).
// Two kinds of fragment reads from a row-major LDS tile (rows x padded head size, bf16):
//   - "natural" fragments (contraction along H): one 128-bit read per lane;
//   - "transposed" fragments (contraction along the row index): two ds_read_b64_tr_b16, where a
//     16-lane group reads 4 consecutive rows x 16 columns and every lane receives a column.
#pragma once
#include <type_traits>

#include "a2d_common.hpp"

namespace a2d {
namespace mfma {

// Head sizes of the MFMA kernels: the tiles are laid out for HD = 64, 96 or 128 columns (multiples
// of the 32-column accumulator tile); a head size of 80 runs as HD = 96 with its last 16 columns
// zero in LDS and in the register fragments and left out of every store.
__host__ __device__ constexpr int padded_head(int h) { return h > 96 ? 128 : (h > 64 ? 96 : 64); }

// compile-time loop: f(std::integral_constant<int, B>{}), ..., f(std::integral_constant<int, E - 1>{})
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// eight consecutive D registers -> one bf16 B/A fragment (round to nearest even)
__device__ __forceinline__ bf16x8 pack8(const f32x16& s, int base) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16_t)s[base + e];
  return r;
}

// the lane's number, computed where it is called (not kept in a register)
__device__ __forceinline__ int lane_again() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// the value another lane holds (a DPP control word: quad_perm, row_half_mirror 0x141, row_mirror 0x140)
template <int CTRL>
__device__ __forceinline__ float lane_swap(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

// A branch of a main loop that is seldom taken: its code is laid out behind the loop, so that the loop
// itself stays in one run of instruction lines (the walk's move to another sub-block inside the forward loop
// cost 1 % at H = 128, 2 % at H = 80, 3 % at 16 x 2048 x 2048).  And one that is taken in every turn but the last: its
// code stays where it stands.  (Macros: of an inlined function the compiler has dropped the hint by the time it is inlined.)
#define A2D_SELDOM(x) __builtin_expect((bool)(x), 0)
#define A2D_OFTEN(x) __builtin_expect((bool)(x), 1)

// a / b and the rest, without a division by one: unsplit walks, heads that are not grouped (a division is some 35 dependent
// instructions on the way to a workgroup's first loads)
struct Split {
  int q, r;
};
__device__ __forceinline__ Split split_by(int a, int b) {
  Split s = {a, 0};
  if (A2D_SELDOM(b != 1)) {
    s.q = a / b;
    s.r = a - s.q * b;
  }
  return s;
}

// of block t of the group x nblocks of a key/value head: its number within its query head (q) and that head (r)
__device__ __forceinline__ Split query_head(int t, int group, int nblocks, bool by_size) {
  Split s = {t, 0};
  if (A2D_SELDOM(group != 1)) {
    const int by = by_size ? group : nblocks, q = t / by, r = t - q * by;
    s.q = by_size ? q : r;
    s.r = by_size ? r : q;
  }
  return s;
}

// s_waitcnt vmcnt(0) only (gfx9 encoding: lgkmcnt and expcnt fields left at their maxima).
// Placed after a prologue's one-off global loads it tells the compiler's wait-count insertion that
// those registers are complete, so that uses inside the main loop do not have to be guarded by
// waits that would also cover the loop's own freshly issued prefetches.
__device__ __forceinline__ void wait_vmem_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }
template <int N>                                     // all but the last N operations (the counter's upper bits stand apart)
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N < 64, "the counter has six bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);
}
// the same for loads into LDS that the wavefront itself reads, with no barrier in between: no read moves up past the wait
template <int N = 0>
__device__ __forceinline__ void wait_dma() {
  wait_vmem<N>();
  asm volatile("" ::: "memory");
}

// Global-memory pointer that is the same in every lane, held in scalar registers, so that loads
// through it use the scalar-base + 32-bit-lane-offset addressing form (no per-lane 64-bit address
// arithmetic).  It carries the global address space: a generic pointer rebuilt from integers would
// turn the loads into FLAT ones, which also count on the LDS wait counter.
typedef const __attribute__((address_space(1))) char* gptr_t;
__device__ __forceinline__ gptr_t uniform_gptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<gptr_t>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ u32x4 gload_b128(gptr_t base, unsigned byte_off) {
  return *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(base + byte_off);
}

// A value that is the same in every lane, in a scalar register.  (The compiler may not know that it is the same: it would fold the
// builtin away, and a product, which only the vector ALU makes, would keep a register of every lane.)
__device__ __forceinline__ float uniform(float x) {
  asm("" : "+v"(x));
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// LDS reads by byte address (address space 3)
__device__ __forceinline__ bf16x8 lds_load_b128(unsigned addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>((uintptr_t)addr);
}
__device__ __forceinline__ bf16x8 lds_load_tr(unsigned addr_lo, unsigned addr_hi) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)addr_lo);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)addr_hi);
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// "Dual" LDS tile layout for tiles read BOTH ways (natural and transposed) with
// immediate-only addressing: rows of 320 B (256 B data + 64 B pad), and within a row the
// 16-byte chunk c sits at position c ^ ((row >> 2) & 3).
//   - the 64 B pad shifts consecutive rows by 16 banks, so the four rows of a transposing
//     32-lane pass use four disjoint 16-bank windows;
//   - the XOR on the two low chunk bits separates the rows r, r+4, r+8, r+12 that share a
//     window in a 16-row natural (128-bit) pass.
// Every fragment address is then one of four per-lane bases plus a compile-time constant:
//   natural fragment x of rows RB + (lane & 31), RB a multiple of 32:
//       (x & 1 ? nat_o : nat_e) + 64 * (x >> 1) + RB * 320
//   transposing reads of column tile ct, rows RB + {0..7 | 8..15}, RB a multiple of 16:
//       (tr_lo | tr_hi) + 64 * ct + RB * 320
constexpr int DUAL_LD = 320;
struct DualAddr {
  unsigned nat_e, nat_o, tr_lo, tr_hi;
  __device__ __forceinline__ void init(int lane, unsigned tile_base) {
    const int l32 = lane & 31, half = lane >> 5;
    const int kap = (l32 >> 2) & 3;
    nat_e = tile_base + l32 * DUAL_LD + 32 * (kap >> 1) + 16 * (half ^ (kap & 1));
    nat_o = nat_e ^ 32;      // bit 5 of the address is exactly the (x & 1) ^ (kap >> 1) term
    const int g16 = lane >> 4, j16 = lane & 15;
    const int row = 4 * (g16 >> 1) + (j16 >> 2);           // 0..7, (row >> 2) & 3 = g16 >> 1
    const int cl = 2 * (g16 & 1) + ((j16 & 3) >> 1);       // logical chunk within a 64-byte column tile
    const int sub = 8 * (j16 & 1);
    tr_lo = tile_base + row * DUAL_LD + 16 * (cl ^ (g16 >> 1)) + sub;
    tr_hi = tile_base + (row + 8) * DUAL_LD + 16 * (cl ^ ((g16 >> 1) + 2)) + sub;
  }
};
// byte offset inside a dual tile at which the 16-byte chunk `c` of row `r` is stored
__device__ __forceinline__ int dual_store_off(int r, int c) { return r * DUAL_LD + ((c ^ ((r >> 2) & 3)) << 4); }

// Tiles that are loaded straight into LDS (dma_b128: lane i of a wavefront writes the 16 bytes at i from a common address on,
// so rows cannot be padded).  A tile is made of blocks of 16 rows x 32 columns, 1 KiB each, one wavefront's load: row r at 64 r,
// its four 16-byte chunks c at c ^ block_swap(r >> 2).  With that both kinds of fragment reads are conflict free:
//   - natural fragment of row tile t, slice sl: nat + block(t, sl);
//   - transposed fragment of column tile ht, row tiles t and t + 1: (ht & 1 ? tr_o : tr_e) + block(t, ht >> 1) and block(t + 1, ht >> 1).
constexpr int BLOCK = 1024;
__device__ __forceinline__ int block_swap(int q) { return 2 * ((q ^ (q >> 1)) & 1) | (q >> 1); }
struct Blocks16 {
  unsigned nat, tr_e, tr_o;
  __device__ __forceinline__ void init(int lane, unsigned tile_base) {
    const int g = lane >> 4, j = lane & 15;
    nat = tile_base + j * 64 + 16 * (g ^ block_swap(j >> 2));
    tr_e = tile_base + (4 * g + (j >> 2)) * 64 + 16 * (((j & 3) >> 1) ^ block_swap(g)) + 8 * (j & 1);
    tr_o = tr_e ^ 32;
  }
};
// Lane i's 16 bytes at base + byte_off go to LDS address `at` + 16 i (lanes that are switched off write nothing).  They count as one
// vector memory operation; the compiler does not know of it, so the caller waits (wait_vmem_all) before the barrier behind
// which the tile is read.  dma_blocks: the N blocks of a row tile, slice after slice of its rows - one lane offset and one
// base for all (the instruction's offset counts for both addresses).
// (NT: read once.  The address goes in as m0 itself, so that the compiler knows of it; the instruction needs a wait state behind a
// write of m0, which it does not put in front of assembly)
#define A2D_DMA(width, more)                                                                                                 \
  asm volatile("s_nop 0\n\tglobal_load_lds_" width " %1, %2 offset:%3" more ::"{m0}"(                                        \
                   __builtin_amdgcn_readfirstlane(at - OFF)),                                                                \
               "v"(byte_off), "s"(base), "n"(OFF)                                                                            \
               : "memory")
template <int OFF, bool NT = false>
__device__ __forceinline__ void dma_b128(unsigned at, gptr_t base, unsigned byte_off) {
  if constexpr (NT) A2D_DMA("dwordx4", " nt"); else A2D_DMA("dwordx4", "");
}
// (four bytes a lane, at `at` + 4 i)
template <int OFF>
__device__ __forceinline__ void dma_b32(unsigned at, gptr_t base, unsigned byte_off) {
  A2D_DMA("dword", "");
}
#undef A2D_DMA
// (H: the head size; chunks past it are left alone)
template <int N, int H>
__device__ __forceinline__ void dma_blocks(unsigned at, gptr_t base, unsigned byte_off, int chunk) {
  static_for<0, N>([&](auto X) {
    constexpr int x = decltype(X)::value;
    if (32 * x + 32 <= H || 32 * x + 8 * chunk < H) dma_b128<64 * x>(at + x * BLOCK, base, byte_off);
  });
}

// maximum, sum over the four lanes of a row (16 apart).  The lane groups are exchanged in pairs by the vector ALU: shuffles
// through LDS are four times the latency.
template <class F>
__device__ __forceinline__ float row_reduce(float x, F&& f) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned a0 = a[0], a1 = a[1];             // (a bit_cast of an element itself is one of the first)
  const unsigned w = __builtin_bit_cast(unsigned, f(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1)));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  const unsigned b0 = b[0], b1 = b[1];
  return f(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}
__device__ __forceinline__ float row_max(float x) { return row_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float row_sum(float x) { return row_reduce(x, [](float a, float b) { return a + b; }); }

// of lane i's rows i % 16 and i % 16 + 16: what lanes of row i % 32 hold
__device__ __forceinline__ void row_pair(float x, float (&of)[2]) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned a0 = a[0], a1 = a[1];
  of[0] = __builtin_bit_cast(float, a0);
  of[1] = __builtin_bit_cast(float, a1);
}

// Stores 16 rows of a transposed accumulator of 16 x 16 tiles (lane j + 16 g: columns 16 ht + 4 g + 0..3 of row j, in each of
// NT row tiles; here tile t), times `mul` of the lane's row, to out, out + row, ..; `n` of the rows exist.  They
// pass through LDS (`area`, acc_area bytes of the wavefront's own), so that an instruction stores whole rows: a lane's pieces
// as they stand are 64 separate 16-byte writes an instruction.  Non-temporal: the results of a turn of workgroups, which all
// store at once, are as large as the L2s and would displace what the next turn reads and be written back when the launch ends.
// us, pieces as they stand / whole rows / non-temporal: 256 workgroups of the forward at H = 128 with one step each 13.2 / 12.5 /
// 11.4 (without any stores 6.7), 16 x 2048 x 2048 forward 37.9 / 37.5 / 36.2 and backward 113.9 / 110.9 / 108.7, backward
// 96 x 4096 x 4096 with dS 2188 / 2173 / 2060.
// (add: onto what the rows already hold; row_of: where row r of the tile goes)
__host__ __device__ constexpr int acc_ld(int ht) { return 64 * ht + 16; }
__host__ __device__ constexpr int acc_area(int ht) { return 16 * acc_ld(ht); }
template <int HT, int NT>
__device__ __forceinline__ void acc_to_lds(char* area, const f32x4 (&acc)[HT][NT], int t, int lane, float mul) {
  asm volatile("" ::: "memory");                     // (lanes read what others write: the wavefront's LDS operations keep their order)
  char* const at = area + (lane & 15) * acc_ld(HT) + 16 * (lane >> 4);
#pragma unroll
  for (int ht = 0; ht < HT; ++ht) {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = acc[ht][t][e] * mul;
    *reinterpret_cast<f32x4*>(at + 64 * ht) = v;
  }
  asm volatile("" ::: "memory");
}
struct Ascending {
  __device__ __forceinline__ int operator()(int r) const { return r; }
};
template <int HT, int NT, class RowOf = Ascending>
__device__ __forceinline__ void store_acc16(float* out, int64_t row, int n, char* area, const f32x4 (&acc)[HT][NT], int t,
                                            int lane, float mul, bool add = false, RowOf&& row_of = {}) {
  acc_to_lds(area, acc, t, lane, mul);
#pragma unroll
  for (int x = 0; x < HT; ++x) {
    const int i = lane + 64 * x, r = i / (4 * HT), ch = i - r * (4 * HT), to = row_of(r);
    f32x4 v = *reinterpret_cast<const f32x4*>(area + r * acc_ld(HT) + 16 * ch);
    if (to >= n) continue;
    f32x4* const p = reinterpret_cast<f32x4*>(out + to * row + 4 * ch);
    if (add) {
      const f32x4 o = *p;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += o[e];
    }
    __builtin_nontemporal_store(v, p);
  }
}
template <int HT, int NT>
__device__ __forceinline__ void store_acc16(bf16_t* out, int64_t row, int n, char* area, const f32x4 (&acc)[HT][NT], int t,
                                            int lane, float mul) {
  acc_to_lds(area, acc, t, lane, mul);
#pragma unroll
  for (int x = 0; x < (HT + 1) / 2; ++x) {
    const int i = lane + 64 * x, r = i / (2 * HT), ch = i - r * (2 * HT);
    if (r >= n || (HT % 2 && r >= 16)) continue;
    const f32x4 a = *reinterpret_cast<const f32x4*>(area + r * acc_ld(HT) + 32 * ch);
    const f32x4 b = *reinterpret_cast<const f32x4*>(area + r * acc_ld(HT) + 32 * ch + 16);
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = (bf16_t)a[e]; v[4 + e] = (bf16_t)b[e]; }
    __builtin_nontemporal_store(v, reinterpret_cast<bf16x8*>(out + r * row + 8 * ch));
  }
}

// XCD-aware work mapping.  MI355X has 8 XCDs, each with its own L2, and hands consecutive
// workgroup ids to consecutive XCDs (id % 8).  All blocks of one head read the same K / V (or
// Q / dO) rows, so they are placed on ONE XCD.  Two orders inside an XCD (k-th workgroup of XCD x,
// id = 8 k + x):
//   by head  (by_size = false): head 8 * (k / nblocks) + x, block k % nblocks - a head's blocks run
//            back to back and share its rows in L2; used when all blocks cost the same;
//   by block (by_size = true):  the XCD's heads in chunks (size_chunk); inside a chunk block b of
//            every head before any block b + 1.  The callers number the blocks heaviest first, so
//            under a causal mask that crosses the tile the workgroups start longest first and the
//            compute units finish together (diagonal forward tile of 96 heads -7 %).  (The unmasked tile
//            loses 2-3 % with this order, which is why it is not the default.)
// That holds for the first 8 * (heads / 8) heads.  The blocks of the remaining heads % 8 heads are
// spread evenly over all XCDs instead (a head on an XCD of its own would leave the other XCDs
// without work: a tile of 1 head used 32 of the 256 compute units, one of 12 heads ran 8 and then
// 4) and start first: by head in runs - XCD x takes the x-th eighth of the blocks, head after head, so
// that few XCDs read the same rows - or, by block, heaviest first across the XCDs.
// Grid size: 8 * (heads / 8 * nblocks + ceil(heads % 8 * nblocks / 8)); the few workgroups without
// a block exit.
constexpr int kXcds = 8;
constexpr int kXcdCus = 32;                        // compute units of an XCD
// Heads of a chunk, for `whole` heads of nblocks blocks on an XCD that holds `turn` workgroups at a time.  Few heads at a
// time share their rows in L2; but every chunk starts its longest walks after the chunk before it, and the last one
// must not start them late.
//   - Launches of six turns or more whose heads make whole chunks of four: four.  Diagonal tiles, H = 128, one chunk of
//     up to 16 heads -> chunks of 4: 96 x 4096 x 4096 reads 854 -> 468 MiB (forward) and 1611 -> 717 (recomputing dQ) in the same
//     time; forward 128 x 4096 x 4096 597 -> 587 us, 192 x 4096 x 4096 887 -> 876, 64 x 8192 x 8192 1073 -> 1067.
//   - Fewer turns, or a rest: one chunk, equal ones from 17 heads on.  Chunks of 4 cost 48 x 4096 x 4096 (three turns) 224 ->
//     229 us, 96 x 2048 x 2048 (three) 128 -> 134, 40 x 1300 x 1300 37.5 -> 46.8 and, with a rest, 80 x 4096 x 4096 369 -> 390.
//   - So do kernels that stream a score-sized operand or share little (turn = 0: dK/dV, dQ from dS).  With chunks of 4 dK/dV
//     reads 1049 -> 966 MiB at 96 x 4096 x 4096, and the backward with dS takes 1397 -> 1415 us, at H = 64 964 -> 1010.
__host__ __device__ inline int size_chunk(int whole, int nblocks, int turn) {
  if (turn > 0 && whole % 4 == 0 && whole * nblocks >= 6 * turn) return 4;
  const int n = (whole + 15) / 16;
  return n <= 1 ? whole : (whole + n - 1) / n;
}
__host__ __device__ inline int xcd_grid(int heads, int nblocks) {
  return kXcds * (heads / kXcds * nblocks + (heads % kXcds * nblocks + kXcds - 1) / kXcds);
}
// (id: the workgroup's number in the launch, or in its own part of one - which then starts at a multiple of kXcds)
__device__ __forceinline__ bool xcd_map(int id, int heads, int nblocks, bool by_size, int& head, int& block, int turn = 0) {
  const int x = id % kXcds;
  int k = id / kXcds;
  const int whole = heads / kXcds, rest = heads % kXcds, spread = rest * nblocks;
  const int per_xcd = (spread + kXcds - 1) / kXcds;
  if (k < per_xcd) {                               // blocks of the last `rest` heads
    if (by_size) {
      const int t = kXcds * k + x;
      head = kXcds * whole + t % rest;
      block = t / rest;
      return t < spread;
    }
    const int first = x * spread / kXcds, end = (x + 1) * spread / kXcds;
    head = kXcds * whole + (first + k) / nblocks;
    block = (first + k) % nblocks;
    return first + k < end;
  }
  k -= per_xcd;
  if (by_size) {
    const int chunk = size_chunk(whole, nblocks, turn);
    const int c = k / (chunk * nblocks), kk = k - c * (chunk * nblocks);
    const int width = min(chunk, whole - c * chunk);             // the last chunk may hold fewer heads
    head = kXcds * (c * chunk + kk % width) + x;
    block = kk / width;
  } else {
    head = kXcds * (k / nblocks) + x;
    block = k % nblocks;
  }
  return true;
}

}  // namespace mfma
}  // namespace a2d
