// Shared by the bf16 backward kernels (a2d_bwd_*).
#pragma once
#include "a2d_mfma.hpp"

namespace a2d {
namespace mfma {

// a transposed accumulator rounded to bf16 (see store_acc_t)
template <int CT>
__device__ __forceinline__ void store_acc_t(bf16_t* __restrict__ out_row, const f32x16 (&acc)[CT], int half, float mul,
                                            int h) {
#pragma unroll
  for (int ht = 0; ht < CT; ++ht)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (32 * ht + 8 * g + 4 * half >= h) continue;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (bf16_t)(acc[ht][4 * g + e] * mul);
      *reinterpret_cast<bf16x4*>(out_row + 32 * ht + 8 * g + 4 * half) = v;
    }
}

// stores a transposed accumulator (lane = one output row, registers = 4-column groups)
// (add: onto what the row already holds)
// CT column tiles of 32; pieces whose columns lie past the head size h are skipped
template <int CT>
__device__ __forceinline__ void store_acc_t(float* __restrict__ out_row, const f32x16 (&acc)[CT],
                                            int half, float mul, int h, bool add = false) {
#pragma unroll
  for (int ht = 0; ht < CT; ++ht)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (32 * ht + 8 * g + 4 * half >= h) continue;
      f32x4 v = {acc[ht][4 * g] * mul, acc[ht][4 * g + 1] * mul, acc[ht][4 * g + 2] * mul,
                 acc[ht][4 * g + 3] * mul};
      f32x4* p = reinterpret_cast<f32x4*>(out_row + 32 * ht + 8 * g + 4 * half);
      if (add) {
        const f32x4 o = *p;
        v[0] += o[0]; v[1] += o[1]; v[2] += o[2]; v[3] += o[3];
      }
      *p = v;
    }
}

__device__ __forceinline__ f32x4 lds_load_f32x4(unsigned addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>((uintptr_t)addr);
}

// A step of the dK/dV pairs: BQ query rows, staged through LDS as a buffer { Q tile, dO tile } (dual
// layout) and two statistics per row
constexpr int BQ = 32;
constexpr int DK_TILE = BQ * DUAL_LD;
constexpr int DK_BUF = 2 * DK_TILE;
constexpr int DK_STAT_BUF = 2 * BQ * 4;

// ---- dS hand-over to the dQ kernel (optional).  The dK/dV kernel can leave dS (bf16, already
// multiplied out: P o (dP - delta)) in a workspace, so that the dQ kernel is a plain contraction
// dQ = scale dS K instead of recomputing S and dP.  Workspace layout: per head, per 32-row tile rt,
// per 64-key block kb one 4 KiB tile [piece T = 0, 1 (32 keys each)][kt = 0, 1 (16 keys each)]
// [g = 0 .. 3][key][8 bf16]: rows 4 g + 0..3 and 16 + 4 g + 0..3 of key 64 kb + 32 T + 16 kt + key - what a lane of the dK/dV
// kernel holds of its key, stored as it is.  The dQ kernel brings the tiles straight into LDS and has
// the transposing read turn them.  (Turned by the producer, through LDS in every step, they cost it 3 %.)
constexpr int DS_TILE_BYTES = 4096;
__host__ __device__ inline int ds_row_tiles(int nq) { return (nq + 31) / 32; }
__host__ __device__ inline int ds_key_blocks(int nkv) { return (nkv + 63) / 64; }
__host__ __device__ inline size_t ds_head_bytes(int nq, int nkv) {
  return (size_t)ds_row_tiles(nq) * ds_key_blocks(nkv) * DS_TILE_BYTES;
}

typedef __attribute__((address_space(1))) char* gwptr_t;
__device__ __forceinline__ gwptr_t uniform_gwptr(void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<gwptr_t>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void gstore_b128(gwptr_t base, unsigned byte_off, bf16x8 v) {
  // streamed once, read back by another kernel: keep it from displacing the Q / dO tiles in L2
  __builtin_nontemporal_store(v, reinterpret_cast<__attribute__((address_space(1))) bf16x8*>(base + byte_off));
}

}  // namespace mfma
}  // namespace a2d
