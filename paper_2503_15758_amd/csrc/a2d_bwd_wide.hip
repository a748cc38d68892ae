// bf16 dK/dV kernel for tiles with many keys: the contractions of bwd_dkdv_kernel (a2d_bwd_mfma.hip) with
// 256 keys per workgroup.
#include "a2d_bwd_wide.hpp"

namespace a2d {
namespace {

using namespace mfma;

template <int HR, bool WRITE_DS>
__global__ __launch_bounds__(WK_THREADS) void bwd_dkdv_wide_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO, const float* __restrict__ lse,
    const float* __restrict__ delta, float* __restrict__ dK, float* __restrict__ dV,
    bf16_t* __restrict__ dS) {
  warm_arguments<9 * 8>();
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  dkdv_wide<HR, WRITE_DS, 0>(blockIdx.x, lds, d, g, g.parts, Q, K, V, dO, lse, delta, dK, dV, dS);
}

template <int HR, bool WRITE_DS>
hipError_t go(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
              const void* dO, const float* lse, const float* delta, float* dK, float* dV, void* dS, hipStream_t s) {
  constexpr int bytes = wk_lds(padded_head(HR));
  if (ph == PREPARE)
    return ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_dkdv_wide_kernel<HR, WRITE_DS>), bytes);
  const dim3 grid(xcd_grid(d.heads / g.group * g.parts, (d.nkv + WK_KEYS - 1) / WK_KEYS));
  A2D_LAUNCH((bwd_dkdv_wide_kernel<HR, WRITE_DS>), grid, dim3(WK_THREADS), bytes, s, d, g, (const bf16_t*)Q,
             (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, lse, delta, dK, dV, (bf16_t*)dS);
  return hipGetLastError();
}

template <int HR>
hipError_t go_h(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                const void* dO, const float* lse, const float* delta, float* dK, float* dV, void* dS, hipStream_t s) {
  if constexpr (HR == 128)
    if (dS) return go<HR, true>(ph, d, g, Q, K, V, dO, lse, delta, dK, dV, dS, s);
  return go<HR, false>(ph, d, g, Q, K, V, dO, lse, delta, dK, dV, dS, s);
}

}  // namespace

hipError_t launch_dkdv_wide(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                            const void* V, const void* dO, const float* lse, const float* delta, float* dK, float* dV,
                            void* dS, hipStream_t s) {
  switch (d.hdim) {
    case 128: return go_h<128>(ph, d, g, Q, K, V, dO, lse, delta, dK, dV, dS, s);
    case 96: return go_h<96>(ph, d, g, Q, K, V, dO, lse, delta, dK, dV, dS, s);
    case 80: return go_h<80>(ph, d, g, Q, K, V, dO, lse, delta, dK, dV, dS, s);
    default: return go_h<64>(ph, d, g, Q, K, V, dO, lse, delta, dK, dV, dS, s);
  }
}

}  // namespace a2d
