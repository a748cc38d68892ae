// Memory for the shared walks of static calls: what the torch binding offers a2d_partial_bwd_static, so that
// its results are bitwise those of the binding's a2d_partial_bwd, which draws on torch's allocator.
// (At most kSplitBytes each for dK with dV and for dQ.)  A translation unit of its own: the array comes
// onto a GPU when its address is first asked for there, and a program that never shares the walks of a
// static call never holds it.
#include "a2d_common.hpp"

namespace a2d {
namespace {

constexpr size_t kBytes = 2 * kSplitBytes;
__device__ __align__(256) char partial_sums[kBytes];
SymbolCache g_partial_sums;

}  // namespace

void* static_partial_sums(size_t bytes) {
  void* p = nullptr;
  if (bytes > kBytes || symbol_address(HIP_SYMBOL(partial_sums), &g_partial_sums, &p) != hipSuccess) return nullptr;
  return p;
}

}  // namespace a2d
