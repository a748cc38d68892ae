// Alg. 1 and Alg. 3 over a whole emulated side x side grid in a handful of launches: the tile kernels, on all
// grid rows or columns per launch (GridView), on the blocks where they lie in the sequence (contiguous or
// cyclic: a stride, not a copy).
#pragma once
#include <hip/hip_runtime_api.h>

#include "a2d.h"

namespace a2d {

bool force_generic();            // the debug switch a2d_debug_force_generic() sets

// scratch memory offered to the tile calls of this host thread (see a2d_common.hpp)
struct ScratchSource {
  void* (*get)(void* ctx, size_t bytes);
  void* ctx;
};
void scratch_offer(const ScratchSource* src);
// `bytes` of a device array of the library's own, the same at every call (a2d_static.hip); NULL: not to be had
void* static_partial_sums(size_t bytes);

// How a call goes out: the kernels it launches, in order, and how they share the work.  From host arithmetic alone
// (diagnostic: no device is needed, nothing is enqueued), by the same plans as the calls.
struct Route {
  const char* kernel[4];
  int kernels;
  int rows, lanes;               // query rows of a forward or dQ workgroup; its key lanes, which share the walk
  int keys;                      // of a dK/dV workgroup (0: a forward)
  int parts_q, parts_kv;         // workgroups that share a walk of the one kind (forward and dQ) and the other
  int phased;                    // a forward's wavefronts in opposite phases
  int apart;                     // a backward of few rows: dK and dV in workgroups of their own
};
enum RouteFlags { ROUTE_BACKWARD = 1, ROUTE_KEEP_DS = 2, ROUTE_SPLIT_GROUPS = 4, ROUTE_SCRATCH = 8 };
// a tile call on a chip of `cus` compute units (0: the current device); ROUTE_SCRATCH: with scratch memory on offer
a2d_status tile_route(const a2d_tile_desc& desc, int kv_heads, int nseg, const a2d_kv_segment* segs, int flags, int cus,
                      Route* out);

struct GridProblem {
  int heads, kv_heads, seq, side, hdim, causal, cyclic;
  float scale;
  a2d_layout q, k, v, o, g;      // layouts of Q, K, V, O, dO over the whole sequence (elements)
  a2d_layout dq, dk, dv;         // of the gradients
};

// Whether the batched path covers the problem (bf16; the kernels' 32-bit offsets)
bool grid_supported(const GridProblem& p);
// Workspace in bytes: partial results of split walks, delta
size_t grid_forward_bytes(const GridProblem& p);
size_t grid_backward_bytes(const GridProblem& p);
// O with the layout p.o, lse plain [heads][seq].  Both only enqueue on `s`.
hipError_t grid_forward(const GridProblem& p, const void* Q, const void* K, const void* V, void* O, float* lse,
                        void* ws, hipStream_t s);
// O, dO and the gradients with the problem's layouts; lse plain
hipError_t grid_backward(const GridProblem& p, const void* Q, const void* K, const void* V, const void* O,
                         const void* dO, const float* lse, void* dQ, void* dK, void* dV, void* ws, hipStream_t s);

// false: not covered, or no device to ask
bool grid_route(const GridProblem& p, bool backward, int cus, Route* out);

}  // namespace a2d
