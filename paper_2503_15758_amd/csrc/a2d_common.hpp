// Shared device-side helpers and the launcher interface between the C-ABI layer
// (a2d_api.hip) and the kernel translation units.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "a2d.h"
#include "a2d_grid.hpp"

namespace a2d {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return (float)x; }

// 2^x on the hardware transcendental unit (about 1 ulp).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// c + the sum of eight products of bf16 pairs, two at a time: half the instructions of unpacked multiply-adds.  (Its error
// against 64 bits, in the sums of whole rows: tests/test_gpu_bwd_routes.py, no larger than that of such multiply-adds.)
__device__ __forceinline__ float dot8(u32x4 a, u32x4 b, float c) {
  typedef __bf16 pair_t __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned x = a[i], y = b[i];               // (a bit cast of a[i] itself takes a[0])
    c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(pair_t, x), __builtin_bit_cast(pair_t, y), c, false);
  }
  return c;
}

template <typename T> struct dtype_of;
template <> struct dtype_of<float> { static constexpr int value = A2D_F32; };
template <> struct dtype_of<bf16_t> { static constexpr int value = A2D_BF16; };

// Key/value sub-blocks of a tile for the causal mask.  Sub-block s covers the local keys
// seg[s].start .. + rows - 1 (the sub-blocks tile 0 .. nkv - 1 in order) and its keys are
// consecutive tokens; rel = q_off - (global index of its first key).  Query row i (local) sees
// key start[s] + kk of sub-block s iff kk <= i + rel.  A plain tile is one sub-block.
// `acc` rides along: != 0 makes the forward start from the (N, m, l) already in its output
// buffers and the backward add to the dQ partial already in its output buffer.
// `norm` != 0: the forward writes the NORMALISED partial O' = N / l in the input dtype (into the
// buffer passed as O_part) and lse' = m + ln l (into the buffer passed as m) instead of (N, m, l).
// `group` >= 1: query heads per key/value head (grouped-query attention: query head h reads
// key/value head h / group; K, V, dK, dV have heads / group heads).
// `by_size` != 0: the blocks of the tile differ in cost (a causal mask crosses it); the kernels then
// order their workgroups by block, heaviest first, over a whole XCD (see xcd_map).
// A launch over a whole emulated side x side grid (side = 0: a plain call).  All blocks of the grid are
// views of the same tensors: block b of Q starts b * q elements after block 0, and so on.  Tile (r, c) =
// query block r against key block c; under the causal mask rel = q_off - kv_off is (r - c) * rows for
// contiguous blocks, 0 / -1 (r >= c / r < c) for cyclic ones.  A workgroup of the forward and dQ kernels walks the
// tiles of a grid row, one of the dK/dV kernels those of a grid column.
// The kernels' GRID parameter: 0 a plain call, 1 contiguous blocks, 2 cyclic ones.
struct GridView {
  int side, cyclic;
  int64_t q, k, v, g, o;  // elements between blocks of Q, K, V, dO, O
  a2d_layout out[3];      // rows of a block of dQ, dK, dV in the whole tensors
  int64_t out_step[3];    // elements between their blocks
};
struct Segment {
  int start, rows;
  int64_t rel;
};
struct SegList {
  int n;
  int acc;
  int norm;
  int group;
  int by_size;
  int parts;      // workgroups that share the walk of one block, each leaving a partial result (>= 1)
  int form;       // which of its workgroup shapes a forward / dQ launch takes (plan_* below)
  int phased;     // a forward's wavefronts in opposite phases (plan_fwd_mfma)
  Segment seg[A2D_MAX_SEGMENTS];
  GridView b;     // (last: a tile's kernels do not read it)
};

// Brings the kernel's arguments - the tile's descriptor, the list's head and first sub-block, the grid, and the
// pointers behind them - into the scalar cache in one go.  A cold line costs about half a microsecond,
// and read one after another as the prologue comes to them they were a good part of the time of small
// tiles.
// (for kernels whose arguments begin with a2d_tile_desc, SegList; `more`: bytes of those that follow)
template <int MORE>
__device__ __forceinline__ void warm_arguments() {
  constexpr int head = (int)(sizeof(a2d_tile_desc) + offsetof(SegList, seg) + sizeof(Segment) + 63) / 64;
  constexpr int grid = (int)(sizeof(a2d_tile_desc) + offsetof(SegList, b)) / 64;
  constexpr int last = (int)(sizeof(a2d_tile_desc) + sizeof(SegList) + MORE - 1) / 64;
  static_assert(head <= 4 && last - grid <= 4, "lines to touch");
  constexpr auto line = [](int n) { return 64 * (n < last ? n : last); };
  int v[9];
  asm volatile(
      "s_load_dword %0, %9, 0x0\n\ts_load_dword %1, %9, 0x40\n\ts_load_dword %2, %9, 0x80\n\t"
      "s_load_dword %3, %9, 0xc0\n\ts_load_dword %4, %9, %10\n\ts_load_dword %5, %9, %11\n\t"
      "s_load_dword %6, %9, %12\n\ts_load_dword %7, %9, %13\n\ts_load_dword %8, %9, %14\n\ts_waitcnt lgkmcnt(0)"
      : "=&s"(v[0]), "=&s"(v[1]), "=&s"(v[2]), "=&s"(v[3]), "=&s"(v[4]), "=&s"(v[5]), "=&s"(v[6]), "=&s"(v[7]), "=&s"(v[8])
      : "s"(__builtin_amdgcn_kernarg_segment_ptr()), "i"(line(grid)), "i"(line(grid + 1)), "i"(line(grid + 2)),
        "i"(line(grid + 3)), "i"(line(last)));
}

// ---- a whole grid: block t (all of them cost-ordered, heaviest first) of the side x nblk blocks of rows that a
// head's row blocks are cut into, nblk each: row block r, block blk of it as the tile kernels number them
struct GridBlock {
  int r, blk;
};
__device__ __forceinline__ GridBlock grid_block(const GridView& b, int nblk, int t) {
  const int per = b.cyclic ? b.side : nblk, x = t / per, y = t - x * per;
  // (cyclic: equal positions of all row blocks cost the same; contiguous: later row blocks cost more)
  return GridBlock{b.cyclic ? y : b.side - 1 - x, b.cyclic ? x : y};
}
// the same of the key blocks of a column: early keys are seen by more rows
__device__ __forceinline__ GridBlock grid_column(const GridView& b, int nblk, int t) {
  const int per = b.cyclic ? b.side : nblk, x = t / per, y = t - x * per;
  return GridBlock{b.cyclic ? y : x, b.cyclic ? x : y};
}
// token of row i of row block r
__device__ __forceinline__ int grid_token(const GridView& b, int rows, int r, int i) {
  return b.cyclic ? i * b.side + r : r * rows + i;
}

// sub-block that holds local key c (c < nkv)
__device__ __forceinline__ int seg_of_key(const SegList& g, int c) {
  int s = 0;
  while (s + 1 < g.n && c >= g.seg[s + 1].start) ++s;
  return s;
}
// does query row i see local key c (causal mask)?
__device__ __forceinline__ bool seg_visible(const SegList& g, int i, int c) {
  const int s = seg_of_key(g, c);
  return (int64_t)(c - g.seg[s].start) <= (int64_t)i + g.seg[s].rel;
}

// ---- per-process caches of HIP runtime queries (a2d_device.hip; thread-safe) ----
// compute units of the current device
hipError_t device_cus(int* cus);
// raises the kernel's dynamic-LDS limit to `bytes` once per (device, kernel)
hipError_t ensure_dynamic_lds(const void* kernel, int bytes);
// Address of a device array on the current device (the first lookup on a device loads it there)
constexpr int kMaxDevices = 64;
struct SymbolCache {
  std::atomic<void*> at[kMaxDevices];
};
hipError_t symbol_address(const void* symbol, SymbolCache* cache, void** out);
// Debugging aid: route every tile call to the vector-ALU kernels.  The default comes from
// A2D_FORCE_GENERIC=1 in the environment, read once per process; a2d_debug_force_generic() sets it.
bool force_generic();
void set_force_generic(bool on);
// Kernel trace of the calling host thread (diagnostic, see a2d_debug_trace): trace_mark records
// the next caller-supplied event on the stream; a no-op (one thread-local test) when no trace is set.
void trace_set(hipEvent_t* events, int n);
int trace_count();
void trace_mark(hipStream_t s);
// every kernel launch of the method goes through this: the launch, then the trace mark
#define A2D_LAUNCH(kernel, grid, block, lds, stream, ...)               \
  do {                                                                  \
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);  \
    ::a2d::trace_mark(stream);                                          \
  } while (0)

// Scratch memory for the partial results of split walks, offered by the caller's thread for the
// duration of a call (it must stay valid for the stream's work); without an offer, or with NULL from
// it, a call runs unsplit (scratch_offer() in a2d_grid.hpp).  At most kSplitBytes for each of the results a call splits.
bool scratch_offered();
void* scratch_get(size_t bytes);
constexpr size_t kSplitBytes = (size_t)32 << 20;

// ---- splitting a walk ----
// A tile kernel's workgroup owns a block of rows and walks the other side of the tile.  When the row
// blocks are too few for the chip, `parts` workgroups share each block's walk and leave partial
// results that a merge or sum kernel adds up in order.  The time of such a launch is modelled as turns
// of workgroups over the slots of the chip (constants measured on MI355X, microseconds), and the
// number of parts - and the workgroup shape, where a kernel has several - is the one with the least.
struct WalkModel {
  int64_t blocks;          // row blocks
  int slots;               // workgroups, or pairs of workgroups, that the chip holds at a time
  double mean, most;       // steps of a block's walk: on average, the longest
  double step, fixed;      // time of a step, of everything else in a workgroup
  double pair_step, pair_fixed;   // the same of two workgroups that share a slot (0: a slot holds one)
  const double* sorted;    // the steps at 8 places, longest first, as multiples of 1 / `per` (NULL: not known)
  double per;
  double tail = 0.5;       // of a workgroup, while the last turn of uneven walks ends
  bool short_walks = false;   // the chip is not busy enough for its clock to fall
  bool capped = false;        // no more than whole turns of mean walks
};
inline double walk_time(const WalkModel& w, int parts) {
  const auto len = [&](double steps, double step, double fixed) {
    const double n = steps / parts;
    return (n < 1.0 ? 1.0 : n) * step + fixed;
  };
  const int64_t wgs = w.blocks * parts;
  // (uneven walks on more than half of the chip: the longest one runs at the clock of a busy chip)
  if (wgs <= w.slots) return len(w.most, w.step, w.fixed) * (w.mean < w.most && parts == 1 && 2 * wgs > w.slots && !w.short_walks ? 1.05 : 1.0);
  const int64_t turns = (wgs + w.slots - 1) / w.slots;
  const bool pairs = w.pair_step > 0;
  if (w.mean >= w.most)
    return pairs ? turns / 2 * len(w.most, w.pair_step, w.pair_fixed) + turns % 2 * len(w.most, w.step, w.fixed)
                 : turns * len(w.most, w.step, w.fixed);
  const double each = pairs ? 0.5 * len(w.mean, w.pair_step, w.pair_fixed) : len(w.mean, w.step, w.fixed);
  double n = (double)wgs / w.slots + w.tail;                              // longest first
  if (w.capped && n > turns) n = (double)turns;
  const double even = n * each;
  double longest = len(w.most, pairs ? w.pair_step : w.step, w.fixed);
  if (w.sorted && !pairs) {
    // the first walk of the last turn: every slot then holds walks no shorter
    const double last = turns * len(w.sorted[(turns - 1) * w.slots * 8 / wgs] * w.per, w.step, w.fixed);
    if (last > longest) longest = last;
  }
  return even > longest ? even : longest;
}
// the best number of parts up to `cap` (ties: the smaller); a split costs merge_us, a launch behind the
// tile kernel, and part_us per part to write and read back
int best_parts(const WalkModel& w, int cap, double merge_us, double part_us, double* time);
// The time of `a.n` workgroups, as a rule the ones that walk longer, followed by `b.n` others over the slots of the chip
struct Kind {
  int64_t n;
  double mean, most;         // us of a workgroup, on average and at most
};
double one_time(const Kind& a, const Kind& b, int slots, bool uneven, double tail);
// The same of a chip that deals its workgroups (the idle ones of the kernels' placement among them) in turn to shader engines
// of kEngineSlots compute units, whatever these still have to do: the time of the engine that comes out worst.
constexpr int kEngineSlots = 8;
double dealt_time(const Kind& a, const Kind& b, int slots, bool uneven, double tail);
// keys that query row i of the tile sees
int64_t visible_keys(const a2d_tile_desc& d, const SegList& g, int64_t i);
// of 8 rows spread over the tile, last rows first; returns the mean
double mean_visible_keys(const a2d_tile_desc& d, const SegList& g, double seen[8]);

// ---- launchers (none synchronises) ----
// Every tile launcher runs in two phases so that a call can finish everything that may fail on the
// host side before its first kernel is enqueued: PREPARE only raises the dynamic-LDS limits of the
// kernels the LAUNCH phase of the same arguments will use (cached per device), LAUNCH only
// launches and returns the launch's hipError_t.
enum Phase { PREPARE = 0, LAUNCH = 1 };

// the partial an accumulating forward call starts from
struct FwdInput {
  const float *N, *m, *l;
};
// Workgroup shape and parts of a forward tile (sets g->form, g->parts); may_split: partial results
// of parts > 1 workgroups per block ([parts][heads][nq] each of N, m, l) can be stored and merged.
void plan_fwd(const a2d_tile_desc& d, SegList* g, bool may_split, int cus);
void plan_fwd_f32(const a2d_tile_desc& d, SegList* g, int cus, int cap);
void plan_fwd_mfma(const a2d_tile_desc& d, SegList* g, int cus, int cap);
// Parts of the two kernels of a backward tile, each at most its cap, and the dQ kernel's workgroup shape
struct BwdParts {
  int kv, q, form, wide;     // wide: dK/dV in workgroups of 256 keys (launch_dkdv_wide)
  int one, q_first;          // one launch (launch_bwd_one), its dQ workgroups first
  int small;                 // that of launch_bwd_small: 1, or 2: dK and dV in workgroups of their own
  int keep_ds;               // dS handed from dK/dV to dQ
  int delta;                 // fp32: delta by a launch of its own
};
// the kernels of a planned forward or backward, without the launches that merge or sum its parts
void route_fwd(const a2d_tile_desc& d, const SegList& g, Route* r);
void route_bwd(const a2d_tile_desc& d, const BwdParts& p, Route* r);
// Walks of a tile's or grid's dK/dV workgroups (steps of 32 query rows) and dQ workgroups (64 keys): on average, the
// longest; uneven: under a mask, longest first
struct BwdWalks {
  double kv_mean, kv_most, q_mean, q_most;
  bool uneven;
};
double plan_bwd_one(const a2d_tile_desc& d, const SegList& g, const BwdWalks& w, int cus, int cap_kv, int cap_q,
                    BwdParts* best, double* dealt);
BwdParts plan_bwd_f32(const a2d_tile_desc& d, const SegList& g, int cus, int cap_kv, int cap_q);
BwdParts plan_bwd_mfma(const a2d_tile_desc& d, const SegList& g, bool ds, int cus, int cap_kv, int cap_q);

// fp32 tile kernels on the fp32 matrix units (H in {64, 80, 96, 128}); nothing to prepare.
hipError_t launch_fwd_f32(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                          float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s);
hipError_t launch_bwd_f32(const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                          const void* O, const void* dO, const float* lse, float* delta, float* dQ, float* dK,
                          float* dV, const BwdParts& parts, hipStream_t s);

// Generic tile kernels: fp32 arithmetic on the vector ALUs for fp32 or bf16
// inputs, any nq / nkv, H in {64, 80, 96, 128}.  Reached with force_generic() only.
hipError_t launch_fwd_generic(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                              const void* V, float* O_part, float* m, float* l, hipStream_t s);
hipError_t launch_bwd_generic(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                              const void* V, const void* dO, const float* lse, const float* delta, float* dQ,
                              float* dK, float* dV, hipStream_t s);

// delta[head][row] = sum_j dO[head][row][j] * O[head][row][j]  (O, dO with the layouts d.lo, d.ldo)
hipError_t launch_delta(const a2d_tile_desc& d, const void* O, const void* dO, float* delta, hipStream_t s);

// bf16 MFMA tile kernels (H in {64, 80, 96, 128}).  `supported` tells whether the shape is covered.
hipError_t launch_fwd_mfma(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                           const void* V, float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s);
// the forms of 32- and 64-row workgroups (a2d_fwd_small.hip); arguments as of launch_fwd_mfma
hipError_t launch_fwd_small(Phase ph, int rows, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                            const void* V, float* O_part, float* m, float* l, const FwdInput& in, hipStream_t s);
bool bwd_mfma_supported(const a2d_tile_desc& d);
// ds_ws: NULL, or a workspace of bwd_ds_bytes(d, g) (> 0) bytes through which the dK/dV kernel
// hands dS to a contraction-only dQ kernel (instead of the dQ kernel recomputing S and dP)
size_t bwd_ds_bytes(const a2d_tile_desc& d, const SegList& g);
// the dK/dV kernel of 256-key workgroups; dS as in launch_bwd_mfma, NULL or the workspace
hipError_t launch_dkdv_wide(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                            const void* V, const void* dO, const float* lse, const float* delta, float* dK, float* dV,
                            void* dS, hipStream_t s);
// dQ (forms 0 and 1) and dK/dV workgroups in one launch, of a tile or of a whole grid (g.b: lse and delta [heads][seq], the
// gradients in its layouts, of split walks the partial buffers); delta is written where parts.wide, else not used
hipError_t launch_bwd_one(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                          const void* V, const void* O, const void* dO, const float* lse, float* delta, float* dQ,
                          float* dK, float* dV, const BwdParts& parts, hipStream_t s);
// the same in 32-row and 32-key workgroups (a2d_bwd_small.hip); delta is not used
hipError_t launch_bwd_small(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                            const void* V, const void* O, const void* dO, const float* lse, float* dQ, float* dK,
                            float* dV, int q_first, int split, hipStream_t s);
// (parts > 1: the outputs are the partial buffers, [parts][heads][rows][H] each)
hipError_t launch_bwd_mfma(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                           const void* V, const void* O, const void* dO, const float* lse, float* delta, float* dQ,
                           float* dK, float* dV, void* ds_ws, const BwdParts& parts, hipStream_t s);

struct FixPtrs {
  const float* o[A2D_MAX_PARTS];
  const float* m[A2D_MAX_PARTS];
  const float* l[A2D_MAX_PARTS];
};
struct SumPtrs {
  const float* p[A2D_MAX_PARTS];
};
// Layout of a merge's output in the model's dtype: plain != 0 -> [rows][H] contiguous; else row r of
// head h (nq rows per head) starts h * head + r * row elements from the base.
struct OutMap {
  int64_t head;
  int64_t row;
  int nq;
  int plain;
  enum { STRIDED, PLAIN, PLAIN_THROUGH };   // (the last: written straight on to memory, the merges' launcher decides)
};
inline OutMap plain_out() { return OutMap{0, 0, 1, OutMap::PLAIN}; }
// The merged output of a whole emulated grid: block b, head h, row i of the merge's input is token
// i * side + b (cyclic) or b * rows + i of head h in a [heads][side * rows][H] tensor.
struct GridMap {
  int side, rows, heads, cyclic, parts;
};
// O (layout lo), lse of a whole grid from its partial triples; sums of up to three sets of gradient partials
hipError_t launch_fix_grid(const GridMap& gm, int hdim, int out_dtype, const FixPtrs& p, const a2d_layout& lo, void* O,
                           float* lse, hipStream_t s);
struct SumSet {
  SumPtrs p;
  GridMap gm;
  void* out;
  a2d_layout lo;
};
hipError_t launch_sum_grid(int nsets, const SumSet* sets, int hdim, int out_dtype, hipStream_t s);
// out[i] (+)= sum of k partials of n floats that follow one another, up to three sets in one launch
struct PartSet {
  const float* p;
  float* out;
  int64_t n;
  int k, add;
};
hipError_t launch_sum_parts(int nsets, const PartSet* sets, hipStream_t s);

hipError_t launch_fix(int k, int64_t rows, int hdim, int out_dtype, const FixPtrs& p, const OutMap& om, void* O,
                      float* lse, hipStream_t s);
hipError_t launch_attnfix(int k, int64_t rows, int hdim, const FixPtrs& p, float* N, float* m, float* l,
                          hipStream_t s);
// (hv = 4-column groups per row, used only when the output is not plain)
hipError_t launch_fix_bwd(int k, int64_t n, int hv, int out_dtype, const SumPtrs& p, const OutMap& om, void* out,
                          hipStream_t s);
// merge of k NORMALISED partials (O'_k in in_dtype, lse_k)
struct NormPtrs {
  const void* o[A2D_MAX_PARTS];
  const float* lse[A2D_MAX_PARTS];
};
hipError_t launch_fix_norm(int k, int64_t rows, int hdim, int in_dtype, int out_dtype, const NormPtrs& p,
                           const OutMap& om, void* O, float* lse, hipStream_t s);

// plain device copy of n16 16-byte pieces (diagnostic: HBM ceiling and counter calibration)
hipError_t launch_copy_probe(void* dst, const void* src, size_t n16, hipStream_t s);
// MFMA-only ceiling probe (diagnostic)
hipError_t launch_mfma_probe(int blocks, int iters, int random_data, float* scratch, hipStream_t s);
// model of the forward loop: MFMA + one LDS fragment per MFMA + softmax arithmetic (diagnostic)
hipError_t launch_mix_probe(int blocks, int iters, float* scratch, hipStream_t s);
hipError_t launch_bwd_mix_probe(int blocks, int iters, int leave_out, float* scratch, hipStream_t s);
hipError_t launch_lds_read_probe(int blocks, int iters, int kind, float* scratch, hipStream_t s);
int mfma_probe_threads();
int mfma_probe_mfma_per_iter();

}  // namespace a2d
