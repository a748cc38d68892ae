// The recomputing backward of a tile or a whole grid in one launch: the dK/dV workgroups and the dQ workgroups side by
// side, for tiles that fill the chip a few times at most.
//
// In launches one behind the other each ends with compute units that wait for its longest walks, and a small tile pays
// a launch and a kernel's first loads twice.  Neither kind of workgroup needs the other's result but for delta: dQ
// workgroups compute it of their rows anyway, dK/dV workgroups in pairs of the rows they stage (OWN_DELTA: an
// eighth more loads in a step, a dozen vector instructions; a launch of delta_kernel in front costs a small tile more).
// Those of 256 keys have no registers for it at H = 128 and serve tiles where that launch costs 3 %: they read it.
// The kind with the longer walks goes first, but for masked tiles with many keys that few rows see (plan_bwd_one).
#include "a2d_bwd_dq.hpp"
#include "a2d_bwd_pairs.hpp"
#include "a2d_bwd_wide.hpp"

namespace a2d {
namespace {

using namespace mfma;

// WIDE: dK/dV in workgroups of 256 keys, else 128.  KL: key lanes of the dQ workgroups (256 or 128 rows).
template <int HR, bool WIDE, int KL, int GRID>
__global__ __launch_bounds__(512) void bwd_one_kernel(
    a2d_tile_desc d, SegList g, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
    const bf16_t* __restrict__ V, const bf16_t* __restrict__ O, const bf16_t* __restrict__ dO,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dQ, float* __restrict__ dK,
    float* __restrict__ dV, int first, int q_first, int parts_q) {
  warm_arguments<10 * 8 + 12>();
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int id = (int)blockIdx.x < first ? blockIdx.x : blockIdx.x - first;
  if (((int)blockIdx.x < first) == (q_first != 0))
    dq_rows<8, HR, KL, GRID>(id, lds, d, g, parts_q, Q, K, V, O, dO, lse, nullptr, dQ);
  else if constexpr (WIDE)
    dkdv_wide<HR, false, GRID>(id, lds, d, g, g.parts, Q, K, V, dO, lse, delta, dK, dV, nullptr);
  else
    dkdv_pairs<HR, true, false, false, GRID, true>(id, lds, d, g, g.parts, Q, K, V, O, dO, lse, nullptr, dK, dV, nullptr);
}

template <int HR, bool WIDE, int KL, int GRID>
hipError_t go(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
              const void* O, const void* dO, const float* lse, const float* delta, float* dQ, float* dK, float* dV,
              const BwdParts& parts, hipStream_t s) {
  constexpr int HD = padded_head(HR), kv_lds = WIDE ? wk_lds(HD) : DK_LDS, q_lds = dq_launch_lds(HD, KL);
  constexpr int bytes = kv_lds > q_lds ? kv_lds : q_lds;
  if (ph == PREPARE) return ensure_dynamic_lds(reinterpret_cast<const void*>(bwd_one_kernel<HR, WIDE, KL, GRID>), bytes);
  constexpr int keys = WIDE ? WK_KEYS : DK_KEYS, rows = 256 / KL;
  const int side = GRID ? g.b.side : 1, kv_heads = d.heads / g.group;
  const int n_kv = xcd_grid(kv_heads * parts.kv, side * ((d.nkv + keys - 1) / keys));
  const int n_q = xcd_grid(kv_heads * parts.q, side * g.group * ((d.nq + rows - 1) / rows));
  A2D_LAUNCH((bwd_one_kernel<HR, WIDE, KL, GRID>), dim3(n_kv + n_q), dim3(512), bytes, s, d, g, (const bf16_t*)Q,
             (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, (const bf16_t*)dO, lse, delta, dQ, dK, dV,
             parts.q_first ? n_q : n_kv, parts.q_first, parts.q);
  return hipGetLastError();
}

template <int HR>
hipError_t go_h(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K, const void* V,
                const void* O, const void* dO, const float* lse, const float* delta, float* dQ, float* dK, float* dV,
                const BwdParts& parts, hipStream_t s) {
#define A2D_GO(WIDE, KL)                                                                                      \
  return g.b.side == 0 ? go<HR, WIDE, KL, 0>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s)      \
         : g.b.cyclic  ? go<HR, WIDE, KL, 2>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s)      \
                       : go<HR, WIDE, KL, 1>(ph, d, g, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s)
  if (parts.wide && parts.form == 0) { A2D_GO(true, 1); }
  if (parts.wide) { A2D_GO(true, 2); }
  if (parts.form == 0) { A2D_GO(false, 1); }
  A2D_GO(false, 2);
#undef A2D_GO
}

}  // namespace

// Workgroup shapes and parts of a tile or grid whose backward goes out in one launch: the ones with the least time in a
// model of the launch, fitted to 60 shapes x up to 100 choices each (1 x 161 x 308 to 32 x 4096 x 4096, grids of 350
// to 8192 tokens); its choice is 1 % off the best of them in the mean.  Parts of the two kinds are tried in step: of one from a
// list, of the other the fewest that make its walks no longer.
// dealt: the time of the chosen one, unless it is that of few rows, with its workgroups dealt to the chip's shader engines
// (see dealt_time).
double plan_bwd_one(const a2d_tile_desc& d, const SegList& g, const BwdWalks& w, int cus, int cap_kv, int cap_q,
                    BwdParts* best, double* dealt) {
  constexpr double kPairUs[3] = {0.81, 0.94, 1.34}, kWideUs[3] = {0.95, 1.05, 1.61}, kRowUs[3] = {1.57, 1.67, 2.68};
  constexpr double kPairFix = 7, kWideFix = 6.1, kRowFix = 5.5, kLane = 1.2, kLaneFix = 0.45, kTail = 0.26, kMerge = 3.7,
                   kDelta = 2.9, kIdle = 0.93;
  static const int kParts[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
  const int hx = d.hdim > 96 ? 2 : d.hdim > 64 ? 1 : 0, kv_heads = d.heads / g.group, side = g.b.side ? g.b.side : 1;
  const double part_kv = (double)side * kv_heads * d.nkv * d.hdim * 16 / 4.5e6;     // written and read back at 4.5 TB/s
  const double part_q = (double)side * d.heads * d.nq * d.hdim * 8 / 4.5e6;
  double least = 0, rest = 0;
  Kind best_kv = {}, best_q = {};
  *best = BwdParts{};
  for (int wide = 0; wide < 2; ++wide) {
    if (wide && !(d.scale > 1e-30f)) continue;             // (it takes lse / scale, which has to stay finite)
    const int keys = wide ? WK_KEYS : DK_KEYS;
    const int64_t n_kv = (int64_t)kv_heads * side * ((d.nkv + keys - 1) / keys);
    const double kv_step = (wide ? kWideUs : kPairUs)[hx], kv_fix = wide ? kWideFix : kPairFix;
    const double before = wide ? kDelta + part_q / 2 : 0;  // delta_kernel reads O and dO
    for (int form = 0; form < 2; ++form) {
      const int rows = form ? 128 : 256;
      const int64_t n_q = (int64_t)d.heads * side * ((d.nq + rows - 1) / rows);
      const double q_step = kRowUs[hx] * (form ? kLane / 2 : 1), q_fix = kRowFix + (form ? kLaneFix : 0);
      const auto len = [](double steps, int z, double step, double fix, double least_steps) {
        const double n = steps / z;
        return (n < least_steps ? least_steps : n) * step + fix;
      };
      const double q_least = form ? 2 : 1;
      const auto fewest = [](double steps, double step, double room, int cap) {      // parts for walks of `room` us
        const double z = room > 0 ? steps * step / room : cap;
        const int n = z >= cap ? cap : (int)z + (z > (int)z);
        return n < 1 ? 1 : n;
      };
      const auto consider = [&](int zk, int zq) {
        const int64_t all = n_kv * zk + n_q * zq;
        const double busy = all < cus ? kIdle + (1 - kIdle) * all / cus : 1;         // (a chip half idle clocks higher)
        const Kind kv = {n_kv * zk, len(w.kv_mean, zk, kv_step * busy, kv_fix, 1), len(w.kv_most, zk, kv_step * busy, kv_fix, 1)};
        const Kind q = {n_q * zq, len(w.q_mean, zq, q_step * busy, q_fix, q_least), len(w.q_most, zq, q_step * busy, q_fix, q_least)};
        const bool q_first = q.most > kv.most;
        const double more = before + (zk > 1 || zq > 1 ? kMerge : 0) + (zk > 1 ? zk * part_kv : 0) + (zq > 1 ? zq * part_q : 0);
        const double t = more + (q_first ? one_time(q, kv, cus, w.uneven, kTail) : one_time(kv, q, cus, w.uneven, kTail));
        if (best->one && t >= least) return;
        least = t;
        rest = more;
        best_kv = kv;
        best_q = q;
        *best = BwdParts{zk, zq, form, wide, 1, q_first};
      };
      for (int z : kParts) {
        if (z > 1 && (z > cap_kv || z > w.kv_most)) break;
        const int most_q = cap_q < (int)w.q_most ? cap_q : (int)w.q_most;
        consider(z, fewest(w.q_most, q_step, len(w.kv_most, z, kv_step, kv_fix, 1) - q_fix, most_q < 1 ? 1 : most_q));
        if (z > 1) consider(z, 1);
      }
      for (int z : kParts) {
        if (z > 1 && (z > cap_q || z > w.q_most)) break;
        const int most_kv = cap_kv < (int)w.kv_most ? cap_kv : (int)w.kv_most;
        consider(fewest(w.kv_most, kv_step, len(w.q_most, z, q_step, q_fix, q_least) - kv_fix, most_kv < 1 ? 1 : most_kv), z);
        if (z > 1) consider(1, z);
      }
      consider(1, 1);
    }
  }
  // 32 rows or keys a workgroup (a2d_bwd_small.hip; a step is a round of 256).  Fitted to 92 shapes of 1 x 41 x 80 to 16 x 512 x 512,
  // 1 x 4096 x 4096: taken up to some 256 of them with walks of 2048, 512 with walks of 512 (under a mask 1024); 1.27 times as
  // fast in the mean there as without that form, 0.5 % off the better of the two.
  constexpr double kSmallKvUs[3] = {1.65, 2.8, 3.0}, kSmallKvFix[3] = {5.3, 5.9, 7.4}, kSmallRowUs[3] = {1.24, 1.69, 2.2},
                   kSmallRowFix[3] = {5.3, 5.9, 7.0}, kSmallIdle = 0.88;
  const int64_t n_kv = (int64_t)kv_heads * side * ((d.nkv + 31) / 32), n_q = (int64_t)d.heads * side * ((d.nq + 31) / 32);
  const double busy = n_kv + n_q < cus ? kSmallIdle + (1 - kSmallIdle) * (n_kv + n_q) / cus : 1;
  const auto of = [&](double rounds, const double* step, const double* fix) { return ((rounds < 1 ? 1 : rounds) * step[hx] + fix[hx]) * busy; };
  const Kind kv = {n_kv, of(w.kv_mean / 8, kSmallKvUs, kSmallKvFix), of(w.kv_most / 8, kSmallKvUs, kSmallKvFix)};
  const Kind q = {n_q, of(w.q_mean / 4, kSmallRowUs, kSmallRowFix), of(w.q_most / 4, kSmallRowUs, kSmallRowFix)};
  const bool q_first = q.most > kv.most;
  const double small = q_first ? one_time(q, kv, cus, w.uneven, kTail) : one_time(kv, q, cus, w.uneven, kTail);
  // (the other model is some 10 % low at few workgroups and with uneven walks at H = 64, this one at many: 7 heads, 3186 tokens on
  // 2 x 2, H = 128, causal 144 us against 120; 15 heads, 936 tokens, H = 64 28 against 33)
  const double trust = n_kv + n_q <= 3 * (int64_t)cus ? 1.04 : w.uneven && hx == 0 ? 1.15 : 0.94;
  if (small < trust * least) {
    // (dK and dV apart where all workgroups run at once, see a2d_bwd_small.hip.  The choice above prices them together, up to a third
    // too high for such calls: near the line one may go out in the other form though this one is faster.)
    *best = BwdParts{1, 1, 0, 0, 1, q_first, n_q + 2 * n_kv <= cus ? 2 : 1};
    return small;
  }
  const int keys = best->wide ? WK_KEYS : DK_KEYS, rows = best->form ? 128 : 256;
  const Kind chosen_kv = best_kv, chosen_q = best_q;
  best_kv.n = xcd_grid(kv_heads * best->kv, side * ((d.nkv + keys - 1) / keys));
  best_q.n = xcd_grid(kv_heads * best->q, side * g.group * ((d.nq + rows - 1) / rows));
  // (Under a mask most key blocks may be seen by few rows or none, which leaves dK / dV one long walk and many short ones, each
  // still with its prologue and its rows to store: behind them the dQ walks start late.  us, dK / dV first / dQ first: 40 x
  // 496 x 2977, H = 128 53.8 / 41.7, 46 x 717 x 4521 86.8 / 71.5, 14 x 339 x 4617 34.6 / 29.2, 44 x 282 x 872, H = 80 22.9 / 19.6.
  // Both times are those of the order that is launched: of 13100 masked shapes of two to six turns 55 go out otherwise than by the
  // times of the other order, 1.04 times as fast in the mean (124/31 x 782 x 5816, H = 64 133 -> 113, at worst 100/25 x 829 x 10756,
  // H = 96 144 -> 157).  The shapes are chosen by the other one: with this one's times in
  // that choice 39 of 28000 drawn shapes changed, as many for the worse, 20 x 572 x 9758, H = 80 56 -> 78, as for the better.)
  if (w.uneven && !g.b.side && best_q.mean > best_kv.mean && best_kv.n + best_q.n > cus && !best->q_first) {
    best->q_first = 1;
    least = rest + one_time(chosen_q, chosen_kv, cus, true, kTail);
  }
  *dealt = rest + (best->q_first ? dealt_time(best_q, best_kv, cus, w.uneven, kTail) : dealt_time(best_kv, best_q, cus, w.uneven, kTail));
  return least;
}

hipError_t launch_bwd_one(Phase ph, const a2d_tile_desc& d, const SegList& g, const void* Q, const void* K,
                          const void* V, const void* O, const void* dO, const float* lse, float* delta, float* dQ,
                          float* dK, float* dV, const BwdParts& parts, hipStream_t s) {
  if (parts.small) return launch_bwd_small(ph, d, g, Q, K, V, O, dO, lse, dQ, dK, dV, parts.q_first, parts.small > 1, s);
  SegList go = g;
  go.parts = parts.kv;
  if (parts.q > 1) go.acc = 0;                             // (the sum over the parts adds)
  if (ph == LAUNCH && parts.wide) {
    a2d_tile_desc all = d;                                 // delta of the tile, or of the whole sequence
    if (g.b.side) {
      all.nq = g.b.side * d.nq;
      all.lo.row = g.b.cyclic ? g.b.o : d.lo.row;
      all.ldo.row = g.b.cyclic ? g.b.g : d.ldo.row;
    }
    const hipError_t e = launch_delta(all, O, dO, delta, s);
    if (e != hipSuccess) return e;
  }
  switch (d.hdim) {
    case 128: return go_h<128>(ph, d, go, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
    case 96: return go_h<96>(ph, d, go, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
    case 80: return go_h<80>(ph, d, go, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
    default: return go_h<64>(ph, d, go, Q, K, V, O, dO, lse, delta, dQ, dK, dV, parts, s);
  }
}

}  // namespace a2d
