// sweep_kernel.hip -- block-sweep kernels for sweeps of BBP_KT steps and BBP_KP positions (this file is compiled
// once per pair, 1..6 each). One wavefront runs one sweep of 64 >> max(BBP_KP, 3) jobs (sweep_item.hpp,
// wave_sweep.hpp).
//   mode 0: BP update of message s.msg_out (Sec. III.D): the new message is normalised (remark 3), damped
//           against the old one (remark 7) and the distance term of the convergence test stored (remark 4);
//   mode 1: closing sweep of block s.block, W_v of the Bethe estimate (Lemma 3.1).
// Grid: one workgroup of one wavefront per item; item = one (jobs, sweep) of one (d, p) group of the launch.
//
// Bound by VALU issue: two instructions per state entry and qubit, which a packed wavefront does for all its jobs at
// once. With the width a template parameter the lane-bit positions, the label lookups and the column's qubit / check
// pattern fold at compile time, the coefficients' lane conditions become scalar masks (one select each) and the
// interior 6 x 6 sweep needs 78 (BF16 cores) or 128 (FP32) registers without spilling. One wavefront per workgroup:
// the wavefront of converged jobs, or one that finishes early, frees its slot at once. Measured, d = 17, 6 x 6 blocks,
// BF16 cores, 4096 syndromes, p = 0.10: 36.6 ms a decode, 52.8 ms with the width a run-time value (three more integer
// divisions per sweep, 1790 against 1174 static VALU instructions); d = 11, 4 x 4 blocks, 1001 syndromes, FP32: 3.05 ms,
// 7.09 ms with one job per wavefront (16 of 64 lanes in use).
#include <hip/hip_runtime.h>

#include "sweep_item.hpp"

#include <utility>

#if !defined(BBP_KT) || !defined(BBP_KP)
#error "compile with -DBBP_KT=<sweep length 1..6> -DBBP_KP=<positions across 1..6>"
#endif
#ifndef BBP_WAVES_PER_EU
#define BBP_WAVES_PER_EU 4   // register budget: at least this many wavefronts per SIMD
#endif

namespace bbp {
namespace {

template <bool BF, int KT, int KP, bool TOP, bool BOT, bool Q00, bool BIASED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(BBP_WAVES_PER_EU)))
void sweep_kernel(SweepArgs a) {
  constexpr int LB = sweep_lane_bits(KP), SUBS = 64 >> LB;
  __shared__ float lds[sweep_lds_floats<KT, LB>()];
  const unsigned item = blockIdx.x;
  int gi = 0;
  for (int k = 1; k < a.ngroups; ++k)
    if (item >= a.g[k].item0) gi = k;
  const SweepGroup& G = a.g[gi];
  unsigned jb, sw;
  // (32-bit: a launch holds fewer than 2^31 items; order 0 divides by the job blocks, order 1 by the sweeps)
  const unsigned q = quotient(item - (unsigned)G.item0, G.by, a.order == 0 ? jb : sw);
  (a.order == 0 ? sw : jb) = q;
  int64_t job = (int64_t)jb * SUBS;
  bool active = true;
  if constexpr (SUBS > 1) {
    job += (int)__lane_id() >> LB;
    active = job < G.jobs;
    job = active ? job : G.jobs - 1;
  }
  sweep_item<BF, KT, KP, TOP, BOT, KP == 1, Q00, BIASED>(a, a.mode, G, G.sweeps[sw], job, active, lds);
}

// variants 0..23: bits 0..2 first site a qubit, bottom and top message present; 8 BF16 middle-site contractions
// (precision 1), 16 biased noise (FP32 only)
// (a sweep of fewer than five steps has no contraction on the matrix cores: both precisions run the FP32 kernel)
template <int V>
void launch_variant(dim3 grid, hipStream_t st, const SweepArgs& a) {
  constexpr bool TOP = (V >> 2) & 1, BOT = (V >> 1) & 1, Q00 = V & 1, BF = ((V >> 3) & 1) && BBP_KT >= 5, BIASED = (V >> 4) & 1;
  sweep_kernel<BF, BBP_KT, BBP_KP, TOP, BOT, Q00, BIASED><<<grid, dim3(64), 0, st>>>(a);
}

template <int... I>
hipError_t dispatch(int variant, dim3 grid, hipStream_t st, const SweepArgs& a, std::integer_sequence<int, I...>) {
  bool done = false;
  ((variant == I ? (launch_variant<I>(grid, st, a), done = true) : false), ...);
  return done ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace

template <>
hipError_t launch_sweeps_of<BBP_KT, BBP_KP>(int variant, unsigned items, hipStream_t st, const SweepArgs& a) {
  return dispatch(variant, dim3(items), st, a, std::make_integer_sequence<int, 24>{});
}

}  // namespace bbp
