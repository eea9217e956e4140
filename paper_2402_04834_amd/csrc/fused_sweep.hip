// fused_sweep.hip -- the block sweeps of all classes of a colour round in one launch, or a job's whole belief
// propagation in one workgroup, for decodes too small to fill the chip (this file is compiled once per block size
// BBP_K, remainder size BBP_R and precision BBP_BF). The class launches of sweep_kernel.hip need a launch per class
// and round, some 350 for one d = 17 decode, and a small round is over long before the next launch has started.
//   round   one wavefront per (job, sweep) of a launch list, the heavy classes first; the caller launches the
//           distance kernel after every second round as for the class launches;
//   loop    one workgroup per job: the iterations run inside the kernel, its wavefronts sharing out a round's sweeps
//           between barriers, until the job has converged; then the closing sweeps. Nothing waits for another
//           workgroup, so the kernel ends whatever order they run in. A workgroup's wavefronts sit on one CU and see
//           each other's messages through its cache after a barrier.
// A wavefront picks its sweep's instantiation by five uniform branches; the sweeps are those of sweep_item.hpp, so every
// route gives the same bits. Blocks of at most BBP_K x BBP_K with one other size along the edges, the depolarizing
// noise; everything else takes the class launches.
#include <hip/hip_runtime.h>

#include "sweep_item.hpp"

#include <algorithm>

#if !defined(BBP_K) || !defined(BBP_R) || !defined(BBP_BF)
#error "compile with -DBBP_K=<block size> -DBBP_R=<remainder, 0: none> -DBBP_BF=<0, 1>"
#endif

namespace bbp {
namespace {

constexpr int KB = BBP_K, RB = BBP_R;
constexpr bool BF = BBP_BF != 0;

constexpr int lds_floats(int kt, int kp) {
  const int lb = sweep_lane_bits(kp);
  return lb == 6 ? 1 : (64 >> lb) * (2 * (1 << kt) + 1);
}
// LDS floats of one wavefront: the most of the shapes that occur
constexpr int LDSF = std::max(std::max(lds_floats(KB, KB), RB ? lds_floats(RB, RB) : 1),
                              RB ? std::max(lds_floats(KB, RB), lds_floats(RB, KB)) : 1);

template <int KT, int KP>
__device__ __forceinline__ void shape_sweep(const SweepArgs& a, int mode, const SweepGroup& G, const SweepDesc& s,
                                            int64_t job, float* lds) {
  const bool active = ((int)__lane_id() >> sweep_lane_bits(KP)) == 0;   // one job: the first lanes
  auto run = [&](auto top, auto bot, auto q00) {
    sweep_item<BF, KT, KP, decltype(top)::value, decltype(bot)::value, KP == 1, decltype(q00)::value, false, true>(
        a, mode, G, s, job, active, lds);
  };
  auto run2 = [&](auto top, auto bot) {
    if (s.geo & GEO_Q00) run(top, bot, std::true_type{});
    else run(top, bot, std::false_type{});
  };
  auto run1 = [&](auto top) {
    if (s.msg_bot >= 0) run2(top, std::true_type{});
    else run2(top, std::false_type{});
  };
  if (s.msg_top >= 0) run1(std::true_type{});
  else run1(std::false_type{});
}

// a sweep record through the scalar unit (the tables do not change while a kernel runs)
__device__ __forceinline__ SweepDesc load_sweep(const SweepDesc* p) {
  typedef const __attribute__((address_space(4))) int32_t* cptr;
  const cptr q = (cptr)(uintptr_t)p;
  SweepDesc s;
  int32_t* w = (int32_t*)&s;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(SweepDesc) / 4); ++i) w[i] = q[i];
  return s;
}

// 128 registers: 16 wavefronts of a workgroup fill a CU's SIMDs
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void fused_kernel(FusedArgs a) {
  extern __shared__ float lds[];
  __shared__ double distance;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const unsigned item = blockIdx.x;
  int gi = 0;
  for (int k = 1; k < a.s.ngroups; ++k)
    if (item >= a.s.g[k].item0) gi = k;
  const SweepGroup& G = a.s.g[gi];
  const FusedGroup& F = a.f[gi];
  unsigned job = item - (unsigned)G.item0, sweep = 0;
  int list = 0, it = 0;
  if (!a.loop) {
    sweep = quotient(job, G.by, job);
    list = a.list;
  }
  for (;;) {
    const int count = F.count[list];
    for (int i = a.loop ? wave : (int)sweep; i < count; i += a.loop ? waves : count) {
      const SweepDesc s = load_sweep(F.sweeps[list] + (count - 1 - i));   // the lists end with the widest sweeps
      float* mine = lds + wave * LDSF;
      const int mode = list == 2 ? 1 : 0;
      if constexpr (RB == 0) {
        shape_sweep<KB, KB>(a.s, mode, G, s, job, mine);
      } else {
        constexpr int R = RB > 0 ? RB : 1;
        if (s.kp == KB) {
          if (s.kt == KB) shape_sweep<KB, KB>(a.s, mode, G, s, job, mine);
          else shape_sweep<R, KB>(a.s, mode, G, s, job, mine);
        } else {
          if (s.kt == KB) shape_sweep<KB, R>(a.s, mode, G, s, job, mine);
          else shape_sweep<R, R>(a.s, mode, G, s, job, mine);
        }
      }
    }
    if (!a.loop || list == 2) return;
    __syncthreads();
    if (list == 0) {
      list = 1;
      continue;
    }
    // the iteration's distance (convergence test of Alg. 1)
    if (wave == 0) {
      const double dl = job_delta(G.terms + (int64_t)job * G.M, G.M);
      if (threadIdx.x == 0) distance = dl;
    }
    __syncthreads();
    ++it;
    list = 0;
    if (it == a.max_iter || (!a.fixed && distance < a.delta0)) {
      if (threadIdx.x == 0) {
        F.delta[job] = distance;
        F.iters[job] = it;
      }
      list = 2;
    }
  }
}

}  // namespace

template <>
hipError_t launch_fused_of<BBP_K, BBP_R, BBP_BF>(unsigned groups, int waves, hipStream_t st, const FusedArgs& a) {
  fused_kernel<<<dim3(groups), dim3(64 * waves), waves * LDSF * sizeof(float), st>>>(a);
  return hipGetLastError();
}

}  // namespace bbp
