// sweep_launch.hpp -- host interface of the block-sweep kernels. The kernels are instantiated per sweep length and
// number of positions across (1..6 each) in separate translation units (sweep_kernel.hip compiled with BBP_KT and
// BBP_KP), the fused ones per block size, remainder and precision (fused_sweep.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "geom.hpp"
#include "plan.hpp"

namespace bbp {

// lane bits of one sweep in the wavefront kernels: its 2^kp configurations, at least 8 (kp = 0: not known at
// compile time, a whole wavefront)
constexpr int sweep_lane_bits(int kp) { return kp == 0 ? 6 : kp < 3 ? 3 : kp; }
// consecutive jobs that one wavefront runs through a sweep of kp positions
constexpr int sweep_jobs_per_wave(int kp) { return 64 >> sweep_lane_bits(kp); }

// x / n for x < 2^31 by one multiply: m = ceil(2^32 / n) is less than 1 above 2^32 / n, so the quotient is at most
// one too large, which the remainder corrects
struct Divide {
  uint32_t n, m;
};
inline Divide divide_by(uint32_t n) { return Divide{n, (uint32_t)(((1ull << 32) + n - 1) / n)}; }
#if defined(__HIP__)
__device__ __forceinline__ unsigned quotient(unsigned x, Divide d, unsigned& rem) {
  unsigned q = d.n == 1 ? x : __umulhi(x, d.m);
  rem = x - q * d.n;
  if ((int)rem < 0) {
    --q;
    rem += d.n;
  }
  return q;
}
#endif

constexpr int MSTRIDE = 64;      // floats per stored message (2^6) for plans whose blocks are at most 6 wide

constexpr int MAX_GROUPS = 8;   // (d, p) groups of one mixed batch

// One (d, p) group of a sweep launch: its sweeps of the launch's class and its job state.
struct SweepGroup {
  const SweepDesc* sweeps;   // the group's sweeps of this class (count of them)
  const uint8_t* labels;     // [job][L*L] coset labels
  float* msgs;               // [job][M][MSTRIDE] dense messages, position 0 most significant
  double* terms;             // [job][M] distance terms of the last update
  const int32_t* conv;       // [job] converged flags (NULL: none has converged)
  double* lnW;               // [job][nblocks] (closing sweeps)
  int64_t jobs;
  int64_t item0;             // first item of the group in the launch
  Divide by;                 // wavefront kernels: the group's job blocks per sweep (order 0) or its sweeps (order 1)
  int32_t count;             // sweeps of this class in the group
  int32_t d, M, nblocks;
  float p00, pe;             // depolarizing noise entries: 1 - p and p / 3
  const double* pdev;        // optional [job / 4] per-syndrome p (overrides p00, pe)
  int32_t biased;            // 1: the qubit entries are pi (Pauli probabilities by code x + 2z)
  float pi[4];
  double pq[4];              // the four Pauli probabilities by code x + 2z in FP64 (truncating kernel)
  int32_t mstride;           // floats per stored message (MSTRIDE unless a block is wider than 6)
  int32_t chi;               // bond dimension (truncating kernel)
};

struct SweepArgs {
  SweepGroup g[MAX_GROUPS];
  int64_t items;             // sum over groups of count * jobs (wavefront kernels: job blocks): one wavefront each
  int32_t ngroups;
  int32_t mode;              // 0: message update, 1: closing sweep (W_v)
  int32_t order;             // item order inside a group: 0 sweep-major (item = sweep * jobs + job), 1 job-major (job blocks)
  int32_t bf16;              // 1: products of BF16-rounded inputs (precision mode 1); 0: FP32 products
  float eta;                 // damping
  int32_t small;             // 1: every block is at most 2x2 tensors: one lane per item (small_sweep.hip)
  double gate;               // > 0: skip an update whose message and input messages all changed by less (terms)
  double* tws;               // truncating kernel: workspace of tws_slots slots of trunc_slot_bytes()
  int64_t tws_slots;         // items per launch of the truncating kernel (larger classes run in chunks)
  int64_t item_base;         // first item of the current chunk
};

// A block update (or closing sum) of small_loop.hip.
struct alignas(16) SmallSweep {
  int16_t r0, c0;   // first site
  int32_t kind;     // (rows == 2, columns == 2, first site a qubit, receiver side): bits 4, 3, 2, 1-0
  int32_t m[4];     // messages entering from E, W, S, N, -1 where there is none
  int32_t out;      // outgoing message (closing: the block)
  int32_t pad;
};
static_assert(sizeof(SmallSweep) == 32, "SmallSweep layout");
struct SmallGroup {
  const SmallSweep* sweeps[3];   // the two colour rounds and the closing sums
  int32_t count[3];
  int32_t* iters;                // [job] results
  double* delta;
};
struct SmallArgs {
  SweepArgs s;                   // group state; items = jobs, one workgroup each
  SmallGroup f[MAX_GROUPS];
  int32_t max_iter, fixed;
  double delta0;
};
// LDS of a job's messages and distance terms; the most that a workgroup may have
constexpr size_t small_loop_lds(int M) { return (size_t)M * 24; }
constexpr size_t SMALL_LOOP_LDS_MAX = 160 * 1024 - 256;
hipError_t launch_small_loop(hipStream_t st, const SmallArgs& a, int threads, size_t lds);

// Sweep classes of the truncating kernel (any length; sweeps with SweepDesc::trunc set): TRUNC_CLASS, and
// TRUNC_CLASS | 1 for the narrow form (trunc_shape.hpp).
constexpr int TRUNC_CLASS = 1 << 12;
inline bool trunc_class(int cls) { return (cls & ~1) == TRUNC_CLASS; }

// workspace bytes of one truncating-kernel item
size_t trunc_slot_bytes();
// launch the a.items truncating sweeps (in chunks of a.tws_slots items), all of the narrow form or none
hipError_t launch_trunc_sweeps(hipStream_t st, const SweepArgs& a, bool narrow);
// the narrow form (trunc_narrow.hip): workspace bytes of one item, launch of one chunk
size_t trunc_narrow_slot_bytes();
void launch_trunc_narrow(unsigned items, hipStream_t st, const SweepArgs& a);

// Class of a sweep: the kernel instantiation that runs it -- length, positions across, caps present, first site a
// qubit: code (((kt - 1) * 6 + kp - 1) * 4 + top * 2 + bottom) * 2 + q00.
inline int sweep_class(const SweepDesc& s) {
  if (s.trunc) return TRUNC_CLASS | (s.trunc == 2 ? 1 : 0);
  return (((s.kt - 1) * 6 + s.kp - 1) * 4 + (s.msg_top >= 0 ? 2 : 0) + (s.msg_bot >= 0 ? 1 : 0)) * 2 +
         ((s.geo & GEO_Q00) ? 1 : 0);
}
inline int class_kt(int cls) { return cls / 48 + 1; }
inline int class_kp(int cls) { return cls / 8 % 6 + 1; }

// Launch the a.items (job, sweep) items of class `cls` on stream st.
hipError_t launch_sweeps(int cls, hipStream_t st, const SweepArgs& a);

// blocks of at most 2x2 tensors, any class, FP32 (small_sweep.hip)
hipError_t launch_small_sweeps(hipStream_t st, const SweepArgs& a);

// per-shape launchers (one translation unit each, 1 <= KT, KP <= 6); variant = class code modulo 8, plus 8 for the
// BF16-input kernels or 16 for the biased-noise kernels
template <int KT, int KP>
hipError_t launch_sweeps_of(int variant, unsigned items, hipStream_t st, const SweepArgs& a);

// All classes of a round in one launch, or a job's whole decode in one workgroup (fused_sweep.hip).
struct FusedGroup {
  const SweepDesc* sweeps[3];   // the two colour rounds and the closing sweeps
  int32_t count[3];
  int32_t* iters;               // [job] results of the loop form
  double* delta;
};
struct FusedArgs {
  SweepArgs s;                  // group state; items = jobs (loop) or jobs * sweeps of the list (round)
  FusedGroup f[MAX_GROUPS];
  int32_t loop;                 // 1: one workgroup per job runs everything; 0: one wavefront per (sweep, job) of `list`
  int32_t list;
  int32_t max_iter, fixed;
  double delta0;
};
// one translation unit each: (K, R) in FUSED_SHAPES, BF 0 or (K >= 5) 1; `groups` workgroups of `waves` wavefronts
template <int K, int R, int BF>
hipError_t launch_fused_of(unsigned groups, int waves, hipStream_t st, const FusedArgs& a);
// block and remainder sizes that occur for odd grid sizes and blocks of 3 to 6 (a grid of one block of 3 or 5 included)
constexpr int FUSED_SHAPES[][2] = {{3, 0}, {3, 1}, {3, 2}, {4, 1}, {4, 3}, {5, 0}, {5, 1},
                                   {5, 2}, {5, 3}, {5, 4}, {6, 1}, {6, 3}, {6, 5}};
constexpr int NUM_FUSED_SHAPES = sizeof(FUSED_SHAPES) / sizeof(FUSED_SHAPES[0]);
hipError_t launch_fused(int shape, bool bf16, unsigned groups, int waves, hipStream_t st, const FusedArgs& a);

}  // namespace bbp
