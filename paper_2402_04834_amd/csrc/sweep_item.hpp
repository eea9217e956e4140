// sweep_item.hpp -- one wavefront's work on a block sweep: SUBS = 64 >> LB consecutive jobs of one sweep, from the
// labels and messages in memory to the updated message (or W_v), around the register sweep of wave_sweep.hpp.
#pragma once
#include "sweep_launch.hpp"
#include "wave_sweep.hpp"

namespace bbp {

__device__ __forceinline__ double wave_sum_d(double v, int lanes) {
  for (int o = lanes / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Convergence distance of a job after an iteration, by one wavefront.
__device__ __forceinline__ double job_delta(const double* terms, int M) {
  double acc = 0.0;
  for (int e = (int)__lane_id(); e < M; e += 64) acc += terms[e];
  return sqrt(fmax(wave_sum_d(acc, 64), 0.0)) / (M > 0 ? M : 1);
}

// entry index of a K-leg dense message with its legs in reverse order
__device__ __forceinline__ int reverse_legs(int idx, int K) { return (int)(__brev((unsigned)idx) >> (32 - K)); }

// floats of LDS that a wavefront of packed sweeps needs: both side messages of every job, the jobs' copies an odd
// number of floats apart so that the jobs' equal-index reads fall on distinct banks
template <int KT, int LB>
constexpr int sweep_lds_floats() { return LB == 6 ? 1 : (64 >> LB) * (2 * (1 << KT) + 1); }

// BF: the contractions with the side messages' middle sites take BF16 operands on the matrix cores (precision
// mode 1; FP32 everywhere else), else FP32 throughout (precision 0). BIASED: some group of the launch has
// biased Pauli noise (otherwise the depolarizing entries are compiled in and the biased selection is removed).
// KP: positions across, 0 where only s.kp tells. job: the lane's job (wave-uniform with LB = 6); active: it takes part
// (inactive lanes follow along on a valid job and write nothing). mode as in sweep_kernel.hip.
// FRESH: the call sits in a loop over sweeps of several shapes: what derives from the lane is formed anew for each (hoisted
// out of the loop, the values of all shapes together spill).
template <bool BF, int KT, int KP, bool TOP, bool BOT, bool SINGLE, bool Q00, bool BIASED, bool FRESH = false>
__device__ __forceinline__ void sweep_item(const SweepArgs& a, int mode, const SweepGroup& G, const SweepDesc& s,
                                           int64_t job, bool active, float* lds) {
  using V = float;
  constexpr int LB = sweep_lane_bits(KP), LANES = 1 << LB, SUBS = 64 / LANES;
  using C = wave::Ctx<V, LB, KP, BIASED>;
  int lane = (int)__lane_id();
  if constexpr (FRESH) asm volatile("" : "+v"(lane));
  const int h = lane & (LANES - 1), sub = lane >> LB;
  if (mode == 0) {
    active = active && !(G.conv && G.conv[job]);
    if (a.gate > 0.0) {
      // residual-gated schedule: skip the update when the message and every input message have settled
      const double* tj = G.terms + job * G.M;
      const double ti = s.msg_init >= 0 ? tj[s.msg_init] : 0.0, tt = s.msg_top >= 0 ? tj[s.msg_top] : 0.0,
                   tb = s.msg_bot >= 0 ? tj[s.msg_bot] : 0.0;
      if (tj[s.msg_out] < a.gate && ti < a.gate && tt < a.gate && tb < a.gate) {
        if (h == 0 && active) G.terms[job * G.M + s.msg_out] = 0.0;
        active = false;
      }
    }
    if (SUBS == 1 ? !active : !__any(active)) return;
  }
  C c;
  c.h = h;
  c.kp_rt = s.kp;
  const int L = 2 * G.d - 1, kp = c.kp(), H = 1 << kp;
  const bool valid = h < H;
  c.geo = s.geo;
  if (G.pdev) {
    const float pj = (float)G.pdev[job >> 2];
    c.p00 = 1.0f - pj;
    c.pe = pj / 3.0f;
  } else {
    c.p00 = G.p00;
    c.pe = G.pe;
  }
  for (int k = 0; k < 4; ++k) {
    c.pib[k] = BIASED ? __float_as_int(G.biased ? G.pi[k] : k == 0 ? c.p00 : c.pe) : 0;
    if constexpr (BIASED && SUBS == 1) c.pib[k] = __builtin_amdgcn_readfirstlane(c.pib[k]);   // (one job: to the scalar unit)
  }
  c.exp2 = 0;

  // labels
  const uint8_t* lab = G.labels + job * L * L;
  auto label_of = [&](int n) {
    const int t = n / kp, i = n - t * kp;
    int r, cc;
    frame_site(s.frame, s.r0, s.c0, s.kr, s.kc, t, i, r, cc);
    return (unsigned)lab[r * L + cc];
  };
  if constexpr (SUBS == 1) {
    const unsigned lb = lane < KT * kp ? label_of(lane) : 0u;
    c.lx = __ballot(lb & 1u);
    c.lz = __ballot(lb & 2u);
  } else {
    constexpr int N = KT * KP, U = (N + LANES - 1) / LANES;   // labels, of each lane
    unsigned lb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) lb[u] = h + LANES * u < N ? label_of(h + LANES * u) & 3u : 0u;
    c.lw[0] = c.lw[1] = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int n = h + LANES * u;
      if (LANES * u < 16) c.lw[0] |= n < 16 ? lb[u] << (2 * n) : 0u;
      if (LANES * (u + 1) > 16) c.lw[1] |= n >= 16 ? lb[u] << (2 * n - 32) : 0u;
    }
    wave::sfor<LB>([&](auto k) {
      c.lw[0] |= wave::xchg<(1 << k)>(c.lw[0]);
      if (N > 16) c.lw[1] |= wave::xchg<(1 << k)>(c.lw[1]);
    });
  }
  // side messages: a sweep toward W or N walks them from their last leg, so read them leg-reversed
  const bool fwd = (s.frame == FRAME_E || s.frame == FRAME_S);
  const float* mbase = G.msgs + job * G.M * MSTRIDE;
  if constexpr (SUBS == 1) {
    const int sl = fwd ? lane : reverse_legs(lane, KT);
    const bool in_msg = lane < (1 << KT);
    c.mtv = V{(TOP && in_msg) ? mbase[s.msg_top * MSTRIDE + sl] : 0.0f};
    c.mbv = V{(BOT && in_msg) ? mbase[s.msg_bot * MSTRIDE + sl] : 0.0f};
  } else if constexpr (TOP || BOT) {
    constexpr int E = 1 << KT, U = (E + LANES - 1) / LANES;
    float* mt = lds + sub * (2 * E + 1);
    float* mb = mt + E;
    float vt[U], vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = h + LANES * u, sl = fwd ? e : reverse_legs(e, KT);
      vt[u] = (TOP && e < E) ? mbase[s.msg_top * MSTRIDE + sl] : 0.0f;
      vb[u] = (BOT && e < E) ? mbase[s.msg_bot * MSTRIDE + sl] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = h + LANES * u;
      if (TOP && e < E) mt[e] = vt[u];
      if (BOT && e < E) mb[e] = vb[u];
    }
    c.mts = mt;
    c.mbs = mb;
    __builtin_amdgcn_wave_barrier();   // (the wavefront's own LDS writes are read in order)
  }

  // message index of this lane's configuration: position i is lane bit pshift(i), message bit kp-1-i
  int mi = 0;
#pragma unroll
  for (int i = 0; i < 6; ++i)
    if (i < kp && (h & (1 << wave::pshift(kp, i)))) mi |= 1 << (kp - 1 - i);

  float x0;
  if (s.msg_init >= 0) {
    x0 = valid ? mbase[s.msg_init * MSTRIDE + mi] : 0.0f;
  } else {
    // the sweep starts at the grid edge: checks whose in-leg leaves the grid are free variables
    const int ia = (s.geo & GEO_IN_EDGE) ? wave::check_lanes(c, Q00) : 0;
    x0 = ((h & ~ia) == 0) ? 1.0f : 0.0f;
  }

  float fin = wave::sweep<V, KT, TOP, BOT, SINGLE, Q00, BF>(x0, c);
  fin = valid ? fin : 0.0f;

  if (mode == 1) {
    // closing contraction with the message from the receiver side (or the grid edge)
    double w = 0.0;
    if (s.msg_close >= 0) w = valid ? (double)mbase[s.msg_close * MSTRIDE + mi] * (double)fin : 0.0;
    else if (h == 0) w = fin;
    w = wave_sum_d(w, LANES);
    if (h == 0 && active)
      G.lnW[job * G.nblocks + s.block] = (w > 0.0) ? c.exp2 * 0.69314718055994530942 + log(w) : NAN;
  } else {
    // normalised new message, damping against the old one (unit norm), distance term. With unit vectors
    // a, b: 2 - 2<a,b>^2 = |a - b|^2 |a + b|^2 / 2, which has no cancellation near convergence in FP32.
    float* mo = G.msgs + job * G.M * MSTRIDE + s.msg_out * MSTRIDE;
    const float old = valid ? mo[mi] : 0.0f;
    const float fn = fin * __builtin_amdgcn_rsqf(wave::wave_sum_sq<LB>(fin));
    const float dm = wave::mul2(a.eta, old, 1.0f - a.eta, fn);
    const float fm = dm * __builtin_amdgcn_rsqf(wave::wave_sum_sq<LB>(dm));
    const float dif = fm - old, sum = fm + old;
    const float dd = wave::wave_sum_sq<LB>(dif), ss = wave::wave_sum_sq<LB>(sum);
    if (valid && active) mo[mi] = fm;
    if (h == 0 && active) G.terms[job * G.M + s.msg_out] = 0.5 * (double)dd * (double)ss;
  }
}

}  // namespace bbp
