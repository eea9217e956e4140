// small_loop.hip -- the whole belief propagation of a job in one workgroup, for blocks of at most 2x2 tensors
// (block size 1 is plain BP between single tensors): the messages and distance terms live in LDS, a lane contracts one
// block at a time as in small_sweep.hip, and the iterations run inside the kernel. Bound by FP32 issue: an update of a
// 2x2 block is 64 assignments of four products and a sum each.
//
// Against a launch per class and round (small_sweep.hip, which serves plans whose messages exceed the LDS and timed
// decodes): its messages of four floats lie 256 bytes apart in memory and moved 64 to 128 bytes per access, and its
// assignments were decoded bit by bit for blocks of any shape. Here the shape, the parity of the first site and the
// receiving side are compile-time, so every assignment's entries are registers; a wavefront whose lanes hold several
// kinds takes them one after the other, and the lists are sorted so that few do. d = 17, 2x2 blocks, 2048
// syndromes: 32.9 -> 4.0 ms for the decode, 3.2 ms of it here.
//
// Every product and sum keeps its order and rounding (nothing is fused but what is written so), so both routes give the
// same bits. A workgroup waits for no other; it ends when its job has converged or at max_iter.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "geom.hpp"
#include "sweep_item.hpp"
#include "sweep_launch.hpp"

#pragma clang fp contract(off)

namespace bbp {
namespace {

constexpr int SIDE_E = 0, SIDE_W = 1, SIDE_S = 2, SIDE_N = 3;

template <class F, int... J>
__device__ __forceinline__ void for_each(std::integer_sequence<int, J...>, F&& f) {
  (f(std::integral_constant<int, J>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void for_each(F&& f) {
  for_each(std::make_integer_sequence<int, N>(), f);
}

// A block of KR x KC tensors whose first site is a qubit (Q00) or a check. Variables are the checks of the block and of
// its one-site halo, numbered (dr + 1) * 4 + dc + 1; an assignment is a 16-bit mask.
template <int KR, int KC, bool Q00>
struct Shape {
  static constexpr int pos(int dr, int dc) { return (dr + 1) * 4 + dc + 1; }
  static constexpr bool check(int dr, int dc) { return ((dr + dc + (Q00 ? 0 : 1)) & 1) != 0; }
  static constexpr int legs(int side) { return side <= SIDE_W ? KR : KC; }
  // inside site of leg i of a side, and the outside one across it
  static constexpr int in_r(int side, int i) { return side <= SIDE_W ? i : side == SIDE_S ? KR - 1 : 0; }
  static constexpr int in_c(int side, int i) { return side == SIDE_E ? KC - 1 : side == SIDE_W ? 0 : i; }
  static constexpr int out_r(int side, int i) { return side == SIDE_S ? KR : side == SIDE_N ? -1 : i; }
  static constexpr int out_c(int side, int i) { return side == SIDE_E ? KC : side == SIDE_W ? -1 : i; }
  // the variable a leg carries: whichever of its sites is a check
  static constexpr int leg(int side, int i) {
    return check(in_r(side, i), in_c(side, i)) ? pos(in_r(side, i), in_c(side, i)) : pos(out_r(side, i), out_c(side, i));
  }
  // the legs of a side whose variable lies outside the block (0 where the side leaves the grid)
  static constexpr int outside(int side) {
    int m = 0;
    for (int i = 0; i < legs(side); ++i)
      if (!check(in_r(side, i), in_c(side, i))) m |= 1 << leg(side, i);
    return m;
  }
  static constexpr int entry(int side, int x) {   // message index of assignment x, leg 0 most significant
    int e = 0;
    for (int i = 0; i < legs(side); ++i) e = e << 1 | (x >> leg(side, i) & 1);
    return e;
  }
  static constexpr int qubits() {
    int n = 0;
    for (int dr = 0; dr < KR; ++dr)
      for (int dc = 0; dc < KC; ++dc) n += check(dr, dc) ? 0 : 1;
    return n;
  }
  static constexpr int site(int q) {   // the q-th qubit, row-major: dr * 2 + dc
    for (int dr = 0; dr < KR; ++dr)
      for (int dc = 0; dc < KC; ++dc)
        if (!check(dr, dc) && q-- == 0) return dr * 2 + dc;
    return -1;
  }
  static constexpr int used() {
    int m = 0;
    for (int dr = 0; dr < KR; ++dr)
      for (int dc = 0; dc < KC; ++dc)
        if (check(dr, dc)) m |= 1 << pos(dr, dc);
        else m |= 1 << pos(dr - 1, dc) | 1 << pos(dr, dc - 1) | 1 << pos(dr + 1, dc) | 1 << pos(dr, dc + 1);
    return m;
  }
  static constexpr int fixed(int side) {
    int m = 0;
    for (int i = 0; i < legs(side); ++i) m |= 1 << leg(side, i);
    return m;
  }
  static constexpr int values(int side, int h) {   // the variables of entry h of the side's message
    int x = 0;
    for (int i = 0; i < legs(side); ++i) x |= (h >> (legs(side) - 1 - i) & 1) << leg(side, i);
    return x;
  }
};
constexpr int deposit(int n, int mask) {   // the bits of n at the set bits of mask, low to high
  int x = 0;
  for (int b = 0; b < 16; ++b)
    if (mask >> b & 1) {
      x |= (n & 1) << b;
      n >>= 1;
    }
  return x;
}

typedef float floats4 __attribute__((ext_vector_type(4), aligned(4)));   // (a workspace is the caller's)

struct Job {
  const uint8_t* lab;   // labels of the job's grid
  int L;
  float pi[4];          // Pauli probabilities by code x + 2z
};

// The block's sum over its assignments. OUT: the receiving side, whose message entries fin[] are formed (side OUT's
// own message is left out); or, CLOSE, the closing sum over all four messages. EDGE: some lane's block lies at the edge
// of the grid: a missing side's message counts as 1 and the variables outside it are 0.
template <int KR, int KC, bool Q00, int OUT, bool EDGE, bool CLOSE>
__device__ __forceinline__ double contract(const Job& j, const SmallSweep& s, const float4* msgs, float (&fin)[4]) {
  using S = Shape<KR, KC, Q00>;
  constexpr int NQ = S::qubits();
  float t[NQ > 0 ? NQ : 1][4];   // qubit entries by (up ^ down) * 2 + (left ^ right)
  for_each<NQ>([&](auto Q) __attribute__((always_inline)) {
    constexpr int q = decltype(Q)::value, dr = S::site(q) >> 1, dc = S::site(q) & 1;
    const int r = s.r0 + dr, lb = j.lab[r * j.L + s.c0 + dc] & 3;
    // horizontal edge (even row): checks above / below flip x, left / right flip z; vertical edge: swapped
    const bool vert = (r & 1) != 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int swapped = (e & 1) << 1 | e >> 1, code = lb ^ (vert ? e : swapped);
      const float lo = (code & 1) ? j.pi[1] : j.pi[0], hi = (code & 1) ? j.pi[3] : j.pi[2];
      t[q][e] = (code & 2) ? hi : lo;
    }
  });
  float m[4][4];
  bool gone[4];
#pragma unroll
  for (int side = 0; side < 4; ++side) {
    gone[side] = false;
    if (!CLOSE && side == OUT) continue;
    const float4 v = msgs[s.m[side] < 0 ? 0 : s.m[side]];
    gone[side] = EDGE && s.m[side] < 0;
    m[side][0] = gone[side] ? 1.0f : v.x;
    m[side][1] = gone[side] ? 1.0f : v.y;
    m[side][2] = gone[side] ? 1.0f : v.z;
    m[side][3] = gone[side] ? 1.0f : v.w;
  }
  // weight of assignment x; 0 where a variable off the grid is set
  auto weight = [&](auto X) __attribute__((always_inline)) -> float {
    constexpr int x = decltype(X)::value;
    float w = 1.0f;
    for_each<NQ>([&](auto Q) __attribute__((always_inline)) {
      constexpr int q = decltype(Q)::value, dr = S::site(q) >> 1, dc = S::site(q) & 1;
      constexpr int ud = (x >> S::pos(dr - 1, dc) ^ x >> S::pos(dr + 1, dc)) & 1;
      constexpr int lr = (x >> S::pos(dr, dc - 1) ^ x >> S::pos(dr, dc + 1)) & 1;
      w = w * t[q][ud * 2 + lr];
    });
    bool off = false;
    for_each<4>([&](auto D) __attribute__((always_inline)) {
      constexpr int side = decltype(D)::value;
      if constexpr (CLOSE || side != OUT) {
        w = w * m[side][S::entry(side, x)];
        if constexpr (EDGE && (x & S::outside(side)) != 0) off = off || gone[side];
      }
    });
    return EDGE && off ? 0.0f : w;
  };
  constexpr int free = CLOSE ? S::used() : S::used() & ~S::fixed(OUT);
  constexpr int N = 1 << __builtin_popcount(free);
  if constexpr (CLOSE) {
    double W = 0.0;
    for_each<N>([&](auto I) __attribute__((always_inline)) {
      W += (double)weight(std::integral_constant<int, deposit(N - 1 - decltype(I)::value, free)>());
    });
    return W;
  } else {
    for_each<1 << S::legs(OUT)>([&](auto H) __attribute__((always_inline)) {
      constexpr int base = S::values(OUT, decltype(H)::value);
      float acc = 0.0f;
      for_each<N>([&](auto I) __attribute__((always_inline)) {
        acc += weight(std::integral_constant<int, base | deposit(N - 1 - decltype(I)::value, free)>());
      });
      fin[decltype(H)::value] = acc;
    });
    return 0.0;
  }
}

template <int KR, int KC, bool Q00, int OUT, bool CLOSE>
__device__ __forceinline__ double contract_at(const Job& j, const SmallSweep& s, const float4* msgs, float (&fin)[4]) {
  if constexpr (KR * KC == 4 && !CLOSE) {
    bool edge = false;
#pragma unroll
    for (int side = 0; side < 4; ++side) edge |= side != OUT && s.m[side] < 0;
    if (!__any(edge)) return contract<KR, KC, Q00, OUT, false, CLOSE>(j, s, msgs, fin);
  }
  return contract<KR, KC, Q00, OUT, true, CLOSE>(j, s, msgs, fin);
}

// the lane's block, of kind `kind` (uniform; 2x2 blocks start at even rows and columns: with a qubit)
template <bool CLOSE>
__device__ __forceinline__ double contract_kind(int kind, const Job& j, const SmallSweep& s, const float4* msgs,
                                                float (&fin)[4]) {
  double W = 0.0;
  auto shape = [&](auto kr, auto kc, auto q00) __attribute__((always_inline)) {
    constexpr int R = decltype(kr)::value, C = decltype(kc)::value;
    constexpr bool Q = decltype(q00)::value;
    if constexpr (CLOSE) {   // (the sum is the same from whichever side)
      W = contract_at<R, C, Q, SIDE_E, true>(j, s, msgs, fin);
    } else {
      switch (kind & 3) {
        case SIDE_E: contract_at<R, C, Q, SIDE_E, false>(j, s, msgs, fin); break;
        case SIDE_W: contract_at<R, C, Q, SIDE_W, false>(j, s, msgs, fin); break;
        case SIDE_S: contract_at<R, C, Q, SIDE_S, false>(j, s, msgs, fin); break;
        default: contract_at<R, C, Q, SIDE_N, false>(j, s, msgs, fin); break;
      }
    }
  };
  using one = std::integral_constant<int, 1>;
  using two = std::integral_constant<int, 2>;
  switch (kind >> 2) {
    case 7: shape(two(), two(), std::true_type()); break;
    case 5: shape(two(), one(), std::true_type()); break;
    case 4: shape(two(), one(), std::false_type()); break;
    case 3: shape(one(), two(), std::true_type()); break;
    case 2: shape(one(), two(), std::false_type()); break;
    case 1: shape(one(), one(), std::true_type()); break;
    default: shape(one(), one(), std::false_type()); break;
  }
  return W;
}

// f(kind) for every kind among the active lanes' `kind`, with those lanes active
template <class F>
__device__ __forceinline__ void by_kind(int kind, F&& f) {
  uint64_t rest = __ballot(1);
  while (rest) {
    const int k = __builtin_amdgcn_readlane(kind, __builtin_ctzll(rest));
    const bool mine = kind == k;
    rest &= ~__ballot(mine);
    if (mine) f(k);
  }
}

// sum of four squares: the first unrounded onto the second's
__device__ __forceinline__ float squares(const float (&x)[4]) {
  return fmaf(x[3], x[3], fmaf(x[2], x[2], fmaf(x[0], x[0], x[1] * x[1])));
}

__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void small_loop_kernel(SmallArgs a) {
  extern __shared__ float4 msgs[];   // [M], then the distance terms (double) [M]
  __shared__ double distance;
  const unsigned item = blockIdx.x;
  int gi = 0;
  for (int k = 1; k < a.s.ngroups; ++k)
    if (item >= a.s.g[k].item0) gi = k;
  const SweepGroup& G = a.s.g[gi];
  const SmallGroup& F = a.f[gi];
  const int64_t job = item - G.item0;
  const int M = G.M;
  double* terms = (double*)(msgs + M);
  float* gm = G.msgs + job * M * MSTRIDE;
  for (int e = threadIdx.x; e < M; e += blockDim.x) {
    const floats4 v = *(const floats4*)(gm + (int64_t)e * MSTRIDE);
    msgs[e] = make_float4(v.x, v.y, v.z, v.w);
    terms[e] = INFINITY;
  }
  Job j;
  j.L = 2 * G.d - 1;
  j.lab = G.labels + job * j.L * j.L;
  if (G.biased) {
#pragma unroll
    for (int k = 0; k < 4; ++k) j.pi[k] = G.pi[k];
  } else {
    j.pi[0] = G.p00;
    float pe = G.pe;
    if (G.pdev) {
      const float pj = (float)G.pdev[job >> 2];
      j.pi[0] = 1.0f - pj;
      pe = pj / 3.0f;
    }
    j.pi[1] = j.pi[2] = j.pi[3] = pe;
  }
  __syncthreads();

  for (int it = 1;; ++it) {
    for (int list = 0; list < 2; ++list) {
      const int count = F.count[list];
      for (int i = threadIdx.x; i < count; i += blockDim.x) {
        const SmallSweep s = F.sweeps[list][i];
        if (s.kind < 0) continue;   // padding
        const int out = s.out;
        if (a.s.gate > 0.0) {
          // residual-gated schedule: skip the update when the message and every input message have settled
          bool settled = terms[out] < a.s.gate;
#pragma unroll
          for (int side = 0; side < 4; ++side)
            if (s.m[side] >= 0) settled = settled && terms[s.m[side]] < a.s.gate;
          if (settled) {
            terms[out] = 0.0;
            continue;
          }
        }
        float fin[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        by_kind(s.kind, [&](int k) __attribute__((always_inline)) { contract_kind<false>(k, j, s, msgs, fin); });
        // normalised new message, damping against the old one, distance term
        const float ss = squares(fin);
        const float rn = ss > 0.0f ? __builtin_amdgcn_rsqf(ss) : 0.0f;
        const float4 o = msgs[out];
        const float old[4] = {o.x, o.y, o.z, o.w};
        float dm[4], df[4], sf[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) dm[h] = fmaf(a.s.eta, old[h], (1.0f - a.s.eta) * (fin[h] * rn));
        const float t2 = squares(dm);
        const float rd = t2 > 0.0f ? __builtin_amdgcn_rsqf(t2) : 0.0f;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          dm[h] = dm[h] * rd;
          df[h] = dm[h] - old[h];
          sf[h] = dm[h] + old[h];
        }
        msgs[out] = make_float4(dm[0], dm[1], dm[2], dm[3]);
        terms[out] = 0.5 * (double)squares(df) * (double)squares(sf);
      }
      __syncthreads();
    }
    // the iteration's distance (convergence test of Alg. 1)
    if (threadIdx.x < 64) {
      const double dl = job_delta(terms, M);
      if (threadIdx.x == 0) distance = dl;
    }
    __syncthreads();
    if (it == a.max_iter || (!a.fixed && distance < a.delta0)) {
      if (threadIdx.x == 0) {
        F.delta[job] = distance;
        F.iters[job] = it;
      }
      break;
    }
    __syncthreads();   // everyone has read the distance
  }
  for (int e = threadIdx.x; e < M; e += blockDim.x) {
    const float4 v = msgs[e];
    *(floats4*)(gm + (int64_t)e * MSTRIDE) = floats4{v.x, v.y, v.z, v.w};
  }
  for (int i = threadIdx.x; i < F.count[2]; i += blockDim.x) {
    const SmallSweep s = F.sweeps[2][i];
    if (s.kind < 0) continue;
    double W = 0.0;
    float none[4];
    by_kind(s.kind, [&](int k) __attribute__((always_inline)) { W = contract_kind<true>(k, j, s, msgs, none); });
    G.lnW[job * G.nblocks + s.out] = (W > 0.0) ? log(W) : NAN;
  }
}

}  // namespace

hipError_t launch_small_loop(hipStream_t st, const SmallArgs& a, int threads, size_t lds) {
  if (a.s.items <= 0) return hipSuccess;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)small_loop_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  small_loop_kernel<<<dim3((unsigned)a.s.items), dim3(threads), lds, st>>>(a);
  return hipGetLastError();
}

}  // namespace bbp
