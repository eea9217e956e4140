// trunc_narrow.hip -- truncating block sweeps whose every bond stays within 8 (trunc_shape.hpp): the algorithm of
// trunc_sweep.hip (boundary MPS of the in-block sweep, QR sweep down and truncating sweep up after every column, FP64)
// in a form of its own.
//
// What it is bound by: FP64 instruction issue and the serial chains of reflections and Jacobi rounds. Against the
// general kernel on these shapes:
//   * the state is held at the bonds' sizes: 167 registers and 10.3 KB of LDS, three wavefronts per SIMD instead of two
//     (four, at 128 registers, spill 31 of them);
//   * a bond's size is the number of singular values kept at it (those above 1e-13 of the norm: 5 on average for a 6 x 6
//     block at chi 8), and absorptions, factorisations, reflections and Jacobi rounds leave out the rows and columns
//     that are zero beyond it;
//   * sums over lanes go through DPP and lane swaps, stored reflections are staged in LDS while the previous bond is
//     decomposed, sites a step ahead, and the column tensors are formed without their 16-entry tables.
// Every sum keeps the order and the fusing of the general kernel's: the distance terms subtract an FP32 message from its
// FP64 successor, so one last bit of a message is 1e-8 of a distance near convergence.
// d = 17, 6 x 6 blocks at chi 8, 32 syndromes: 298 -> 124 ms; d = 9, 3 x 3 at chi 2, 20 syndromes: 49.4 -> 11.8 ms. (A
// pivoted Householder factorisation that reveals the rank in place of the Jacobi rounds where the bond does not bind
// took 84 ms, with distances off by up to 1e-7.)
//
// Layouts (lane ln): factor (c, q) = (ln / 4, ln % 4), rows 4 k + q of column c; reflections on the carry (kc, g) =
// (ln / 8, ln % 8), rows 4 g + r of column kc; bond matrix (l, u) = (ln / 4, ln % 4), entries 4 u + e of row l.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "geom.hpp"
#include "sweep_launch.hpp"
#include "trunc_shape.hpp"
#include "wave_mps.hpp"

namespace bbp {
namespace {

using namespace wmps;

constexpr int B = 8, KN = 7;            // largest bond; longest sweep and widest state
constexpr int SITE = B * 2 * B;         // one site [a][h][b], or one cap operator [P][v][Q]
constexpr int FACTOR = 16 * 32 + 16;    // pass-1 reflections [j][row], their coefficients
// workspace of an item, in doubles
constexpr int W_A = 0;                            // sites 0 .. kp + 1 (the caps [q][d] and [d][q])
constexpr int W_Q = W_A + (KN + 2) * SITE;        // factors of sites 0 .. kp
constexpr int W_CT = W_Q + (KN + 1) * FACTOR;     // cap operators: top t = 0 .. kt - 1, then bottom
constexpr int W_SLOT = W_CT + 2 * KN * SITE;

// LDS of the wavefront, in doubles
constexpr int L_R = 0;                  // carry R [row < 16][col < 16]
constexpr int L_C = L_R + 16 * 16;      // carry C [row < 16][col < 8]
constexpr int L_V = L_C + 16 * B;       // vectors: pass 1 the current one, twice; pass 2 a factor
constexpr int L_X = L_V + FACTOR;       // site, bottom operator; X [32][9]; Jacobi exchange [64][6], then V [16][16]
constexpr int L_END = L_X + 64 * 6;
constexpr int L_P = L_END;              // Pauli probabilities
constexpr int L_N = L_P + 4;            // bond sizes (int)
constexpr int L_TOTAL = L_N + 16;

// product of the split-off norms as mantissa and exponent
struct Scale {
  double m = 1.0;
  int e = 0;
  __device__ __forceinline__ void take(double f) {
    m *= f;
    const int x = __builtin_amdgcn_frexp_exp(m);
    m = __builtin_amdgcn_ldexp(m, -x);
    e += x;
  }
  __device__ __forceinline__ double log_value() const { return log(m) + e * 0.69314718055994530942; }
};

// Left-canonical chain of the K-leg vector in W[0 .. 2^K) (leg 0 most significant; W is overwritten; K <= 7): site
// j = A_j[a][v][q] with natural bonds. transposed: written as the cap operator CT_{K-1-j}[q][v][a] (the chain
// absorbed from its weighted end); else as site j itself, [a][v][q]. out must be zero beyond the bonds.
__device__ __forceinline__ void chain(double* W, double* Hv, double* Hb, int K, double* out, bool transposed) {
  const int ln = threadIdx.x;
  int b = 1;
  for (int j = 0; j < K - 1; ++j) {
    const int m = 2 * b, n = 1 << (K - j - 1), k = min(m, n);
    for (int c = 0; c < k; ++c) {
      const double xr = (ln < m && ln >= c) ? W[ln * n + c] : 0.0;
      const double alpha = W[c * n + c];
      const double n2 = wsum(xr * xr);
      double beta = 0.0, vj = alpha, diag = alpha;
      const double nrm = sqrt(n2);
      if (nrm > 0.0) {
        const double sg = (alpha >= 0.0) ? 1.0 : -1.0;
        vj = alpha + sg * nrm;
        beta = 1.0 / (nrm * (nrm + fabs(alpha)));
        diag = -sg * nrm;
      }
      if (ln < 16) Hv[c * 16 + ln] = (ln == c) ? vj : ((ln > c && ln < m) ? xr : 0.0);
      if (ln == 0) Hb[c] = beta;
      wave_sync();
      for (int col = c + 1 + ln; col < n; col += 64) {
        double w = 0.0;
        for (int r = c; r < m; ++r) w += Hv[c * 16 + r] * W[r * n + col];
        w *= beta;
        for (int r = c; r < m; ++r) W[r * n + col] -= w * Hv[c * 16 + r];
      }
      wave_sync();
      if (ln == 0) W[c * n + c] = diag;
      if (ln > c && ln < m) W[ln * n + c] = 0.0;
      wave_sync();
    }
    // Q (m x k): lane q forms column q by applying the reflections to the unit vector e_q
    if (ln < k) {
      double qv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) qv[r] = (r == ln) ? 1.0 : 0.0;
      for (int c = k - 1; c >= 0; --c) {
        double w = 0.0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
#pragma clang fp contract(off)
          w += Hv[c * 16 + r] * qv[r];   // (the general kernel's products are rounded here, behind its row limits)
        }
        w *= Hb[c];
#pragma unroll
        for (int r = 0; r < 16; ++r) qv[r] -= w * Hv[c * 16 + r];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (r >= m) break;
        const int a = r >> 1, v = r & 1;
        if (transposed) out[(K - 1 - j) * SITE + ln * 16 + v * 8 + a] = qv[r];
        else out[j * SITE + a * 16 + v * 8 + ln] = qv[r];
      }
    }
    wave_sync();   // W now holds R (k x n): rows 0 .. k-1, the next step's (2k) x (n/2) matrix
    b = k;
  }
  // last site: A_{K-1}[a][v][0] = rest[a][v]
  for (int e = ln; e < 2 * b; e += 64) {
    const int a = e >> 1, v = e & 1;
    if (transposed) out[v * 8 + a] = W[e];
    else out[(K - 1) * SITE + a * 16 + v * 8] = W[e];
  }
  wave_sync();
}

// QR of the site matrix held as x[k] = M[4 k + q][c] (32 x 16, the columns >= ncol and rows >= 2 nrow zero): jmax =
// min(ncol, rows) reflections, vectors broadcast through LDS. R (unit Frobenius norm) into the LDS carry, vectors and
// coefficients into the factor slot. Returns the norm.
__device__ __forceinline__ double factor(double (&x)[8], int jmax, double* lds, double* Vg) {
  const int ln = threadIdx.x, c = ln >> 2, q = ln & 3;
  double* vb = lds + L_V;
  double rd = 0.0;
  for_each(std::make_integer_sequence<int, 16>(), [&](auto J) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value, kj = j >> 2, qj = j & 3;   // pivot row j = 4 kj + qj
    if (j >= jmax) return;
    double* v = vb + (j & 1) * 32;
    if (c == j) {
#pragma unroll
      for (int k = kj; k < 8; ++k) v[4 * k + q] = x[k];
    }
    wave_sync();
    double hv[8];
#pragma unroll
    for (int k = kj; k < 8; ++k) {
      hv[k] = v[4 * k + q];
      if (k == kj) hv[k] = q < qj ? 0.0 : hv[k];   // rows above the pivot are not part of the vector
    }
    const double nrm = sqrt(sum4(squares(hv, kj)));
    const double alpha = v[j];
    const bool live = nrm > 0.0;
    const double sg = (alpha >= 0.0) ? 1.0 : -1.0;
    const double vj = live ? alpha + sg * nrm : alpha, diag = live ? -sg * nrm : alpha;
    const double rec = 1.0 / (nrm * (nrm + fabs(alpha))), beta = live ? rec : 0.0;
    hv[kj] = (q == qj) ? vj : hv[kj];   // the pivot entry of the vector is v_j, not alpha
    double pw = 0.0;
#pragma unroll
    for (int k = kj; k < 8; ++k) pw += hv[k] * x[k];
    const double w = sum4(pw) * beta;
    if (c > j) {
#pragma unroll
      for (int k = kj; k < 8; ++k) x[k] -= w * hv[k];
    } else if (c == j) {
      rd = diag;
      if (q == qj) x[kj] = vj;
      if (q == 0) Vg[512 + j] = beta;
    }
  });
  double r[4];   // R's rows: the first 16
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int row = 4 * k + q;
    r[k] = row < c ? x[k] : (row == c ? rd : 0.0);
  }
  const double fro = sqrt(wsum(squares(r)));
  const double inv = (fro > 0.0) ? 1.0 / fro : 0.0;
  wave_sync();   // every lane has read the previous carry
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int row = 4 * k + q;
    if (k < 4) lds[L_R + row * 16 + c] = r[k & 3] * inv;
    if (c < jmax) Vg[c * 32 + row] = (row >= c) ? x[k] : 0.0;
  }
  wave_sync();
  return fro;
}

// QR of the top cap's matrix, rows q' < 8, held as x[k] = M[2 k + par][hi] by lane (hi, par) = (ln / 2, ln % 2), in the
// layout and order of wmps::qr64u<16, 8>; R and the reflections (rows < 8) as factor() leaves them. Returns the norm.
__device__ __forceinline__ double factor_top(double (&x)[8], int jmax, double* lds, double* Vg) {
  const int ln = threadIdx.x, hi = ln >> 1, par = ln & 1;
  double* vb = lds + L_V;
  double rd = 0.0;
  for_each(std::make_integer_sequence<int, 8>(), [&](auto J) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value, k0 = j >> 1, jp = j & 1;
    if (j >= jmax) return;
    double* v = vb + (j & 1) * 32;
    if (hi == j) {
#pragma unroll
      for (int k = k0; k < 8; ++k) v[2 * k + par] = x[k];
    }
    wave_sync();
    double hv[8];
#pragma unroll
    for (int k = k0; k < 8; ++k) {
      hv[k] = v[2 * k + par];
      if (k == k0 && jp == 1) hv[k] = par ? hv[k] : 0.0;
    }
    const double pn = squares(hv, k0);
    const double nrm = sqrt(pn + dpp<0xB1>(pn));
    const double alpha = v[j];
    const bool live = nrm > 0.0;
    const double sg = (alpha >= 0.0) ? 1.0 : -1.0;
    const double vj = live ? alpha + sg * nrm : alpha, diag = live ? -sg * nrm : alpha;
    const double rec = 1.0 / (nrm * (nrm + fabs(alpha))), beta = live ? rec : 0.0;
    hv[k0] = (par == jp) ? vj : hv[k0];
    double pw = 0.0;
#pragma unroll
    for (int k = k0; k < 8; ++k) pw += hv[k] * x[k];
    const double w = (pw + dpp<0xB1>(pw)) * beta;
    if (hi > j) {
#pragma unroll
      for (int k = k0; k < 8; ++k) x[k] -= w * hv[k];
    } else if (hi == j) {
      rd = diag;
      if (par == jp) x[k0] = vj;
      if (par == 0) Vg[512 + j] = beta;
    }
  });
  double r[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int row = 2 * k + par;
    r[k] = row < hi ? x[k] : (row == hi ? rd : 0.0);
  }
  const double fro = sqrt(wsum(squares(r)));
  const double inv = (fro > 0.0) ? 1.0 / fro : 0.0;
  wave_sync();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int row = 2 * k + par;
    if (hi < 16) lds[L_R + row * 16 + hi] = r[k] * inv;
    if (hi < jmax) Vg[hi * 32 + row] = (row >= hi) ? x[k] : 0.0;
  }
  wave_sync();
  return fro;
}

// X = Q C: the jmax stored reflections (staged in LDS) on the carry C [row][kc] (scaled by cs), rows 4 g + r of column
// kc in X[r].
__device__ __forceinline__ void apply(double (&X)[4], int jmax, const double* lds, double cs) {
  const int ln = threadIdx.x, kc = ln >> 3, g = ln & 7;
  const double* V = lds + L_V;
#pragma unroll
  for (int r = 0; r < 4; ++r) X[r] = (g < 4) ? lds[L_C + (4 * g + r) * B + kc] * cs : 0.0;
  for (int j = jmax - 1; j >= 0; --j) {
    double v[4], p = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = V[j * 32 + 4 * g + r];
      p += v[r] * X[r];
    }
    const double w = sum8(p) * V[512 + j];
#pragma unroll
    for (int r = 0; r < 4; ++r) X[r] -= w * v[r];
  }
}

// A factor slot from the workspace into registers (as soon as its address is known) and from there into LDS.
struct Staged {
  double v[8], b;
  __device__ __forceinline__ void load(const double* Vg, int jmax) {
    const int ln = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = 2 * k < jmax ? Vg[ln + 64 * k] : 0.0;   // 64 entries are two vectors
    b = ln < 16 ? Vg[512 + ln] : 0.0;
  }
  __device__ __forceinline__ void put(double* lds) const {
    const int ln = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 8; ++k) lds[L_V + ln + 64 * k] = v[k];
    if (ln < 16) lds[L_V + 512 + ln] = b;
  }
};

// Bond of the matrix N held as y[e] = N[l][4 u + e] (left bond x (leg, right bond), rows l >= n zero): one-sided Jacobi
// on the rows as wmps::svd_step, 16 rows of four lanes each; the chi largest singular values are kept, their right
// singular vectors become the site's rows ([j][t][k] with 4 u + e = 8 t + k; the bottom cap keeps t = 0 as [j][k]) and N
// V the carry C [l][j] (not normalised). Returns the bond's size, the number of values kept; norm is |C|_F.
__device__ __forceinline__ int bond(double (&y)[4], int n, int chi, double* lds, double* site, bool bottom, double& norm) {
  constexpr int XN = 6;   // exchange row stride: 4 entries and the row norm, 16-byte aligned
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int ln = threadIdx.x, l = ln >> 2, u = ln & 3, t = u >> 1, k0 = 4 * (u & 1);
  double* Xsh = lds + L_X;
  double y0[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) y0[e] = y[e];
  const double thr2 = wsum(squares(y)) * (RANKTOL * RANKTOL);
  double* own_row = Xsh + ln * XN;
  *(d2*)own_row = d2{y[0], y[1]};
  *(d2*)(own_row + 2) = d2{y[2], y[3]};
  for (int sw = 0; sw < SWEEPS; ++sw) {
    int rotated = 0;
    double c2max = 0.0, own = sum4(squares(y));
    own_row[4] = own;
    wave_sync();
    // round rd pairs rows l and pl: 15 and rd, the others (2 rd - l) mod 15, stepped by 2 each round. With n < 16 rows,
    // rounds none of whose pairs lie within them -- their row numbers add up to 2 rd mod 15, or 15 more -- do nothing.
    int cyc = (30 - l) % 15;
    for (int rd = 0; rd < 15; ++rd, cyc = (cyc + 2 >= 15) ? cyc + 2 - 15 : cyc + 2) {
      const int sum = 2 * rd >= 15 ? 2 * rd - 15 : 2 * rd;
      if (n < 16 && !(sum >= 1 && sum <= 2 * n - 3) && sum + 15 > 2 * n - 3) continue;
      const int pl = (l == 15) ? rd : (l == rd) ? 15 : cyc;
      const double* P = Xsh + (4 * pl + u) * XN;
      const d2 z01 = *(const d2*)P, z23 = *(const d2*)(P + 2);
      const double z[4] = {z01[0], z01[1], z23[0], z23[1]};
      double gg = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) gg += y[e] * z[e];
      const double other = P[4];
      wave_sync();
      gg = sum4(gg);
      const bool lower = l < pl;
      const double al = lower ? own : other, be = lower ? other : own;
      const Rotation t(al, be, gg, thr2);
      c2max = t.c2 > c2max ? t.c2 : c2max;
      if (t.c2 > JAC * JAC) {
        const double sz = lower ? -t.sn : t.sn;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = fma(sz, z[e], t.cs * y[e]);
        own = t.norm2(lower, al, be, gg);
        *(d2*)own_row = d2{y[0], y[1]};
        *(d2*)(own_row + 2) = d2{y[2], y[3]};
        own_row[4] = own;
        rotated = 1;
      }
      wave_sync();
    }
    if (!__any(rotated) || !__any(c2max >= 1e-12)) break;
  }
  const double s2r = sum4(squares(y));
  const double sv = (s2r > thr2) ? sqrt(s2r) : 0.0;
  const double key = (sv == sv) ? sv : -1.0;
  double* sig = lds + L_R;   // the carry R is not needed in pass 2
  if (u == 0) sig[l] = key;
  wave_sync();
  int rank = 0;
  for (int i = 0; i < 16; ++i) {
    const double o = sig[i];
    rank += (o > key || (o == key && i < l)) ? 1 : 0;
  }
  const bool kept = rank < chi && sv > 0.0;
  const double inv = kept ? 1.0 / sv : 0.0;
  double* Vsh = Xsh;   // [j][16]: the exchange buffer is free now
  if (rank < B) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      Vsh[rank * 16 + 4 * u + e] = y[e] * inv;
      if (!bottom) site[(rank * 2 + t) * B + k0 + e] = y[e] * inv;
      else if (t == 0) site[rank * B + k0 + e] = y[e] * inv;
    }
  }
  norm = sqrt(wsum((u == 0 && kept) ? sv * sv : 0.0));
  const int size = __builtin_popcountll(__ballot(u == 0 && kept));
  wave_sync();
#pragma unroll
  for (int j = 0; j < B; ++j) {
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc += y0[e] * Vsh[j * 16 + 4 * u + e];
    acc = sum4(acc);
    if ((j & 3) == u) lds[L_C + l * B + j] = acc;
  }
  wave_sync();
  return size;
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void trunc_narrow_kernel(SweepArgs a) {
  const int ln = threadIdx.x;
  const int64_t item = a.item_base + (int64_t)blockIdx.x;
  if (item >= a.items) return;
  int gi = 0;
  for (int k = 1; k < a.ngroups; ++k)
    if (item >= a.g[k].item0) gi = k;
  const SweepGroup& G = a.g[gi];
  const int64_t local = item - G.item0;
  int64_t job, sw;
  if (a.order == 0) {
    sw = local / G.jobs;
    job = local - sw * G.jobs;
  } else {
    job = local / G.count;
    sw = local - job * G.count;
  }
  if (a.mode == 0 && G.conv[job]) return;
  const SweepDesc s = G.sweeps[sw];
  if (a.mode == 0 && a.gate > 0.0) {
    const double* tj = G.terms + job * G.M;
    const double ti = s.msg_init >= 0 ? tj[s.msg_init] : 0.0, tt = s.msg_top >= 0 ? tj[s.msg_top] : 0.0,
                 tb = s.msg_bot >= 0 ? tj[s.msg_bot] : 0.0;
    if (tj[s.msg_out] < a.gate && ti < a.gate && tt < a.gate && tb < a.gate) {
      if (ln == 0) G.terms[job * G.M + s.msg_out] = 0.0;
      return;
    }
  }
  const int L = 2 * G.d - 1, kt = s.kt, kp = s.kp, chi = G.chi, ms = G.mstride;
  const uint8_t* lab = G.labels + job * (int64_t)L * L;
  const float* mbase = G.msgs + job * G.M * (int64_t)ms;
  double* ws = a.tws + (int64_t)blockIdx.x * W_SLOT;
  double* A = ws + W_A;
  double* Q = ws + W_Q;
  double* CT = ws + W_CT;

  __shared__ __align__(16) double lds[L_TOTAL];
  // bond sizes: the left bond of site i (1 .. kp + 1), and the reflections of site i's factor (0 .. kp)
  int* left = (int*)(lds + L_N);
  int* refl = left + 16;
  const bool top = s.msg_top >= 0, bot = s.msg_bot >= 0, fwd = (s.frame == FRAME_E || s.frame == FRAME_S);
  if (ln < 4) {
    double v = G.pq[ln];
    if (G.pdev) {
      const double pj = G.pdev[job >> 2];
      v = ln == 0 ? 1.0 - pj : pj / 3.0;
    }
    lds[L_P + ln] = v;
  }

  // ---- caps and the initial state (the chains fill the natural bonds only: clear what is read around them)
  if (top)
    for (int e = ln; e < kt * SITE; e += 64) CT[e] = 0.0;
  if (bot)
    for (int e = ln; e < kt * SITE; e += 64) CT[KN * SITE + e] = 0.0;
  for (int e = ln; e < (kp + 2) * SITE; e += 64) A[e] = 0.0;
  wave_sync();
  {
    double* W = lds;                 // 128
    double* Hv = lds + 128;          // 8 x 16
    double* Hb = Hv + 128;
    for (int side = 0; side < 2; ++side) {
      const int id = side == 0 ? s.msg_top : s.msg_bot;
      if (id < 0) continue;
      for (int w = ln; w < (1 << kt); w += 64)
        W[w] = (double)mbase[id * (int64_t)ms + (fwd ? (int)(__brev((unsigned)w) >> (32 - kt)) : w)];
      wave_sync();
      chain(W, Hv, Hb, kt, CT + side * KN * SITE, true);
    }
    if (s.msg_init >= 0) {
      for (int w = ln; w < (1 << kp); w += 64) W[w] = (double)mbase[s.msg_init * (int64_t)ms + w];
      wave_sync();
      chain(W, Hv, Hb, kp, A + SITE, false);
      if (ln >= 1 && ln <= kp + 1) left[ln] = 1 << min(ln - 1, kp + 1 - ln);
    } else {
      if (ln >= 1 && ln <= kp) A[ln * SITE] = 1.0;   // every in-leg at its only value 0
      if (ln >= 1 && ln <= kp + 1) left[ln] = 1;
    }
    if (ln == 0) {
      A[0] = 1.0;                    // top cap [q = 0][d = 0]
      A[(kp + 1) * SITE] = 1.0;      // bottom cap [d = 0][q = 0]
    }
  }
  wave_sync();

  Scale scale;
  const int c = ln >> 2, q = ln & 3;
  for (int t = 0; t < kt; ++t) {
    // cap bonds before and after this column (1 without a side message)
    const int pq0 = 1 << min(t, kt - t), pq1 = 1 << min(t + 1, kt - t - 1);
    // ---------------- pass 1: absorb and factor, top to bottom ----------------
    double x[8];
    int nrow;   // rows of R that can be nonzero
    {
      // top cap: M_0[q'][(d, v)] = sum_P S_0[P][d] CT[P][v][q'], rows q' = 2 k + par < 8 of column (d, v) = ln / 2
      const int d = ln >> 2, v = (ln >> 1) & 1, par = ln & 1;
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = 0.0;
      if (top) {
        if (d < B)
          for (int P = 0; P < pq0; ++P) {
            const double sp = A[P * B + d];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] += sp * CT[t * SITE + P * 16 + v * 8 + 2 * k + par];
          }
      } else if (v == 0 && par == 0 && d < B) {
        x[0] = A[d];
      }
      nrow = __builtin_amdgcn_readfirstlane(min(top ? pq1 : 1, 2 * left[1]));
      scale.take(factor_top(x, nrow, lds, Q));
      if (ln == 0) refl[0] = nrow;
    }
    double a0 = A[SITE + ln], a1 = A[SITE + 64 + ln];   // site i's 128 entries, a column ahead of their use
    for (int i = 1; i <= kp; ++i) {
      lds[L_X + ln] = a0;
      lds[L_X + 64 + ln] = a1;
      const int na = __builtin_amdgcn_readfirstlane(left[i]), nb = __builtin_amdgcn_readfirstlane(left[i + 1]);
      a0 = A[(i + 1) * SITE + ln];
      a1 = A[(i + 1) * SITE + 64 + ln];
      // lane (c, q): column c = (b, dn), rows 4 k + q = (R row 2 k + q / 2, leg q % 2)
      const int b = c >> 1, dn = c & 1, h = q & 1, m0 = q >> 1;
      int sr, sc;
      frame_site(s.frame, s.r0, s.c0, s.kr, s.kc, t, i - 1, sr, sc);
      const bool au = sr == 0, al = sc == 0, ad = sr == L - 1, ar = sc == L - 1;
      // absent legs in the frame: up, in, down, out
      const bool ew = s.frame <= FRAME_W;
      const bool n_up = ew ? au : al, n_dn = ew ? ad : ar;
      const bool n_in = s.frame == FRAME_E ? al : s.frame == FRAME_W ? ar : s.frame == FRAME_S ? au : ad;
      const bool n_out = s.frame == FRAME_E ? ar : s.frame == FRAME_W ? al : s.frame == FRAME_S ? ad : au;
      const bool dead = (n_dn && dn) || (n_out && h);
      double tt[2][2];   // [up][in]
      if (((sr + sc) & 1) == 0) {
        const int lb = lab[sr * L + sc] & 3;
        const bool swap = ((sr & 1) != 0) != (s.frame >= FRAME_S);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int in = 0; in < 2; ++in) {
            const int pv = u ^ dn, ph = in ^ h;
            const int code = lb ^ (swap ? (ph | (pv << 1)) : (pv | (ph << 1)));
            const double p = lds[L_P + code];
            tt[u][in] = (dead || (n_up && u) || (n_in && in)) ? 0.0 : p;
          }
      } else {
        // COPY: the present legs agree, the absent ones are 0
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int in = 0; in < 2; ++in) {
            const bool one = (n_up || u) && (n_in || in) && (n_dn || dn) && (n_out || h);
            const bool zero = !u && !in && !dn && !h;
            const bool some = !(n_up && n_in && n_dn && n_out);
            tt[u][in] = (dead || (n_up && u) || (n_in && in)) ? 0.0 : ((one && some) || zero) ? 1.0 : 0.0;
          }
      }
      wave_sync();
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = 0.0;
      for (int aa = 0; aa < na; ++aa) {
        const double s0 = lds[L_X + aa * 16 + b], s1 = lds[L_X + aa * 16 + 8 + b];
        const double b0 = s0 * tt[0][0] + s1 * tt[0][1], b1 = s0 * tt[1][0] + s1 * tt[1][1];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (2 * k >= nrow) break;
          const double* R = lds + L_R + (2 * k + m0) * 16 + 2 * aa;
          x[k] += R[0] * b0 + R[1] * b1;
        }
      }
      const int rows = 2 * nrow;
      nrow = min(rows, 2 * nb);
      scale.take(factor(x, nrow, lds, Q + i * FACTOR));
      if (ln == 0) refl[i] = nrow;
    }
    // bottom cap: Bb[(d, v)][q'] = sum_P S[d][P] CT[P][v][q'] (16 x 8), then y = R Bb as the bond matrix
    double y[4];
    {
      const int nd = __builtin_amdgcn_readfirstlane(left[kp + 1]);
      // (a0, a1 hold the cap site: entry d 8 + P in lane d 8 + P of a0)
      lds[L_X + ln] = a0;
      wave_sync();
      double bv[2];
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int e = ln + 64 * w, dv = e >> 3, qq = e & 7, d = dv >> 1, v = dv & 1;
        double acc = 0.0;
        if (bot) {
          for (int P = 0; P < pq0; ++P) acc += lds[L_X + d * B + P] * CT[(KN + t) * SITE + P * 16 + v * 8 + qq];
        } else if (v == 0 && qq == 0) {
          acc = lds[L_X + d * B];
        }
        bv[w] = acc;
      }
#pragma unroll
      for (int w = 0; w < 2; ++w) lds[L_X + 64 + ln + 64 * w] = bv[w];
      wave_sync();
      const int l = ln >> 2, u = ln & 3;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = 0.0;
      if (u < 2)
        for (int dv = 0; dv < 2 * nd; ++dv) {
          const double r = lds[L_R + l * 16 + dv];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] += r * lds[L_X + 64 + dv * B + 4 * u + e];
        }
      wave_sync();
    }

    // ---------------- pass 2: bottom to top ----------------
    double cs = 1.0;
    Staged st;
    for (int i = kp + 1; i >= 1; --i) {
      if (i <= kp) {
        // N = Q_i C, then from columns to rows: lane (l, u) takes y[e] = X[2 l + u / 2][4 (u % 2) + e]
        const int n = __builtin_amdgcn_readfirstlane(refl[i]);
        st.put(lds);
        wave_sync();
        double X[4];
        apply(X, n, lds, cs);
        const int kc = ln >> 3, g = ln & 7;
#pragma unroll
        for (int r = 0; r < 4; ++r) lds[L_X + (4 * g + r) * 9 + kc] = X[r];
        wave_sync();
        const int l = ln >> 2, u = ln & 3;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = lds[L_X + (2 * l + (u >> 1)) * 9 + 4 * (u & 1) + e];
        wave_sync();
      }
      st.load(Q + (i - 1) * FACTOR, __builtin_amdgcn_readfirstlane(refl[i - 1]));   // for the next step
      double nrm;
      // (N has the rows of site i - 1's R)
      const int r = bond(y, __builtin_amdgcn_readfirstlane(refl[i - 1]), chi, lds, A + i * SITE, i == kp + 1, nrm);
      cs = (nrm > 0.0) ? 1.0 / nrm : 0.0;
      scale.take(nrm);
      if (ln == 0) left[i] = r;
    }
    // top cap: S_0[q'][j] = sum_m Q_0[q'][m] C[m][j], unit Frobenius norm; lane j < 8 holds the column's 8 rows
    {
      const int n = __builtin_amdgcn_readfirstlane(refl[0]);
      st.put(lds);
      wave_sync();
      double X[B], f = 0.0;
      const int kc = ln & 7;
#pragma unroll
      for (int r = 0; r < B; ++r) X[r] = lds[L_C + r * B + kc] * cs;
      for (int j = n - 1; j >= 0; --j) {
        double v[B], p = 0.0;
#pragma unroll
        for (int r = 0; r < B; ++r) v[r] = lds[L_V + j * 32 + r];
#pragma unroll
        for (int r = 0; r < B; ++r) p += v[r] * X[r];
        const double w = p * lds[L_V + 512 + j];
#pragma unroll
        for (int r = 0; r < B; ++r) X[r] -= w * v[r];
      }
#pragma unroll
      for (int r = 0; r < B; ++r) f += (ln < B) ? X[r] * X[r] : 0.0;
      const double fro = sqrt(wsum(f));
      const double inv = (fro > 0.0) ? 1.0 / fro : 0.0;
      if (ln < B) {
#pragma unroll
        for (int r = 0; r < B; ++r) A[r * B + ln] = X[r] * inv;
      }
      scale.take(fro);
    }
    wave_sync();
  }

  // ---------------- the dense message: left chain x right chain ----------------
  const int hl = kp / 2, hr = kp - hl;
  double* lch = lds;          // [2][8 * 8], ping-pong
  double* rch = lds + 128;    // [2][16 * 8]
  if (ln < 8) {
    lch[ln] = A[ln];                        // top cap row q' = 0
    rch[ln] = A[(kp + 1) * SITE + ln * B];  // bottom cap column q' = 0
  }
  wave_sync();
  int lc = 0, rc = 0;
  for (int i = 1; i <= hl; ++i) {   // L_i[(pre, h)][b] = sum_a L_{i-1}[pre][a] S_i[a][h][b]
    const int na = __builtin_amdgcn_readfirstlane(left[i]), nb = __builtin_amdgcn_readfirstlane(left[i + 1]);
    const int b = ln & 7, ph = ln >> 3, pre = ph >> 1, h = ph & 1;
    if (ph < (1 << i)) {
      double acc = 0.0;
      for (int aa = 0; aa < na; ++aa) acc += lch[lc * 64 + pre * B + aa] * (b < nb ? A[i * SITE + aa * 16 + h * 8 + b] : 0.0);
      lch[(lc ^ 1) * 64 + ln] = acc;
    }
    wave_sync();
    lc ^= 1;
  }
  for (int i = kp; i > hl; --i) {   // R_i[(h, suf)][a] = sum_b S_i[a][h][b] R_{i+1}[suf][b]
    const int na = __builtin_amdgcn_readfirstlane(left[i]), nb = __builtin_amdgcn_readfirstlane(left[i + 1]);
    const int nsuf = 1 << (kp - i), n = 2 * nsuf * B;
    for (int e = ln; e < n; e += 64) {
      const int aa = e & 7, hs = e >> 3, h = hs / nsuf, suf = hs - h * nsuf;
      double acc = 0.0;
      if (aa < na)
        for (int b = 0; b < nb; ++b) acc += A[i * SITE + aa * 16 + h * 8 + b] * rch[rc * 128 + suf * B + b];
      rch[(rc ^ 1) * 128 + e] = acc;
    }
    wave_sync();
    rc ^= 1;
  }
  double out[2];
  const int H = 1 << kp, nm = __builtin_amdgcn_readfirstlane(left[hl + 1]);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int e = ln + 64 * r;
    double acc = 0.0;
    if (e < H) {
      const int hL = e >> hr, hR = e & ((1 << hr) - 1);
      for (int b = 0; b < nm; ++b) acc += lch[lc * 64 + hL * B + b] * rch[rc * 128 + hR * B + b];
    }
    out[r] = acc;
  }

  if (a.mode == 1) {
    double w = 0.0;
    if (s.msg_close >= 0) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int e = ln + 64 * r;
        if (e < H) w += out[r] * (double)mbase[s.msg_close * (int64_t)ms + e];
      }
    } else if (ln == 0) {
      w = out[0];
    }
    w = wsum(w);
    if (ln == 0) G.lnW[job * G.nblocks + s.block] = (w > 0.0) ? scale.log_value() + log(w) : NAN;
    return;
  }
  // normalised new message, damping against the old one (unit norm), distance term
  float* mo = G.msgs + (job * G.M + s.msg_out) * (int64_t)ms;
  const double inv = 1.0 / sqrt(wsum(squares(out)));
  double old[2], dm[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int e = ln + 64 * r;
    old[r] = (e < H) ? (double)mo[e] : 0.0;
    dm[r] = fma((double)a.eta, old[r], (1.0 - (double)a.eta) * out[r] * inv);
  }
  const double ginv = 1.0 / sqrt(wsum(squares(dm)));
  double df[2], sf[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    df[r] = fma(dm[r], ginv, -old[r]);
    sf[r] = fma(dm[r], ginv, old[r]);
    dm[r] = dm[r] * ginv;
  }
  const double dd = wsum(squares(df)), ss = wsum(squares(sf));
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int e = ln + 64 * r;
    if (e < H) mo[e] = (float)dm[r];
  }
  if (ln == 0) G.terms[job * G.M + s.msg_out] = 0.5 * dd * ss;
}

}  // namespace

size_t trunc_narrow_slot_bytes() { return (size_t)W_SLOT * sizeof(double); }

void launch_trunc_narrow(unsigned items, hipStream_t st, const SweepArgs& a) {
  trunc_narrow_kernel<<<dim3(items), dim3(64), 0, st>>>(a);
}

}  // namespace bbp
