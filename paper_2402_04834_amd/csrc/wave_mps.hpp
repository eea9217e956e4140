// wave_mps.hpp -- one-wavefront FP64 building blocks of the boundary-MPS compression (Sec. III.A, III.D): the
// QR sweep's Householder factorisation of a site and the truncating sweep's SVD of a bond, shared by the
// truncating block sweeps (trunc_sweep.hip) and the single-block boundary-MPS decoder (bmps.hip).
//
// Shapes (bond dimensions padded to 2 chi_max = 32, chi <= 16):
//   factor   the 64 x 32 matrix M of a site after absorbing a column, rows 2l + h (left bond l, leg h), held
//            as x[k] = M[2k + par][hi] by lane (hi, par); M = Q R by Householder reflections j < jmax whose
//            vectors are broadcast through LDS from the lanes that own them (no memory round trip while
//            factoring) and then stored once in compact form with their coefficients (a factor slot);
//   carry    R (32 x 32, unit Frobenius norm) down the QR sweep, C (32 x 16, unit norm) up the SVD sweep;
//   bond     N = Q C as a 32 x 32 (left bond) x (leg, right bond) matrix, formed by applying the stored
//            reflections to [C; 0] (Q itself is never formed), then one-sided Jacobi on its rows: the chi
//            largest singular values are kept, their right singular vectors become the site and N V (unit
//            norm) the carry to the site above.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>
#include <utility>

namespace bbp {
namespace wmps {

constexpr int XS = 17;                                        // Jacobi exchange row stride (LDS banks)
constexpr int TQ = 32 * 64 + 32;  // one factor slot: reflection vectors [j][row] (rows 2l + h, l < 32), betas

// Jacobi: rotate while |<c_p, c_q>| > JAC |c_p| |c_q|; a row of norm at most RANKTOL |N|_F is rounding noise
constexpr double JAC = 1e-13, RANKTOL = 1e-13;
constexpr int SWEEPS = 16;

// Orders the memory accesses of the lanes of a one-wavefront workgroup: they complete in issue order, so only the
// compiler has to keep them (__syncthreads also waits for every outstanding LDS access).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lane exchanges by DPP and lane swaps: no LDS round trip as a shuffle takes.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t x = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)x, CTRL, 0xF, 0xF, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(x >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// the two halves of an exchange of 16-lane (W = 16) or 32-lane groups: {own group's, other group's} values
template <int W>
__device__ __forceinline__ void halves(double v, double& a, double& b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
  unsigned l0, l1, h0, h1;
  if constexpr (W == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
  }
  a = __builtin_bit_cast(double, (uint64_t)l0 | ((uint64_t)h0 << 32));
  b = __builtin_bit_cast(double, (uint64_t)l1 | ((uint64_t)h1 << 32));
}
__device__ __forceinline__ double sum4(double v) {   // over a quad: lane ^ 1, then ^ 2
  v += dpp<0xB1>(v);
  return v + dpp<0x4E>(v);
}
__device__ __forceinline__ double sum8(double v) {   // over 8 lanes: ^ 1, ^ 2, then the other quad
  v = sum4(v);
  return v + dpp<0x141>(v);
}
// over the wavefront: lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1 (a rotation by 4 of 16 lanes brings the value of lane ^ 4 once
// lanes 8 apart agree)
__device__ __forceinline__ double wsum(double v) {
  double a, b;
  halves<32>(v, a, b);
  v = a + b;
  halves<16>(v, a, b);
  v = a + b;
  v += dpp<0x128>(v);
  v += dpp<0x124>(v);
  v += dpp<0x4E>(v);
  return v + dpp<0xB1>(v);
}

// Sum of x[k0 .. N)^2: the first square is added unrounded to the second, rounded one, the others unrounded in turn.
template <int N>
__device__ __forceinline__ double squares(const double (&x)[N], int k0 = 0) {
#pragma clang fp contract(off)
  const double second = k0 + 1 < N ? x[k0 + 1 < N ? k0 + 1 : k0] * x[k0 + 1 < N ? k0 + 1 : k0] : 0.0;
  double s = fma(x[k0], x[k0], second);
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (k >= k0 + 2) s = fma(x[k], x[k], s);
  return s;
}

__device__ __forceinline__ double wmax(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  return v;
}

// f(0), f(1), ... with compile-time arguments (a loop that may end early is not unrolled fully by the compiler, and its
// registers would be indexed in scratch memory)
template <class F, int... J>
__device__ __forceinline__ void for_each(std::integer_sequence<int, J...>, F&& f) {
  (f(std::integral_constant<int, J>()), ...);
}

// Householder QR of the 64 x 32 matrix held as x[k] = M[2k + par][hi] by lane (hi, par), reflections j < jmax <= JMAX
// (uniform; those beyond the matrix's nonzero rows or columns would do nothing). On return x holds R above the diagonal
// and reflection vector j (pivot entry v_j) from the diagonal down in lanes hi = j, rd the diagonal entry of R of the
// lane's column, Hb[j] the coefficients. The reflections are unrolled: reflection j touches registers k >= j / 2 only,
// and its pivot is a compile-time register. KR: only rows below 2 KR can be nonzero (x[k] = 0 for k >= KR, untouched), as
// in a cap's 16-row matrix, or a site's when the carry has at most 16 rows.
template <int JMAX, int KR = 32>
__device__ __forceinline__ void qr64u(double (&x)[32], double& rd, int jmax, double* vb, double* Hb) {
  static_assert(KR <= 32 && JMAX <= 2 * KR, "reflections within the nonzero rows");
  const int ln = threadIdx.x, hi = ln >> 1, par = ln & 1;
  rd = 0.0;
  for_each(std::make_integer_sequence<int, JMAX>(), [&](auto J) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value, k0 = j >> 1, jp = j & 1;   // pivot row j = 2 k0 + jp
    if (j >= jmax) return;
    double* v = vb + (j & 1) * 64;
    if (hi == j) {
#pragma unroll
      for (int k = k0; k < KR; ++k) v[2 * k + par] = x[k];
    }
    wave_sync();
    double hv[KR];
#pragma unroll
    for (int k = k0; k < KR; ++k) {
      hv[k] = v[2 * k + par];
      if (k == k0 && jp == 1) hv[k] = par ? hv[k] : 0.0;   // row 2 k0 < j is not part of the vector
    }
    const double pn = squares<KR>(hv, k0);
    // (a cap's last row: its own square is added unrounded)
    const double n2 = (KR == 8 && k0 == KR - 1) ? fma(hv[k0], hv[k0], dpp<0xB1>(pn)) : pn + dpp<0xB1>(pn);
    const double nrm = sqrt(n2), alpha = v[j];
    const bool live = nrm > 0.0;
    const double sg = (alpha >= 0.0) ? 1.0 : -1.0;
    const double vj = live ? alpha + sg * nrm : alpha, diag = live ? -sg * nrm : alpha;
    const double rec = 1.0 / (nrm * (nrm + fabs(alpha))), beta = live ? rec : 0.0;
    // the pivot entry of the vector is v_j, not alpha
    hv[k0] = (par == jp) ? vj : hv[k0];
    double pw = 0.0;
#pragma unroll
    for (int k = k0; k < KR; ++k) pw += hv[k] * x[k];
    const double w = (pw + dpp<0xB1>(pw)) * beta;
    if (hi > j) {
#pragma unroll
      for (int k = k0; k < KR; ++k) x[k] -= w * hv[k];
    } else if (hi == j) {
      rd = diag;
      if (par == jp) x[k0] = vj;
    }
    if (ln == 0) Hb[j] = beta;
  });
  wave_sync();
}

// The reflection vectors left in x by qr64u (rows >= j of column j, zero above) and their coefficients into a
// pass-1 factor slot: Vg[j * 64 + row], Vg[2048 + j].
__device__ __forceinline__ void store_v(const double (&x)[32], int jmax, const double* Hb, double* Vg) {
  const int ln = threadIdx.x, hi = ln >> 1, par = ln & 1;
  if (hi < jmax) {
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int row = 2 * k + par;
      Vg[hi * 64 + row] = (row >= hi) ? x[k] : 0.0;
    }
  }
  if (ln < jmax) Vg[2048 + ln] = Hb[ln];
}

// X = Q C for the carry C (Csh [m][k], m < 32, k < 16) and the factor stored by store_v, Q = H_0 ... H_{jmax-1}
// on the first 32 unit columns: X = H_0 (H_1 (... [C; 0])). Lane (kc, qt) = (ln & 15, ln >> 4) holds rows
// 16 qt + r of column kc in X[r]; a reflection is a 16-term partial product, two cross-quarter additions and
// a 16-term update. The vectors are read once, from the slot pass 1 wrote.
__device__ __forceinline__ void apply_q(double (&X)[16], int jmax, const double* Vg, const double* Csh) {
  const int ln = threadIdx.x, kc = ln & 15, qt = ln >> 4;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = qt * 16 + r;
    X[r] = (row < 32) ? Csh[row * 16 + kc] : 0.0;
  }
  // the vector quarters and coefficients of the next two reflections are loaded while one is applied (the loads come
  // from the workspace, through L2: one reflection's latency each, otherwise)
  double vn[3][16], bn[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int j = jmax - 1 - u > 0 ? jmax - 1 - u : 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) vn[u][r] = Vg[j * 64 + qt * 16 + r];
    bn[u] = Vg[2048 + j];
  }
  for (int j0 = jmax - 1; j0 >= 0; j0 -= 3) {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int j = j0 - u;
      if (j < 0) break;
      double p = 0.0, a, b;
#pragma unroll
      for (int r = 0; r < 16; ++r) p += vn[u][r] * X[r];
      halves<16>(p, a, b);
      p = a + b;
      halves<32>(p, a, b);
      p = a + b;
      const double w = p * bn[u];
#pragma unroll
      for (int r = 0; r < 16; ++r) X[r] -= w * vn[u][r];
      if (j >= 3) {
#pragma unroll
        for (int r = 0; r < 16; ++r) vn[u][r] = Vg[(j - 3) * 64 + qt * 16 + r];
        bn[u] = Vg[2048 + j - 3];
      }
    }
  }
}

// From apply_q's column layout to the row layout of svd_step: y[k] = X[ln][k] (N[l][(t, k)] for ln = 2l + t).
__device__ __forceinline__ void cols_to_rows(const double (&X)[16], double* Xsh, double (&y)[16]) {
  const int ln = threadIdx.x;
#pragma unroll
  for (int r = 0; r < 16; ++r) Xsh[((ln >> 4) * 16 + r) * XS + (ln & 15)] = X[r];
  wave_sync();
#pragma unroll
  for (int k = 0; k < 16; ++k) y[k] = Xsh[ln * XS + k];
  wave_sync();
}

// The carry R (rows 0..31 of the factored matrix) into Rsh [row][col], unit Frobenius norm; returns ln |R|_F.
__device__ __forceinline__ double store_r(const double (&x)[32], double rd, double* Rsh) {
  const int ln = threadIdx.x, hi = ln >> 1, par = ln & 1;
  double r[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int row = 2 * k + par;
    r[k] = row < hi ? x[k] : (row == hi ? rd : 0.0);
  }
  const double fro = sqrt(wsum(squares(r)));
  const double inv = (fro > 0.0) ? 1.0 / fro : 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int row = 2 * k + par;
    Rsh[row * 32 + hi] = r[k] * inv;
  }
  wave_sync();
  return log(fro);
}

// Rotation of two rows with squared norms al, be and product gg.
struct Rotation {
  double c2, cs, sn, tt;
  __device__ __forceinline__ Rotation(double al, double be, double gg, double thr2) {
    // squared cosine of the pair (approximate reciprocal: it only decides whether to rotate)
    c2 = (al > thr2 && be > thr2) ? gg * gg * __builtin_amdgcn_rcp(al * be) : 0.0;
    // The angle only has to bring the pair closer to orthogonal, so t = tan(theta) (the smaller root) is formed in FP32
    // (the hardware's approximate reciprocal and square root, one instruction each; above the noise threshold zeta stays
    // within 1e30); cos and sin are then formed in FP64 from that t, so that the rotation is orthogonal to FP64
    // rounding. (Formed for every pair, used or not: the chain runs beside that of c2.)
    const float zf = (float)(be - al) * __builtin_amdgcn_rcpf(2.0f * (float)gg), azf = fabsf(zf);
    const float denf = azf + (azf < 1e18f ? __builtin_amdgcn_sqrtf(fmaf(zf, zf, 1.0f)) : azf);
    tt = (double)copysignf(__builtin_amdgcn_rcpf(denf), zf);
    const double xx = fma(tt, tt, 1.0);
    cs = __builtin_amdgcn_rsq(xx);
    cs = cs * (1.5 - 0.5 * xx * cs * cs);
    cs = cs * (1.5 - 0.5 * xx * cs * cs);
    sn = cs * tt;
  }
  // squared norm of the lower or the higher row afterwards
  __device__ __forceinline__ double norm2(bool lower, double al, double be, double gg) const {
    const double cc = cs * cs;
    return lower ? cc * (al - 2.0 * tt * gg + tt * tt * be) : cc * (be + 2.0 * tt * gg + tt * tt * al);
  }
};

// One-sided Jacobi SVD of the 32 x 32 matrix N held as y[k] = N[l][(par, k)] by lane (l = hi, par), its entries
// k >= KE and rows l >= n zero, the chi largest singular values kept. Writes the kept right singular vectors (rows j < 16 of V, zero
// beyond chi) as site [j][par][k] (or, bottom cap, [j][k] from the par = 0 half) and the carry C = N V / |.|_F into Csh
// [l][j]; returns the log of that norm, and in size the number of values kept.
template <int KE>
__device__ __forceinline__ double svd_rows(const double (&yin)[16], int chi, double* Xsh, double* Csh, double* sig,
                                           double* site, bool bottom, int n, int& size) {
  const int ln = threadIdx.x, hi = ln >> 1, par = ln & 1;
  double y[KE], y0[KE];
#pragma unroll
  for (int k = 0; k < KE; ++k) y[k] = y0[k] = yin[k];
  const double thr2 = wsum(squares(y)) * (RANKTOL * RANKTOL);
  double* own_row = Xsh + ln * XS;
#pragma unroll
  for (int k = 0; k < KE; ++k) own_row[k] = y[k];
  for (int sw = 0; sw < SWEEPS; ++sw) {
    int rotated = 0;
    double c2max = 0.0;
    double own = squares(y);
    own += dpp<0xB1>(own);
    own_row[16] = own;
    wave_sync();
    // round rd pairs rows hi and pl: 31 and rd, the others (2 rd - hi) mod 31, stepped by 2 each round. With n <= 16
    // rows only sums 1 .. 2 n - 3 of two row numbers occur: the other rounds would do nothing.
    int cyc = (62 - hi) % 31;
    for (int rd = 0; rd < 31; ++rd, cyc = (cyc + 2 >= 31) ? cyc + 2 - 31 : cyc + 2) {
      const int sum = 2 * rd >= 31 ? 2 * rd - 31 : 2 * rd;
      if (n <= 16 && (sum < 1 || sum > 2 * n - 3)) continue;
      const int pl = (hi == 31) ? rd : (hi == rd) ? 31 : cyc;
      double z[KE], gg = 0.0;
#pragma unroll
      for (int k = 0; k < KE; ++k) {
        z[k] = Xsh[(2 * pl + par) * XS + k];
        gg += y[k] * z[k];
      }
      const double other = Xsh[(2 * pl + par) * XS + 16];
      wave_sync();
      gg += dpp<0xB1>(gg);
      const bool lower = hi < pl;
      const double al = lower ? own : other, be = lower ? other : own;
      const Rotation t(al, be, gg, thr2);
      c2max = t.c2 > c2max ? t.c2 : c2max;
      if (t.c2 > JAC * JAC) {
        // lower row p: c p - s q; higher row q: c q + s p -- one multiply and one fused multiply-add each. Only rows
        // that turn are written again.
        const double sz = lower ? -t.sn : t.sn;
#pragma unroll
        for (int k = 0; k < KE; ++k) y[k] = fma(sz, z[k], t.cs * y[k]);
        own = t.norm2(lower, al, be, gg);
#pragma unroll
        for (int k = 0; k < KE; ++k) own_row[k] = y[k];
        own_row[16] = own;
        rotated = 1;
      }
      wave_sync();
    }
    // a sweep whose pairs all started within cos 1e-6 of orthogonal leaves them within about 1e-12
    // (quadratic convergence): far below the FP32 messages the singular vectors end up in
    if (!__any(rotated) || !__any(c2max >= 1e-12)) break;
  }
  const double s2 = squares(y), s2r = s2 + dpp<0xB1>(s2);
  const double sv = (s2r > thr2) ? sqrt(s2r) : 0.0;
  const double key = (sv == sv) ? sv : -1.0;
  if (par == 0) sig[hi] = key;
  wave_sync();
  int rank = 0;
  for (int i = 0; i < 32; ++i) {
    const double o = sig[i];
    rank += (o > key || (o == key && i < hi)) ? 1 : 0;
  }
  const bool kept = rank < chi && sv > 0.0;
  const double inv = kept ? 1.0 / sv : 0.0;
  double* Vsh = Xsh;   // the exchange buffer is free now
  if (rank < 16) {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const double v = k < KE ? y[k < KE ? k : 0] * inv : 0.0;
      if (bottom) {
        if (par == 0) site[rank * 16 + k] = v;
      } else {
        site[(rank * 2 + par) * 16 + k] = v;
      }
      if (k < KE) Vsh[rank * 32 + par * 16 + k] = v;
    }
  }
  size = __builtin_popcountll(__ballot(par == 0 && kept));
  const double fro = sqrt(wsum((par == 0 && kept) ? sv * sv : 0.0));
  wave_sync();
  const double finv = (fro > 0.0) ? 1.0 / fro : 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    double acc = 0.0;
    if (j < size) {
#pragma unroll
      for (int k = 0; k < KE; ++k) acc += y0[k] * Vsh[j * 32 + par * 16 + k];
      acc += dpp<0xB1>(acc);
    }
    if ((j >> 3) == par) Csh[hi * 16 + j] = acc * finv;
  }
  wave_sync();
  return log(fro);
}

// (nk: the size of the right bond)
__device__ __forceinline__ double svd_step(const double (&y)[16], int n, int nk, int chi, double* Xsh, double* Csh,
                                           double* sig, double* site, bool bottom, int& size) {
  if (nk <= 8) return svd_rows<8>(y, chi, Xsh, Csh, sig, site, bottom, n, size);
  return svd_rows<16>(y, chi, Xsh, Csh, sig, site, bottom, n, size);
}

}  // namespace wmps
}  // namespace bbp
