// trunc_sweep.hip -- block sweeps with a binding chi (Sec. III.D, Fig. 3): the boundary MPS of the in-block
// sweep compressed back to chi after every column by a Householder QR sweep and a truncated one-sided Jacobi
// SVD sweep, in FP64. The dense kernels (sweep_kernel.hip) serve every sweep whose boundary state provably
// stays within chi (the plan's rank analysis); this kernel serves the others, and every sweep of a plan whose
// blocks are wider than 6 (their state does not fit a wavefront's registers).
//
// One wavefront runs one (job, sweep):
//   caps     every side message enters with the part still to be absorbed an isometry: the left-canonical
//            chain (successive Householder QR) of the message -- of its leg-reversed form when the sweep walks
//            it from its first site -- is consumed from its weighted end. Cap operator t is CT_t[P][v][Q]
//            (old cap bond P, emitted vertical bond v, new cap bond Q), bonds min(2^j, 2^(K-j)) <= 16.
//   state    the boundary MPS: top cap site [q][d], the kp crossing sites [a][h][b], bottom cap site [d][q],
//            bonds padded to 16 (chi <= 16), to 32 once a column is absorbed.
//   column   pass 1, top to bottom: each site absorbs its column tensor (the caps their cap operator), is
//            multiplied by the carry R of the site above and factored M = Q R by Householder reflections whose
//            vectors stay in the wavefront while it factors (the owning lanes' registers, broadcast through
//            LDS); the vectors (Q in compact form) go to the item's workspace slot, R (unit Frobenius norm, the
//            norm into the log-scale) down to the next site. The bottom cap keeps M. Pass 2, bottom to top:
//            N = Q C (the reflections applied to the carry C from below; Q is never formed) as a (left bond) x
//            (leg, right bond) matrix, one-sided Jacobi SVD, the chi largest singular values kept: their right
//            singular vectors are the new site, N V (unit norm) the carry; the top cap takes Q C.
//   end      the chain contracted to the dense 2^kp message; normalisation (remark 3), damping (remark 7) and
//            distance term (remark 4) as in the dense kernels, or the closing overlap of Lemma 3.1.
// Bound by the latency of one wavefront's chain of reflections and Jacobi rounds (few jobs) or by FP64 issue (many).
// Bonds are tracked at the number of values kept: rows, columns, reflections and Jacobi rounds beyond them are left out
// (they are zero and would change nothing), half the registers where a carry has at most 16 rows or a bond at most 8
// values. d = 13, 8 x 8 blocks at chi 16, 16 syndromes: 475 -> 271 ms; d = 9, 6 x 6 at chi 12, 4: 184 -> 72 ms.
// Sweeps whose every bond stays within 8 (trunc_shape.hpp) have a kernel of their own, trunc_narrow.hip.
// Keeping the chi largest values at every bond is the textbook QR + truncated-SVD compression: the part left
// of a bond is an isometry when it is truncated, so each cut keeps the chi largest Schmidt values of the
// current state. Where a bond carries at most chi values the SVD keeps them all (the state is unchanged).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "geom.hpp"
#include "sweep_launch.hpp"
#include "trunc_shape.hpp"
#include "wave_mps.hpp"

namespace bbp {
namespace {

using namespace wmps;

constexpr int KM = TRUNC_KMAX;
constexpr int TS = 16 * 2 * 16;   // one compressed site [a][h][b] (a, b < 16), or one cap operator [P][v][Q]
// workspace slot of one item, in doubles
constexpr int W_A = 0;                      // sites 0 .. kp+1
constexpr int W_Q = W_A + (KM + 2) * TS;    // pass-1 factors of sites 0 .. kp; site kp+1 keeps its matrix M
constexpr int W_CT = W_Q + (KM + 2) * TQ;   // cap operators: top t = 0 .. kt-1, then bottom
constexpr int W_SLOT = W_CT + 2 * KM * TS;

// LDS pool in doubles (the phases never overlap)
constexpr int P1 = 32 * 32 + 2 * 64 + 32 + 2 * TS;            // R carry, vector buffers, betas, site, CT (or Bb)
constexpr int P2 = 64 * XS + 32 * 16 + 32;                    // exchange (then V), carry C, singular values
constexpr int PC = 256 + 32 * 32 + 32;                        // chain: matrix, vectors, betas
constexpr int PE = 4 * 256;                                   // end: left / right chains (ping-pong)
constexpr int POOL = std::max(std::max(P1, P2), std::max(PC, PE));

__device__ __forceinline__ int bitrev(int w, int K) { return (int)(__brev((unsigned)w) >> (32 - K)); }

// Entry e = up*8 + in*4 + down*2 + out of the frame table at sweep step t, position i, in FP64: checks are
// COPY tensors (0 / 1), qubits one of the four Pauli probabilities pq (indexed x * 2 + z, as site_entry's).
__device__ __forceinline__ double tab(const SweepDesc& s, int L, const uint8_t* lab, const double* pq, int t, int i,
                                      int e) {
  int r, c;
  frame_site(s.frame, s.r0, s.c0, s.kr, s.kc, t, i, r, c);
  const float m = site_entry(s.frame, L, r, c, lab[r * L + c], 1.0f, 2.0f, 3.0f, 4.0f, e);
  if ((r + c) & 1) return (double)m;
  const int k = (int)m;
  return k == 0 ? 0.0 : pq[k - 1];
}

// Left-canonical chain of the K-leg vector in W[0 .. 2^K) (leg 0 most significant; W is overwritten): site
// j = A_j[a][v][q] with natural bonds. transposed: written as the cap operator CT_{K-1-j}[q][v][a] (the chain
// absorbed from its weighted end); else as site j itself, [a][v][q]. out must be zero beyond the bonds.
__device__ __forceinline__ void chain(double* W, double* Hv, double* Hb, int K, double* out, bool transposed) {
  const int ln = threadIdx.x;
  int b = 1;
  for (int j = 0; j < K - 1; ++j) {
    const int m = 2 * b, n = 1 << (K - j - 1), k = std::min(m, n);
    // Householder QR of W as an m x n row-major matrix
    for (int c = 0; c < k; ++c) {
      const double xr = (ln < m && ln >= c) ? W[ln * n + c] : 0.0;
      const double alpha = W[c * n + c];
      const double nrm = sqrt(wsum(xr * xr));
      double beta = 0.0, vj = alpha, diag = alpha;
      if (nrm > 0.0) {
        const double sg = (alpha >= 0.0) ? 1.0 : -1.0;
        vj = alpha + sg * nrm;
        beta = 1.0 / (nrm * (nrm + fabs(alpha)));
        diag = -sg * nrm;
      }
      if (ln < 32) Hv[c * 32 + ln] = (ln == c) ? vj : ((ln > c && ln < m) ? xr : 0.0);
      if (ln == 0) Hb[c] = beta;
      wave_sync();
      for (int col = c + 1 + ln; col < n; col += 64) {
        double w = 0.0;
        for (int r = c; r < m; ++r) w += Hv[c * 32 + r] * W[r * n + col];
        w *= beta;
        for (int r = c; r < m; ++r) W[r * n + col] -= w * Hv[c * 32 + r];
      }
      wave_sync();
      if (ln == 0) W[c * n + c] = diag;
      if (ln > c && ln < m) W[ln * n + c] = 0.0;
      wave_sync();
    }
    // Q (m x k): lane q forms column q by applying the reflections to the unit vector e_q
    if (ln < k) {
      double qv[32];
#pragma unroll
      for (int r = 0; r < 32; ++r) qv[r] = (r == ln) ? 1.0 : 0.0;
      for (int c = k - 1; c >= 0; --c) {
        double w = 0.0;
#pragma unroll
        for (int r = 0; r < 32; ++r) w += (r >= c && r < m) ? Hv[c * 32 + r] * qv[r] : 0.0;
        w *= Hb[c];
#pragma unroll
        for (int r = 0; r < 32; ++r)
          if (r >= c && r < m) qv[r] -= w * Hv[c * 32 + r];
      }
#pragma unroll
      for (int r = 0; r < 32; ++r) {
        if (r >= m) break;
        const int a = r >> 1, v = r & 1;
        if (transposed) out[(K - 1 - j) * TS + ln * 32 + v * 16 + a] = qv[r];
        else out[j * TS + a * 32 + v * 16 + ln] = qv[r];
      }
    }
    wave_sync();   // W now holds R (k x n): rows 0 .. k-1, the next step's (2k) x (n/2) matrix
    b = k;
  }
  // last site: A_{K-1}[a][v][0] = rest[a][v]
  for (int e = ln; e < 2 * b; e += 64) {
    const int a = e >> 1, v = e & 1;
    if (transposed) out[0 * TS + v * 16 + a] = W[e];
    else out[(K - 1) * TS + a * 32 + v * 16] = W[e];
  }
  wave_sync();
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void trunc_sweep_kernel(SweepArgs a) {
  const int ln = threadIdx.x, hi = ln >> 1, par = ln & 1;
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
  double pq[4];
  if (G.pdev) {
    const double pj = G.pdev[job >> 2];
    pq[0] = 1.0 - pj;
    pq[1] = pq[2] = pq[3] = pj / 3.0;
  } else {
    for (int k = 0; k < 4; ++k) pq[k] = G.pq[(k & 1) << 1 | k >> 1];   // (from the order of codes x + 2z)
  }
  const float* mbase = G.msgs + job * G.M * (int64_t)ms;
  double* ws = a.tws + (int64_t)blockIdx.x * W_SLOT;
  double* A = ws + W_A;
  double* Q = ws + W_Q;
  double* CT = ws + W_CT;

  __shared__ double pool[POOL];
  __shared__ int left[KM + 2], refl[KM + 1];   // left bond of site i (1 .. kp + 1), reflections of site i (0 .. kp)
  const bool top = s.msg_top >= 0, bot = s.msg_bot >= 0, fwd = (s.frame == FRAME_E || s.frame == FRAME_S);

  // ---- caps and the initial state ----
  // the chains fill the natural bonds only: clear the padded operators and sites they are read as
  if (top)
    for (int e = ln; e < kt * TS; e += 64) CT[e] = 0.0;
  if (bot)
    for (int e = ln; e < kt * TS; e += 64) CT[KM * TS + e] = 0.0;
  for (int e = ln; e < (kp + 2) * TS; e += 64) A[e] = 0.0;
  wave_sync();
  {
    double* W = pool;
    double* Hv = pool + 256;
    double* Hb = Hv + 32 * 32;
    for (int side = 0; side < 2; ++side) {
      const int id = side == 0 ? s.msg_top : s.msg_bot;
      if (id < 0) continue;
      for (int w = ln; w < (1 << kt); w += 64) W[w] = (double)mbase[id * (int64_t)ms + (fwd ? bitrev(w, kt) : w)];
      wave_sync();
      chain(W, Hv, Hb, kt, CT + side * KM * TS, true);
    }
    if (s.msg_init >= 0) {
      for (int w = ln; w < (1 << kp); w += 64) W[w] = (double)mbase[s.msg_init * (int64_t)ms + w];
      wave_sync();
      chain(W, Hv, Hb, kp, A + TS, false);
      if (ln >= 1 && ln <= kp + 1) left[ln] = 1 << std::min(ln - 1, kp + 1 - ln);
    } else {
      if (ln >= 1 && ln <= kp + 1) left[ln] = 1;
      for (int i = 1; i <= kp; ++i)
        if (ln == 0) A[i * TS] = 1.0;   // every in-leg at its only value 0
    }
    if (ln == 0) {
      A[0] = 1.0;                  // top cap [q = 0][d = 0]
      A[(kp + 1) * TS] = 1.0;      // bottom cap [d = 0][q = 0]
    }
  }
  wave_sync();

  double logs = 0.0;
  for (int t = 0; t < kt; ++t) {
    // cap bonds before and after this column (1 without a side message)
    const int pq0 = 1 << std::min(t, kt - t), pq1 = 1 << std::min(t + 1, kt - t - 1);
    // ---------------- pass 1: absorb and factor, top to bottom ----------------
    double* Rsh = pool;
    double* vb = Rsh + 32 * 32;
    double* Hb = vb + 2 * 64;
    double* Ash = Hb + 32;
    double* CTs = Ash + TS;
    double* Bb = CTs;   // the bottom cap's product replaces the cap operator it is formed from
    double x[32], rd;
    // top cap: M_0[q'][(d, v)] = sum_P S_0[P][d] CT[P][v][q'], rows q' < 16
    for (int e = ln; e < 256; e += 64) Ash[e] = A[e];
    if (top)
      for (int e = ln; e < TS; e += 64) CTs[e] = CT[t * TS + e];
    wave_sync();
    {
      const int d = hi >> 1, v = hi & 1;
#pragma unroll
      for (int k = 0; k < 32; ++k) x[k] = 0.0;
      if (top) {
        for (int P = 0; P < pq0; ++P) {
          const double sp = Ash[P * 16 + d];
#pragma unroll
          for (int k = 0; k < 8; ++k) x[k] += sp * CTs[P * 32 + v * 16 + 2 * k + par];
        }
      } else if (v == 0 && par == 0) {
        x[0] = Ash[d];
      }
    }
    // rows q' < 16: registers k < 8. nrow: the rows of R that can be nonzero
    int nrow = __builtin_amdgcn_readfirstlane(std::min(top ? pq1 : 1, 2 * left[1]));
    qr64u<16, 8>(x, rd, nrow, vb, Hb);
    logs += store_r(x, rd, Rsh);
    store_v(x, nrow, Hb, Q);
    if (ln == 0) refl[0] = nrow;
    // crossing sites: M [(k, h)][(b, dn)] = sum_(a, u) R[k][(a, u)] (A_i T)[(a, u)][(h, b, dn)], factored
    for (int i = 1; i <= kp; ++i) {
      for (int e = ln; e < TS; e += 64) Ash[e] = A[i * TS + e];
      wave_sync();
      const int na = __builtin_amdgcn_readfirstlane(left[i]), nb = __builtin_amdgcn_readfirstlane(left[i + 1]);
      const int jmax = std::min(2 * nrow, 2 * nb);
      const int b = hi >> 1, dn = hi & 1;
      const double t00 = tab(s, L, lab, pq, t, i - 1, 0 * 8 + 0 * 4 + dn * 2 + par);
      const double t01 = tab(s, L, lab, pq, t, i - 1, 0 * 8 + 1 * 4 + dn * 2 + par);
      const double t10 = tab(s, L, lab, pq, t, i - 1, 1 * 8 + 0 * 4 + dn * 2 + par);
      const double t11 = tab(s, L, lab, pq, t, i - 1, 1 * 8 + 1 * 4 + dn * 2 + par);
#pragma unroll
      for (int k = 0; k < 32; ++k) x[k] = 0.0;
      // x[k] belongs to R's row k
      auto site = [&](auto rows) __attribute__((always_inline)) {
        constexpr int KR = decltype(rows)::value;
        for (int aa = 0; aa < na; ++aa) {
          const double a0 = Ash[(aa * 2 + 0) * 16 + b], a1 = Ash[(aa * 2 + 1) * 16 + b];
          const double b0 = a0 * t00 + a1 * t01, b1 = a0 * t10 + a1 * t11;
#pragma unroll
          for (int k = 0; k < KR; ++k) x[k] += Rsh[k * 32 + aa * 2] * b0 + Rsh[k * 32 + aa * 2 + 1] * b1;
        }
        wave_sync();   // every lane has read R
        qr64u<32, KR>(x, rd, jmax, vb, Hb);
      };
      if (nrow <= 16) site(std::integral_constant<int, 16>());
      else site(std::integral_constant<int, 32>());
      logs += store_r(x, rd, Rsh);
      store_v(x, jmax, Hb, Q + i * TQ);
      if (ln == 0) refl[i] = jmax;
      nrow = jmax;
    }
    // bottom cap: Bb[(d, v)][q'] = sum_P S[d][P] CT[P][v][q'], then M[l][q'] = sum R[l][(d, v)] Bb[(d, v)][q']
    for (int e = ln; e < 256; e += 64) Ash[e] = A[(kp + 1) * TS + e];
    if (bot)
      for (int e = ln; e < TS; e += 64) CTs[e] = CT[(KM + t) * TS + e];
    wave_sync();
    {
      double bv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = ln + 64 * u, dv = e >> 4, q = e & 15, d = dv >> 1, v = dv & 1;
        double acc = 0.0;
        if (bot) {
          for (int P = 0; P < pq0; ++P) acc += Ash[d * 16 + P] * CTs[P * 32 + v * 16 + q];
        } else if (v == 0 && q == 0) {
          acc = Ash[d * 16];
        }
        bv[u] = acc;
      }
      wave_sync();   // every lane has read the operator before Bb overwrites it
#pragma unroll
      for (int u = 0; u < 8; ++u) Bb[ln + 64 * u] = bv[u];
    }
    wave_sync();
    {
      double* Mg = Q + (kp + 1) * TQ;
      const int nd = __builtin_amdgcn_readfirstlane(left[kp + 1]);
#pragma unroll 1
      for (int qq = 0; qq < 8; ++qq) {
        const int q = 8 * par + qq;
        double acc = 0.0;
#pragma unroll 4
        for (int dv = 0; dv < 2 * nd; ++dv) acc += Rsh[hi * 32 + dv] * Bb[dv * 16 + q];
        Mg[hi * 16 + q] = acc;
      }
    }
    wave_sync();

    // ---------------- pass 2: truncating SVD sweep, bottom to top ----------------
    double* Xsh = pool;
    double* Csh = Xsh + 64 * XS;
    double* sig = Csh + 32 * 16;
    int nk = bot ? pq1 : 1;   // the right bond
    for (int i = kp + 1; i >= 1; --i) {
      const double* Mg = Q + (kp + 1) * TQ;   // the bottom cap's M [l][q']
      double y[16];
      if (i == kp + 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) y[k] = par == 0 ? Mg[hi * 16 + k] : 0.0;
      } else {
        // N = Q_i C, then from the column layout to rows: lane (l, t) takes N[l][(t, k)] = X[2l + t][k]
        double X[16];
        apply_q(X, __builtin_amdgcn_readfirstlane(refl[i]), Q + i * TQ, Csh);
        cols_to_rows(X, Xsh, y);
      }
      // (N has the rows of site i - 1's R)
      logs += svd_step(y, __builtin_amdgcn_readfirstlane(refl[i - 1]), nk, chi, Xsh, Csh, sig, A + i * TS, i == kp + 1, nk);
      if (ln == 0) left[i] = nk;
    }
    // top cap: S_0[q'][j] = sum_m Q_0[q'][m] C[m][j], unit Frobenius norm
    {
      // rows q' < 16 of Q_0 C sit in the lanes of quarter 0: S_0[q'][kc] = X[q']
      double X[16];
      apply_q(X, __builtin_amdgcn_readfirstlane(refl[0]), Q, Csh);
      double f = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) f += (ln < 16) ? X[r] * X[r] : 0.0;
      const double fro = sqrt(wsum(f));
      const double inv = (fro > 0.0) ? 1.0 / fro : 0.0;
      if (ln < 16) {
#pragma unroll
        for (int r = 0; r < 16; ++r) A[r * 16 + ln] = X[r] * inv;
      }
      logs += log(fro);
    }
    wave_sync();
  }

  // ---------------- the dense message: left chain x right chain ----------------
  const int hl = kp / 2, hr = kp - hl;
  // left chain in pool[0 .. 512) and right chain in pool[512 .. 1024), each ping-ponging between halves
  for (int e = ln; e < 16; e += 64) {
    pool[e] = A[e];                              // top cap row q' = 0
    pool[512 + e] = A[(kp + 1) * TS + e * 16];   // bottom cap column q' = 0
  }
  wave_sync();
  int lc = 0, rc = 0;
  for (int i = 1; i <= hl; ++i) {   // L_i[(pre, h)][b] = sum_a L_{i-1}[pre][a] S_i[a][h][b]
    const int n = (1 << i) * 16;
    for (int e = ln; e < n; e += 64) {
      const int b = e & 15, ph = e >> 4, pre = ph >> 1, h = ph & 1;
      double acc = 0.0;
      for (int aa = 0; aa < 16; ++aa) acc += pool[lc * 256 + pre * 16 + aa] * A[i * TS + aa * 32 + h * 16 + b];
      pool[(lc ^ 1) * 256 + e] = acc;
    }
    wave_sync();
    lc ^= 1;
  }
  for (int i = kp; i > hl; --i) {   // R_i[(h, suf)][a] = sum_b S_i[a][h][b] R_{i+1}[suf][b]
    const int nsuf = 1 << (kp - i), n = 2 * nsuf * 16;
    for (int e = ln; e < n; e += 64) {
      const int aa = e & 15, hs = e >> 4, h = hs / nsuf, suf = hs - h * nsuf;
      double acc = 0.0;
      for (int b = 0; b < 16; ++b) acc += A[i * TS + aa * 32 + h * 16 + b] * pool[512 + rc * 256 + suf * 16 + b];
      pool[512 + (rc ^ 1) * 256 + e] = acc;
    }
    wave_sync();
    rc ^= 1;
  }
  double out[4];
  const int H = 1 << kp;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int e = ln + 64 * r;
    double acc = 0.0;
    if (e < H) {
      const int hL = e >> hr, hR = e & ((1 << hr) - 1);
      for (int b = 0; b < 16; ++b) acc += pool[lc * 256 + hL * 16 + b] * pool[512 + rc * 256 + hR * 16 + b];
    }
    out[r] = acc;
  }

  if (a.mode == 1) {
    double w = 0.0;
    if (s.msg_close >= 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = ln + 64 * r;
        if (e < H) w += out[r] * (double)mbase[s.msg_close * (int64_t)ms + e];
      }
    } else if (ln == 0) {
      w = out[0];
    }
    w = wsum(w);
    if (ln == 0) G.lnW[job * G.nblocks + s.block] = (w > 0.0) ? logs + log(w) : NAN;
    return;
  }
  // normalised new message, damping against the old one (unit norm), distance term
  float* mo = G.msgs + (job * G.M + s.msg_out) * (int64_t)ms;
  double f2 = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) f2 += out[r] * out[r];
  const double inv = 1.0 / sqrt(wsum(f2));
  double old[4], dm[4], g2 = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int e = ln + 64 * r;
    old[r] = (e < H) ? (double)mo[e] : 0.0;
    dm[r] = (1.0 - (double)a.eta) * out[r] * inv + (double)a.eta * old[r];
    g2 += dm[r] * dm[r];
  }
  const double ginv = 1.0 / sqrt(wsum(g2));
  double dd = 0.0, ss = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double fm = dm[r] * ginv;
    dd += (fm - old[r]) * (fm - old[r]);
    ss += (fm + old[r]) * (fm + old[r]);
    dm[r] = fm;
  }
  dd = wsum(dd);
  ss = wsum(ss);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int e = ln + 64 * r;
    if (e < H) mo[e] = (float)dm[r];
  }
  if (ln == 0) G.terms[job * G.M + s.msg_out] = 0.5 * dd * ss;
}

}  // namespace

size_t trunc_slot_bytes() { return std::max((size_t)W_SLOT * sizeof(double), trunc_narrow_slot_bytes()); }

hipError_t launch_trunc_sweeps(hipStream_t st, const SweepArgs& a, bool narrow) {
  if (a.items <= 0) return hipSuccess;
  if (!a.tws || a.tws_slots <= 0) return hipErrorInvalidValue;
  SweepArgs b = a;
  for (int64_t base = 0; base < a.items; base += a.tws_slots) {
    b.item_base = base;
    const int64_t n = std::min<int64_t>(a.tws_slots, a.items - base);
    if (narrow)
      launch_trunc_narrow((unsigned)n, st, b);
    else
      trunc_sweep_kernel<<<dim3((unsigned)n), dim3(64), 0, st>>>(b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace bbp
