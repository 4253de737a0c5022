// kernels_eig.hip - lowest eigenpairs of the projected matrix T = Q^T H Q (Rayleigh-Ritz, eq. tilde_H):
// one workgroup, Householder tridiagonalisation, multisection, inverse iteration, back-transformation.
//
// T is small (m <= 512, mostly <= 128), so every phase is a chain of dependent steps and the time is
// latency: m = 64, 4 pairs 235 -> 163 us, m = 128, 8 pairs 630 -> 387 us against the form with three
// barriers a step, a division per Sturm row and the vector in LDS.
//   tridiagonalisation  the trailing block of at most 128 rows lives in the registers of 4 waves, one per
//                       SIMD (wave w holds rows w, w + 4, ...; lane i columns i and i + 64).  Each wave
//                       forms the Householder vector for itself, so a step has one barrier (the partial
//                       sums of A v) instead of three; square root and divisions from the hardware
//                       approximations with Newton steps.  A step is bound by the issue of its few hundred
//                       dependent instructions: with two waves per SIMD the part that all waves repeat
//                       costs twice (1.6 us a step at m = 64).  The wave's own entries of u, w and v are
//                       read back from LDS as pairs: a readlane per entry costs more.
//   multisection        Sturm counts by the three-term recurrence of the leading minors, rescaled every
//                       8 steps: one dependent FMA per row instead of a division.
//   inverse iteration   one lane per vector, operands of the next rows independent of the carried
//                       values, reciprocal pivots kept; arrays interleaved by vector (no bank conflicts).
//   back-transformation one wave per vector, its entries in registers.
#include <type_traits>

#include "common.h"
#include "wave.h"

namespace sppc {

namespace {

constexpr int EIG_T = 128;        // rows of the trailing block held in registers
constexpr int EIG_MAX = 512;
constexpr int EIG_BUF = 16384;    // doubles of LDS work space
constexpr int EIG_HV = EIG_T * (EIG_T - 1) / 2;  // packed Householder vectors of the trailing block

// 1 / b refined by two Newton-Raphson steps (relative error 4.6e-8 of the hardware's, 2.1e-15 after one step,
// 1.1e-16 after two); b nonzero, finite, and of ordinary size
__device__ inline double fast_rcp(double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(r, fma(-b, r, 1.0), r);
  return fma(r, fma(-b, r, 1.0), r);
}

// Householder vector of the row x (alpha = x[j + 1], sigma = the sum of squares beyond): e = the new
// off-diagonal, beta, and rv with v = (1, rv x[j + 2], ...)
__device__ inline void reflector(double alpha, double sigma, double& e, double& beta, double& rv) {
  if (!(sigma > 0.0)) {
    e = alpha;
    beta = 0.0;
    rv = 0.0;
    return;
  }
  const double q = fma(alpha, alpha, sigma);
  double mu, rmu;
  if (q > 1e-280 && q < 1e280) {
    double y = __builtin_amdgcn_rsq(q);
    y = fma(0.5 * y, fma(-q * y, y, 1.0), y);
    y = fma(0.5 * y, fma(-q * y, y, 1.0), y);
    mu = q * y;
    mu = fma(0.5 * y, fma(-mu, mu, q), mu);
    rmu = y;
    rv = fast_rcp(fabs(alpha) + mu);
  } else {
    mu = sqrt(q);
    rmu = 1.0 / mu;
    rv = 1.0 / (fabs(alpha) + mu);
  }
  beta = fma(fabs(alpha), rmu, 1.0);
  e = alpha < 0.0 ? mu : -mu;
  if (alpha < 0.0) rv = -rv;
}

// Sturm count (eigenvalues below x) of the tridiagonal (d, sqrt(e2)): sign changes of the leading minors
// p_i = (d_i - x) p_{i-1} - e2_{i-1} p_{i-2}.  The matrix is scaled to norm < 1 and e2 >= 1e-34 (a coupling
// of 1e-17, below the rounding of the norm), so 8 steps neither overflow nor underflow.  A minor that is
// exactly zero counts as either sign: the next has the sign opposite to its predecessor's.  Rows beyond m
// (up to a multiple of 8) hold d = 4, which changes no sign.
__device__ __forceinline__ int sturm_count(int m, const double* d, const double* e2, double x) {
  double p = 1.0, pm = 0.0;
  uint32_t sg = 0;  // signs of the minors, the latest in bit 0
  int cnt = 0;
  for (int i = 0; i < m; i += 8) {
    double dd[8], ee[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      dd[u] = d[i + u] - x;
      ee[u] = e2[i + u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double pn = fma(dd[u], p, -(ee[u] * pm));
      pm = p;
      p = pn;
      sg = __builtin_amdgcn_alignbit(sg, (uint32_t)__double2hiint(pn), 31);
    }
    cnt += __popc((sg ^ (sg >> 1)) & 0xFFu);
    const int f = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pm)));
    p = ldexp(p, f);
    pm = ldexp(pm, f);
  }
  return cnt;
}

// Two solves (Tri - lam I) y = y by Gaussian elimination with partial pivoting, from a random start
// (the shift is the eigenvalue to a few ulp: two suffice).  Row k of this vector: index k * nw of the
// arrays; r0 = 1 / u0, u2 = e[k + 1] where the rows were interchanged.  Rows go in batches of B whose
// operands are loaded together and whose results are stored together, so that the chain of carried
// values waits for LDS once a batch.
template <int B>
__device__ __forceinline__ void inverse_iteration(int m, int nw, const double* d, const double* e, double lam,
                                                  double epsp, uint32_t seed, double* u1, double* l, double* r0,
                                                  double* y, unsigned char* piv) {
  uint32_t h = seed;
  auto start = [&]() {  // in [0.5, 1)
    h = h * 1664525u + 1013904223u;
    return __hiloint2double((int)(0x3FE00000u | (h >> 12)), 0);
  };
  auto away = [&](double a) { return fabs(a) < epsp ? (a >= 0.0 ? epsp : -epsp) : a; };
  double ca = d[0] - lam, cb = m > 1 ? e[0] : 0.0, cur = start();
  for (int k0 = 0; k0 < m - 1; k0 += B) {
    double ee[B + 1], na[B], b1[B], bl[B], br[B], by[B];
    unsigned swb = 0;
#pragma unroll
    for (int u = 0; u < B + 1; ++u) ee[u] = e[min(k0 + u, m - 1)];  // e[m - 1] = 0
#pragma unroll
    for (int u = 0; u < B; ++u) na[u] = d[min(k0 + u + 1, m - 1)] - lam;
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (k0 + u < m - 1) {
        const double yn = start();
        const bool sw = fabs(ca) < fabs(ee[u]);
        const double pv = away(sw ? ee[u] : ca);
        const double r = fast_rcp(pv);
        const double mult = (sw ? ca : ee[u]) * r;
        b1[u] = sw ? na[u] : cb;
        by[u] = sw ? yn : cur;
        cur = fma(-mult, by[u], sw ? cur : yn);
        ca = fma(-mult, b1[u], sw ? cb : na[u]);
        cb = sw ? -mult * ee[u + 1] : ee[u + 1];
        bl[u] = mult;
        br[u] = r;
        swb |= sw ? 1u << u : 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (k0 + u < m - 1) {
        const int q = (k0 + u) * nw;
        u1[q] = b1[u];
        l[q] = bl[u];
        r0[q] = br[u];
        y[q] = by[u];
        piv[q] = (swb >> u) & 1u;
      }
    }
  }
  const double rl = fast_rcp(away(ca));
  for (int it = 0; it < 2; ++it) {
    if (it == 1) {
      cur = y[0];
      for (int k0 = 0; k0 < m - 1; k0 += B) {
        double yn[B], ml[B];
        bool sw[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int q = min(k0 + u, m - 2) * nw;
          yn[u] = y[q + nw];
          ml[u] = l[q];
          sw[u] = piv[q];
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (k0 + u < m - 1) {
            const double yk = sw[u] ? yn[u] : cur;
            cur = fma(-ml[u], yk, sw[u] ? cur : yn[u]);
            yn[u] = yk;
          }
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
          if (k0 + u < m - 1) y[(k0 + u) * nw] = yn[u];
      }
    }
    double y1 = cur * rl, y2 = 0.0;
    y[(m - 1) * nw] = y1;
    for (int k0 = m - 2; k0 >= 0; k0 -= B) {
      double a1[B], a2[B], rr[B], yk[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int k = max(k0 - u, 0), q = k * nw;
        a1[u] = u1[q];
        rr[u] = r0[q];
        yk[u] = y[q];
        a2[u] = piv[q] ? e[k + 1] : 0.0;  // (e[m - 1] = 0)
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        if (k0 - u >= 0) {
          const double v = fma(-a1[u], y1, fma(-a2[u], y2, yk[u])) * rr[u];
          y2 = y1;
          y1 = v;
          yk[u] = v;
        }
      }
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (k0 - u >= 0) y[(k0 - u) * nw] = yk[u];
    }
  }
}

// Normalisation, Gram-Schmidt within clusters of close eigenvalues, back-transformation and output.
// Y: vectors as inverse_iteration left them; Yn: nw x m, row by row.  hv: packed Householder vectors
// (HVL), else they are the rows of A (ld m); load_hv packs them from A first.
template <int NR, int NTH, bool HVL>
__device__ __forceinline__ void eig_vectors(int m, int nw, const double* lam, double ctol, const double* Y, double* Yn,
                                            const double* A, double* hv, bool load_hv, const double* bl, double* dots,
                                            double unscale, double* __restrict__ wout, double* __restrict__ V,
                                            int64_t ldv) {
  constexpr int NW = NTH / 64;
  const int t = threadIdx.x, wv = t >> 6, ln = t & 63;
  for (int c = wv; c < nw; c += NW) {
    double y[NR], mx = 0.0, s = 0.0;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int i = ln + 64 * q;
      y[q] = i < m ? Y[(int64_t)i * nw + c] : 0.0;
      mx = fmax(mx, fabs(y[q]));
    }
    mx = wave_max(mx);
    const double rmx = mx > 0.0 ? 1.0 / mx : 0.0;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      y[q] *= rmx;
      s = fma(y[q], y[q], s);
    }
    s = wave_sum(s);
    const double rs = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
    for (int q = 0; q < NR; ++q)
      if (ln + 64 * q < m) Yn[(int64_t)c * m + ln + 64 * q] = y[q] * rs;
  }
  if (load_hv) {
    __syncthreads();  // the vectors loaded overwrite Y
    for (int j = wv; j + 2 < m; j += NW) {
      const int len = m - 1 - j;
      double* dst = hv + (int64_t)j * (m - 1) - (int64_t)j * (j - 1) / 2;
      for (int i = ln; i < len; i += 64) dst[i] = A[(int64_t)j * m + j + 1 + i];
    }
  }
  __syncthreads();
  // vectors of close eigenvalues: classical Gram-Schmidt twice against the earlier members of their
  // cluster (dots by all waves, the update by wave 0)
  for (int c = 1; c < nw; ++c) {
    int c0 = c;
    while (c0 > 0 && lam[c0] - lam[c0 - 1] <= ctol) --c0;
    if (c0 == c) continue;  // uniform across the block
    double* yc = Yn + (int64_t)c * m;
    for (int pass = 0; pass < 2; ++pass) {
      for (int c2 = c0 + wv; c2 < c; c2 += NW) {
        const double* y2 = Yn + (int64_t)c2 * m;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q)
          if (ln + 64 * q < m) s = fma(yc[ln + 64 * q], y2[ln + 64 * q], s);
        s = wave_sum(s);
        if (ln == 0) dots[c2] = s;
      }
      __syncthreads();
      if (wv == 0) {
        double y[NR], s = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) y[q] = ln + 64 * q < m ? yc[ln + 64 * q] : 0.0;
        for (int c2 = c0; c2 < c; ++c2) {
          const double dt = dots[c2];
          const double* y2 = Yn + (int64_t)c2 * m;
#pragma unroll
          for (int q = 0; q < NR; ++q)
            if (ln + 64 * q < m) y[q] = fma(-dt, y2[ln + 64 * q], y[q]);
        }
#pragma unroll
        for (int q = 0; q < NR; ++q) s = fma(y[q], y[q], s);
        s = wave_sum(s);
        const double rs = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q)
          if (ln + 64 * q < m) yc[ln + 64 * q] = y[q] * rs;
      }
      __syncthreads();
    }
  }
  // V = H_0 H_1 ... H_{m-3} Y: each wave applies all reflectors to its own columns, two at a time;
  // lane ln holds the entries ln, ln + 64, ... of a column.  The largest entry becomes positive.
  for (int c = wv; c < nw; c += 2 * NW) {
    const int cb = c + NW < nw ? c + NW : c;
    double y[2][NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int i = ln + 64 * q;
      y[0][q] = i < m ? Yn[(int64_t)c * m + i] : 0.0;
      y[1][q] = i < m ? Yn[(int64_t)cb * m + i] : 0.0;
    }
    // the vector of step j is requested a step ahead (v_j: entries j + 1..; an index that stays
    // non-negative in every part)
    auto vec_of = [&](int j, double (&x)[NR]) {
      const int v0 = HVL ? j * (m - 1) - j * (j - 1) / 2 : j * m + j + 1;
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = ln + 64 * q;
        x[q] = 0.0;
        if (i > j && i < m) x[q] = HVL ? hv[v0 + (i - j - 1)] : A[v0 + (i - j - 1)];
      }
    };
    double xn[NR];
    if (m >= 3) vec_of(m - 3, xn);
    for (int j = m - 3; j >= 0; --j) {
      const double b = bl[j];
      double x[NR], s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int q = 0; q < NR; ++q) x[q] = xn[q];
      if (j > 0) vec_of(j - 1, xn);
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        s0 = fma(x[q], y[0][q], s0);
        s1 = fma(x[q], y[1][q], s1);
      }
      s0 = wave_sum(s0) * b;
      s1 = wave_sum(s1) * b;
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        y[0][q] = fma(-s0, x[q], y[0][q]);
        y[1][q] = fma(-s1, x[q], y[1][q]);
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int cc = k ? cb : c;
      if (k && cb == c) break;
      double best = -1.0, val = 0.0;
      int bi = 0;
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = ln + 64 * q;
        if (i < m && fabs(y[k][q]) > best) {
          best = fabs(y[k][q]);
          val = y[k][q];
          bi = i;
        }
      }
      for (int o = 32; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best, o), ov = __shfl_xor(val, o);
        const int oi = __shfl_xor(bi, o);
        if (ob > best || (ob == best && oi < bi)) {
          best = ob;
          val = ov;
          bi = oi;
        }
      }
      const double sgn = val < 0.0 ? -1.0 : 1.0;
#pragma unroll
      for (int q = 0; q < NR; ++q)
        if (ln + 64 * q < m) V[(int64_t)(ln + 64 * q) * ldv + cc] = sgn * y[k][q];
      if (ln == 0) wout[cc] = lam[cc] * unscale;
    }
  }
}

// NTH = 512: m <= 64 C, all in registers and LDS (C columns of the block per lane).  NTH = 1024, C = 2: the leading rows of a larger T are
// reduced in global memory by all 16 waves until the trailing block fits.
// scratch (doubles): A[m*m] | d[m] | e[m] | beta[m] | work of the inverse iteration when LDS is short
template <int NTH, int C>
__global__ __launch_bounds__(NTH) void k_sym_eig(int m, int nw, const double* __restrict__ S, int64_t lds,
                                                 double* __restrict__ wout, double* __restrict__ V, int64_t ldv,
                                                 double* __restrict__ scr) {
  constexpr bool HEAD = NTH > 512;
  constexpr int TW = HEAD ? 8 : 4;     // waves that hold the trailing block (128 registers a lane cap HEAD's)
  constexpr int RW = 64 * C / TW;      // rows a wave holds
  constexpr int RL = 64 / TW;          // its rows below 64
  constexpr int GR = HEAD ? 4 : 8;     // rows taken together
  constexpr int LDV = (HEAD ? EIG_MAX : EIG_T) + 8;
  __shared__ double buf[EIG_BUF];
  __shared__ double vec[(HEAD ? 7 : 6) * LDV];
  __shared__ double sc;
  const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), ln = t & 63;
  double* const A = scr;
  double* const dg = scr + (int64_t)m * m;
  double* const eg = dg + m;
  double* const bg = eg + m;
  double* const wkg = bg + m;
  // d, e, beta, e^2 of the tridiagonal, eigenvalues, dots; in the first phase of HEAD the same space
  // holds v, v', 4 partial sums of A v, and w
  double* const dl = vec + (HEAD ? 2 * LDV : 0);
  double* const el = dl + LDV;
  double* const bl = el + LDV;
  double* const e2l = bl + LDV;
  double* const lam = e2l + LDV;
  double* const dots = HEAD ? vec : lam + LDV;
  int o = 0;  // rows reduced in global memory

  // The rank-2 update of step j - 1 is not applied in a pass of its own: step j applies it to row j as
  // it forms its Householder vector, and to the rest of the trailing block in the pass that forms A v.
  if constexpr (HEAD) {
    const int tg = t >> 8, tc = t & 255;
    for (int r = tg; r < m; r += 4)
      for (int c = tc; c < m; c += 256) A[(int64_t)r * m + c] = S[(int64_t)r * lds + c];
    __syncthreads();
    double* const psh = vec + 2 * LDV;
    double* const wsh = vec + 6 * LDV;
    for (; m - o > EIG_T; ++o) {
      const int j = o;
      const bool pend = j > 0;
      double* const vc = vec + (j & 1) * LDV;
      const double* const up = vec + ((j & 1) ^ 1) * LDV;
      const int len = m - 1 - j;
      const double* xr = A + (int64_t)j * m + j + 1;
      if (w == 0) {
        const double u0 = pend ? up[0] : 0.0, w0 = pend ? wsh[0] : 0.0;
        double part = 0.0;
        for (int i = 1 + ln; i < len; i += 64) {
          const double x = pend ? xr[i] - (u0 * wsh[1 + i] + w0 * up[1 + i]) : xr[i];
          part = fma(x, x, part);
        }
        const double sigma = wave_sum(part);
        const double alpha = pend ? xr[0] - (u0 * wsh[1] + w0 * up[1]) : xr[0];
        double e, b, rv;
        reflector(alpha, sigma, e, b, rv);
        if (ln == 0) {
          dg[j] = A[(int64_t)j * m + j] - 2.0 * u0 * w0;
          eg[j] = e;
          bg[j] = b;
          sc = b;
        }
        for (int i = ln; i < len; i += 64) {
          const double x = pend ? xr[i] - (u0 * wsh[1 + i] + w0 * up[1 + i]) : xr[i];
          vc[i] = i == 0 ? 1.0 : x * rv;
        }
      }
      __syncthreads();
      const double b = sc;
      // keep v for the back-transformation in row j (no longer needed otherwise)
      for (int i = t; i < len; i += NTH) A[(int64_t)j * m + j + 1 + i] = vc[i];
      // p = b A v with the pending update (4 row groups x 256 columns)
      const int l0 = (len * tg) / 4, l1 = (len * (tg + 1)) / 4;
      for (int i = tc; i < len; i += 256) {
        double* col = A + (int64_t)(j + 1) * m + (j + 1) + i;
        const double ui = pend ? up[1 + i] : 0.0, wi = pend ? wsh[1 + i] : 0.0;
        double s0 = 0.0, s1 = 0.0;
        int l = l0;
        if (pend) {
          for (; l + 1 < l1; l += 2) {
            const double a0 = col[(int64_t)l * m] - (up[1 + l] * wi + wsh[1 + l] * ui);
            const double a1 = col[(int64_t)(l + 1) * m] - (up[2 + l] * wi + wsh[2 + l] * ui);
            col[(int64_t)l * m] = a0;
            col[(int64_t)(l + 1) * m] = a1;
            s0 += a0 * vc[l];
            s1 += a1 * vc[l + 1];
          }
          for (; l < l1; ++l) {
            const double a0 = col[(int64_t)l * m] - (up[1 + l] * wi + wsh[1 + l] * ui);
            col[(int64_t)l * m] = a0;
            s0 += a0 * vc[l];
          }
        } else {
          for (; l + 1 < l1; l += 2) {
            s0 += col[(int64_t)l * m] * vc[l];
            s1 += col[(int64_t)(l + 1) * m] * vc[l + 1];
          }
          for (; l < l1; ++l) s0 += col[(int64_t)l * m] * vc[l];
        }
        psh[tg * LDV + i] = s0 + s1;
      }
      __syncthreads();  // every read of the previous step's w is done
      // w = p - (b/2)(v^T p) v, by wave 0 (zero when b = 0: the update is then empty)
      if (w == 0) {
        double kp = 0.0;
        for (int i = ln; i < len; i += 64) {
          const double pi = b * (psh[i] + psh[LDV + i] + psh[2 * LDV + i] + psh[3 * LDV + i]);
          wsh[i] = pi;
          kp = fma(pi, vc[i], kp);
        }
        const double K = 0.5 * b * wave_sum(kp);
        for (int i = ln; i < len; i += 64) wsh[i] -= K * vc[i];
      }
      __syncthreads();
    }
  }

  // ---- the trailing block, rows o.. of T, in the registers of waves 0..TW-1
  const int L = m - o;
  double* const hv = buf;                   // packed v_j, j = 0..L-3
  double* const pp = buf + EIG_HV;          // [2][TW][128] partial sums of A v by step parity
  double* const rowb = pp + 2 * TW * EIG_T;  // [2][128] the next row, by step parity
  double* const own = rowb + 2 * EIG_T;     // [TW][3][RW] per wave: u, w and v at its own rows
  double* const kps = own + TW * 3 * RW;    // [2][TW] partial sums of v^T A v, by step parity
  double a[RW][C], u[2] = {0.0, 0.0}, wr[2] = {0.0, 0.0};  // with C = 1 the second entries stay 0
  if (w < TW) {
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int l = w + TW * r, i = ln + 64 * c;
        double x = 0.0;
        if (l < L && i < L) {
          if constexpr (HEAD) {
            const double* up = vec + ((o & 1) ^ 1) * LDV;
            const double* wsh = vec + 6 * LDV;
            x = A[(int64_t)(o + l) * m + o + i];
            if (o > 0) x -= up[l] * wsh[i] + wsh[l] * up[i];
          } else {
            x = S[(int64_t)l * lds + i];
          }
        }
        a[r][c] = x;
      }
    if (w == 0) {
      rowb[ln] = a[0][0];
      if constexpr (C == 2) rowb[64 + ln] = a[0][1];
    }
    for (int i = ln; i < 3 * RW; i += 64) own[w * 3 * RW + i] = 0.0;
  }
  __syncthreads();
  if constexpr (HEAD) {
    for (int i = t; i < o; i += NTH) {
      dl[i] = dg[i];
      el[i] = eg[i];
      bl[i] = bg[i];
    }
  }
  const bool two = C == 2 && L > 64;
  for (int j = 0; j + 2 < L; ++j) {
    double v[2] = {0.0, 0.0}, b = 0.0;
    if (w < TW) {
      const double* rb = rowb + (j & 1) * EIG_T;
      const double uj = lane_get(j < 64 ? u[0] : u[1], j & 63), wj = lane_get(j < 64 ? wr[0] : wr[1], j & 63);
      double x[2] = {0.0, 0.0};
#pragma unroll
      for (int c = 0; c < C; ++c) x[c] = rb[ln + 64 * c] - (uj * wr[c] + wj * u[c]);
      double sg = 0.0;
      if (ln > j + 1) sg = x[0] * x[0];
      if (two && ln + 64 > j + 1) sg = fma(x[1], x[1], sg);
      sg = wave_sum(sg);
      const double alpha = lane_get(j + 1 < 64 ? x[0] : x[1], (j + 1) & 63);
      double e, rv;
      reflector(alpha, sg, e, b, rv);
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int i = ln + 64 * c;
        v[c] = i <= j || i >= L ? 0.0 : i == j + 1 ? 1.0 : x[c] * rv;
      }
      if (w == 0) {
        const double dj = lane_get(j < 64 ? x[0] : x[1], j & 63);
        if (ln == 0) {
          dl[o + j] = dj;
          el[o + j] = e;
          bl[o + j] = b;
        }
      }
      if (w == j % TW) {
        double* dst = hv + j * (L - 1) - j * (j - 1) / 2 - (j + 1);
        if (ln > j && ln < L) dst[ln] = v[0];
        if (two && ln + 64 > j && ln + 64 < L) dst[ln + 64] = v[1];
      }
      // apply the pending update of step j - 1 to this wave's rows and form its part of A v, GR rows
      // at a time; the rows' own entries of u, w and v come from LDS (u and w written in the step before),
      // the next rows' requested ahead where registers allow.  (Rows up to j: v is zero there, and they are read no more.)
      double* const ow = own + w * 3 * RW;
      if (ln % TW == w) {
        ow[2 * RW + ln / TW] = v[0];
        if constexpr (C == 2) ow[2 * RW + RL + ln / TW] = v[1];
      }
      wave_lds_fence();
      double s0 = 0.0, s1 = 0.0;
      double* const nrow = rowb + ((j + 1) & 1) * EIG_T;
      const int g1 = (L - w + GR * TW - 1) / (GR * TW);  // groups of GR rows that this wave holds
      const int g0 = j >= w ? (j - w) / TW / GR : 0;      // first one with a row beyond j
      double ul[GR], wl[GR], vl[GR];
      auto own_rows = [&](int g, double (&ul_)[GR], double (&wl_)[GR], double (&vl_)[GR]) {
#pragma unroll
        for (int r = 0; r < GR; ++r) {
          ul_[r] = ow[GR * g + r];
          wl_[r] = ow[RW + GR * g + r];
          vl_[r] = ow[2 * RW + GR * g + r];
        }
      };
      if constexpr (!HEAD) own_rows(g0, ul, wl, vl);
#pragma unroll
      for (int g = 0; g < RW / GR; ++g) {
        if (g >= g0 && g < g1) {
          double un[GR], wn[GR], vn[GR];
          if constexpr (HEAD) own_rows(g, ul, wl, vl);
          else own_rows(g + 1 < RW / GR ? g + 1 : g, un, wn, vn);
#pragma unroll
          for (int r = 0; r < GR; ++r) {
            double* const ar = a[GR * g + r];
            ar[0] = fma(-ul[r], wr[0], fma(-wl[r], u[0], ar[0]));
            s0 = fma(ar[0], vl[r], s0);
            if constexpr (C == 2) {
              if (two) {
                ar[1] = fma(-ul[r], wr[1], fma(-wl[r], u[1], ar[1]));
                s1 = fma(ar[1], vl[r], s1);
              }
            }
            if (w + TW * (GR * g + r) == j + 1) {  // the next step's row
              nrow[ln] = ar[0];
              if constexpr (C == 2) nrow[64 + ln] = ar[1];
            }
          }
          if constexpr (!HEAD) {
#pragma unroll
            for (int r = 0; r < GR; ++r) {
              ul[r] = un[r];
              wl[r] = wn[r];
              vl[r] = vn[r];
            }
          }
        }
      }
      double* pj = pp + ((j & 1) * TW + w) * EIG_T;
      pj[ln] = s0;
      if (two) pj[64 + ln] = s1;
      const double kp = wave_sum(fma(s0, v[0], s1 * v[1]));
      if (ln == 0) kps[(j & 1) * TW + w] = kp;
    }
    __syncthreads();
    if (w < TW) {
      const double* pj = pp + (j & 1) * TW * EIG_T;
      double p[2] = {0.0, 0.0}, kp = 0.0;
#pragma unroll
      for (int g = 0; g < TW; ++g) {
        p[0] += pj[g * EIG_T + ln];
        if (two) p[1] += pj[g * EIG_T + 64 + ln];
        kp += kps[(j & 1) * TW + g];
      }
      // w = p - (b / 2)(v^T p) v with p = b A v
      const double K = 0.5 * b * b * kp;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int i = ln + 64 * c;
        wr[c] = i > j && i < L ? fma(-K, v[c], p[c] * b) : 0.0;
        u[c] = v[c];
      }
      double* const ow = own + w * 3 * RW;
      if (ln % TW == w) {
        ow[ln / TW] = u[0];
        if constexpr (C == 2) ow[RL + ln / TW] = u[1];
        ow[RW + ln / TW] = wr[0];
        if constexpr (C == 2) ow[RW + RL + ln / TW] = wr[1];
      }
      wave_lds_fence();
    }
  }
  // the last two rows, with the pending update of the last step
  if (w < TW) {
    if (w == 0 && L >= 2) {
      const int j = L - 2;
      const double* rb = rowb + (j & 1) * EIG_T;
      const double uj = lane_get(j < 64 ? u[0] : u[1], j & 63), wj = lane_get(j < 64 ? wr[0] : wr[1], j & 63);
      const double x0 = rb[ln] - (uj * wr[0] + wj * u[0]);
      const double x1 = C == 2 ? rb[64 + ln] - (uj * wr[1] + wj * u[1]) : 0.0;
      const double dj = lane_get(j < 64 ? x0 : x1, j & 63), ej = lane_get(j + 1 < 64 ? x0 : x1, (j + 1) & 63);
      if (ln == 0) {
        dl[o + j] = dj;
        el[o + j] = ej;
        bl[o + j] = 0.0;
      }
    }
    if (w == (L - 1) % TW) {
      double x = 0.0;
#pragma unroll
      for (int r = 0; r < RW; ++r)
        if (w + TW * r == L - 1) x = L - 1 < 64 ? a[r][0] - 2.0 * u[0] * wr[0] : a[r][C - 1] - 2.0 * u[1] * wr[1];
      x = lane_get(x, (L - 1) & 63);
      if (ln == 0) {
        dl[m - 1] = x;
        el[m - 1] = 0.0;
        bl[m - 1] = 0.0;
      }
    }
  }
  __syncthreads();

  // ---- scale by a power of two to norm < 1
  double tn = 0.0;
  for (int i = ln; i < m; i += 64)
    tn = fmax(tn, fabs(dl[i]) + (i > 0 ? fabs(el[i - 1]) : 0.0) + (i < m - 1 ? fabs(el[i]) : 0.0));
  tn = fmax(wave_max(tn), 1e-290);
  const int ex = __builtin_amdgcn_frexp_exp(tn);
  tn = ldexp(tn, -ex);
  __syncthreads();
  for (int i = t; i < m + 7; i += NTH) {  // e2l[i] couples rows i - 1 and i
    const double e = i < m ? ldexp(el[i], -ex) : 0.0;
    dl[i] = i < m ? ldexp(dl[i], -ex) : 4.0;
    el[i] = e;
    e2l[i + 1] = fmax(e * e, 1e-34);
    if (i == 0) e2l[0] = 0.0;
  }
  // the work arrays of the inverse iteration after the packed Householder vectors when they fit there,
  // else the vectors move to A (whose rows hold those of the steps in global memory already)
  const int64_t need = 4LL * nw * m + cdiv((int64_t)nw * m, 8);
  const bool keep = !HEAD && need <= EIG_BUF - EIG_HV;
  const bool inlds = keep || need <= EIG_BUF;
  if (!keep) {
    for (int j = w; j + 2 < L; j += NTH / 64) {
      const double* src = hv + j * (L - 1) - j * (j - 1) / 2;
      for (int i = ln; i < L - 1 - j; i += 64) A[(int64_t)(o + j) * m + o + j + 1 + i] = src[i];
    }
  }
  __syncthreads();

  // ---- eigenvalues: one wave per wanted eigenvalue; in each round its lanes evaluate the Sturm count
  // at 64 interior points of the current interval, which shrinks 65-fold (counts are monotone in x, so
  // the crossing is found by a ballot)
  {
    double lo = 1e300, hi = -1e300;
    for (int i = ln; i < m; i += 64) {
      const double r = (i > 0 ? fabs(el[i - 1]) : 0.0) + (i < m - 1 ? fabs(el[i]) : 0.0);
      lo = fmin(lo, dl[i] - r);
      hi = fmax(hi, dl[i] + r);
    }
    lo = -wave_max(-lo);
    hi = wave_max(hi);
    for (int idx = w; idx < nw; idx += NTH / 64) {
      double x0 = lo - 1e-14 * tn, x1 = hi + 1e-14 * tn;
      for (int it = 0; it < 40; ++it) {
        if (x1 - x0 <= 2.220446049250313e-16 * fmax(fabs(x0), fabs(x1)) + 1e-300) break;
        const double h = (x1 - x0) * (1.0 / 65.0);
        const double x = x0 + (ln + 1) * h;
        // the lowest P points have count <= idx (monotone); the eigenvalue lies between points P and P + 1
        const int P = __popcll(__ballot(x < x1 && sturm_count(m, dl, e2l, x) <= idx));
        const double na = P > 0 ? x0 + P * h : x0;
        const double nb = P < 64 ? x0 + (P + 1) * h : x1;
        if (!(na < nb) || (na == x0 && nb == x1)) break;
        x0 = na;
        x1 = fmin(nb, x1);
      }
      if (ln == 0) lam[idx] = 0.5 * (x0 + x1);
    }
  }
  __syncthreads();

  // ---- eigenvectors of the tridiagonal by inverse iteration, one lane per vector, then
  // eig_vectors: the normalised vectors take the place of u1; the Householder vectors go back to LDS
  // (packed) when they fit: each of the m sequential steps of the back-transformation then reads LDS,
  // not L2.  Where the arrays are is a template argument: an LDS array is reached through LDS
  // addresses alone.  (A pointer that may be either becomes a flat address, whose constant offset the
  // compiler folds into the instruction: the base then may lie below the LDS aperture, a fault.)
  const double epsp = 2.220446049250313e-16 * tn;
  const double unscale = ldexp(1.0, ex);
  const int yl = inlds && !keep ? nw * m : 0;
  const bool load_hv = !keep && m >= 3 && yl + (int64_t)(m - 1) * m / 2 <= EIG_BUF;
  auto vectors = [&](auto hvl, double* u1, double* hvp) __attribute__((always_inline)) {
    double* const ll = u1 + (int64_t)nw * m;
    double* const r0 = ll + (int64_t)nw * m;
    double* const Y = r0 + (int64_t)nw * m;
    unsigned char* const piv = (unsigned char*)(Y + (int64_t)nw * m);
    if (t < nw) {
      // repeated eigenvalues: separate the shifts slightly so the vectors differ
      int rep = 0;
      for (int c2 = t - 1; c2 >= 0 && lam[t] - lam[c2] < 10.0 * epsp; --c2) ++rep;
      inverse_iteration<HEAD ? 4 : 8>(m, nw, dl, el, lam[t] + 10.0 * epsp * rep, epsp, 0x9E3779B9u * (uint32_t)(t + 1), u1 + t,
                        ll + t, r0 + t, Y + t, piv + t);
    }
    __syncthreads();
    constexpr bool HVL = decltype(hvl)::value;
    if constexpr (HEAD) {
      if (m <= 256)
        eig_vectors<4, NTH, HVL>(m, nw, lam, 1e-3 * tn, Y, u1, A, hvp, load_hv, bl, dots, unscale, wout, V, ldv);
      else
        eig_vectors<8, NTH, HVL>(m, nw, lam, 1e-3 * tn, Y, u1, A, hvp, load_hv, bl, dots, unscale, wout, V, ldv);
    } else {
      if (m <= 64)
        eig_vectors<1, NTH, HVL>(m, nw, lam, 1e-3 * tn, Y, u1, A, hvp, load_hv, bl, dots, unscale, wout, V, ldv);
      else
        eig_vectors<2, NTH, HVL>(m, nw, lam, 1e-3 * tn, Y, u1, A, hvp, load_hv, bl, dots, unscale, wout, V, ldv);
    }
  };
  using Y_ = std::true_type;
  using N_ = std::false_type;
  if (keep) {
    if constexpr (!HEAD) vectors(Y_{}, buf + EIG_HV, buf);
  } else if (inlds) {
    if (load_hv) vectors(Y_{}, buf, buf + yl);
    else vectors(N_{}, buf, nullptr);
  } else {
    if (load_hv) vectors(Y_{}, wkg, buf);
    else vectors(N_{}, wkg, nullptr);
  }
}

}  // namespace

int64_t eig_scratch(int m, int nwant) {
  return (int64_t)m * m + 4LL * m + 5LL * nwant * m + cdiv((int64_t)nwant * m, 8) + 64;
}

void sym_eig_lowest(int m, int nwant, const double* S, int64_t lds, double* w, double* V, int64_t ldv,
                    double* scratch, hipStream_t s) {
  if (m < 1 || m > EIG_MAX || nwant < 1 || nwant > m || nwant > 64)
    throw Error(1, "sym_eig_lowest: need 1 <= nwant <= min(m, 64), m <= 512");
  if (nwant == m && m <= 32)
    sym_eig_block(m, S, lds, w, V, ldv, s);
  else if (m <= 64)  // half the work of a step: 88 -> 72 us, mean over m = 8, 12, .. 64 with 4 pairs
    k_sym_eig<512, 1><<<1, 512, 0, s>>>(m, nwant, S, lds, w, V, ldv, scratch);
  else if (m <= EIG_T)
    k_sym_eig<512, 2><<<1, 512, 0, s>>>(m, nwant, S, lds, w, V, ldv, scratch);
  else
    k_sym_eig<1024, 2><<<1, 1024, 0, s>>>(m, nwant, S, lds, w, V, ldv, scratch);
  SPPC_LAUNCH_CHECK();
}

}  // namespace sppc
