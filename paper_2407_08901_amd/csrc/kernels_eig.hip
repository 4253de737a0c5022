// kernels_eig.hip - lowest eigenpairs of the projected matrix T = Q^T H Q (Rayleigh-Ritz, eq. tilde_H):
// one workgroup, Householder tridiagonalisation, multisection, inverse iteration, back-transformation.
//
// T is small (m <= 512, mostly <= 128), so every phase is a chain of dependent steps and the time is
// latency: m = 64, 4 pairs 200 us, m = 128, 8 pairs 630 us before the form below.
//   tridiagonalisation  the trailing block of at most 128 rows lives in the registers of 8 waves (wave w
//                       holds rows w, w + 8, ...; lane i columns i and i + 64).  Each wave forms the
//                       Householder vector for itself, so a step has one barrier (the 8 partial sums of
//                       A v) instead of three; square root and divisions from the hardware
//                       approximations with Newton steps.
//   multisection        Sturm counts by the three-term recurrence of the leading minors, rescaled every
//                       8 steps: one dependent FMA per row instead of a division; 128 points a round.
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

// 1 / b refined by two Newton-Raphson steps; b nonzero, finite, and of ordinary size
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

// Sturm counts (eigenvalues below x) of the tridiagonal (d, sqrt(e2)) at two points: sign changes of
// the leading minors p_i = (d_i - x) p_{i-1} - e2_{i-1} p_{i-2}.  The matrix is scaled to norm < 1 and
// e2 >= 1e-60, so 8 steps neither overflow nor underflow; a minor that is exactly zero takes the sign
// opposite to its predecessor's.
template <bool ZERO>
__device__ inline double minor_step(double dd, double ee, double& p, double& pm, int& cnt) {
  double pn = fma(dd, p, -(ee * pm));
  if (ZERO && pn == 0.0) pn = p > 0.0 ? -1e-150 : 1e-150;
  cnt += (int)(((uint32_t)(__double2hiint(pn) ^ __double2hiint(p))) >> 31);
  pm = p;
  p = pn;
  return pn;
}
__device__ inline void minor_scale(double& p, double& pm) {
  const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pm)));
  p = ldexp(p, ex);
  pm = ldexp(pm, ex);
}
__device__ __forceinline__ int2 sturm_pair(int m, const double* d, const double* e2, double x0, double x1) {
  double p0 = 1.0, q0 = 0.0, p1 = 1.0, q1 = 0.0;
  int c0 = 0, c1 = 0;
  for (int i = 0; i < m; i += 8) {
    double dd[8], ee[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = min(i + u, m - 1);
      dd[u] = d[r];
      ee[u] = r > 0 ? e2[r - 1] : 0.0;
    }
    const double sp0 = p0, sq0 = q0, sp1 = p1, sq1 = q1;
    const int sc0 = c0, sc1 = c1;
    bool zero = false;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (i + u < m) {
        zero |= minor_step<false>(dd[u] - x0, ee[u], p0, q0, c0) == 0.0;
        zero |= minor_step<false>(dd[u] - x1, ee[u], p1, q1, c1) == 0.0;
      }
    }
    if (zero) {
      p0 = sp0, q0 = sq0, p1 = sp1, q1 = sq1;
      c0 = sc0, c1 = sc1;
      for (int u = 0; u < 8; ++u) {
        if (i + u < m) {
          minor_step<true>(dd[u] - x0, ee[u], p0, q0, c0);
          minor_step<true>(dd[u] - x1, ee[u], p1, q1, c1);
        }
      }
    }
    minor_scale(p0, q0);
    minor_scale(p1, q1);
  }
  return make_int2(c0, c1);
}

// Two solves (Tri - lam I) y = y by Gaussian elimination with partial pivoting, from a random start
// (the shift is the eigenvalue to a few ulp: two suffice).  Row k of this vector: index k * nw of the
// arrays; r0 = 1 / u0, u2 = e[k + 1] where the rows were interchanged.
__device__ __forceinline__ void inverse_iteration(int m, int nw, const double* d, const double* e, double lam, double epsp,
                                  uint32_t seed, double* __restrict__ u1, double* __restrict__ l,
                                  double* __restrict__ r0, double* __restrict__ y, unsigned char* __restrict__ piv) {
  uint32_t h = seed;
  auto start = [&]() {
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    return 0.5 + (double)(h & 0xFFFFFF) / (double)0x1000000;
  };
  auto away = [&](double a) { return fabs(a) < epsp ? (a >= 0.0 ? epsp : -epsp) : a; };
  double ca = d[0] - lam, cb = m > 1 ? e[0] : 0.0, cur = start();
#pragma unroll 4
  for (int k = 0; k < m - 1; ++k) {
    const double sub = e[k], na = d[k + 1] - lam, nb = k + 2 < m ? e[k + 1] : 0.0, yn = start();
    const bool sw = fabs(ca) < fabs(sub);
    const double pv = away(sw ? sub : ca);
    double r = __builtin_amdgcn_rcp(pv);
    r = fma(r, fma(-pv, r, 1.0), r);
    const double mult = (sw ? ca : sub) * r;
    const double a1 = sw ? na : cb;
    const double yk = sw ? yn : cur;
    cur = fma(-mult, yk, sw ? cur : yn);
    ca = fma(-mult, a1, sw ? cb : na);
    cb = sw ? -mult * nb : nb;
    u1[k * nw] = a1;
    l[k * nw] = mult;
    r0[k * nw] = r;
    y[k * nw] = yk;
    piv[k * nw] = sw;
  }
  const double rl = fast_rcp(away(ca));
  for (int it = 0; it < 2; ++it) {
    if (it == 1) {
      cur = y[0];
#pragma unroll 4
      for (int k = 0; k < m - 1; ++k) {
        const double yn = y[(k + 1) * nw], mult = l[k * nw];
        const bool sw = piv[k * nw];
        const double yk = sw ? yn : cur;
        cur = fma(-mult, yk, sw ? cur : yn);
        y[k * nw] = yk;
      }
    }
    double y1 = cur * rl, y2 = 0.0;
    y[(m - 1) * nw] = y1;
#pragma unroll 4
    for (int k = m - 2; k >= 0; --k) {
      const double a2 = k + 2 < m && piv[k * nw] ? e[k + 1] : 0.0;
      const double v = fma(-u1[k * nw], y1, fma(-a2, y2, y[k * nw])) * r0[k * nw];
      y2 = y1;
      y1 = v;
      y[k * nw] = v;
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
    for (int j = m - 3; j >= 0; --j) {
      const double b = bl[j];
      // entry j + 1 of v_j: index (a sum that stays non-negative in every part)
      const int v0 = HVL ? j * (m - 1) - j * (j - 1) / 2 : j * m + j + 1;
      double x[NR], s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = ln + 64 * q;
        x[q] = 0.0;
        if (i > j && i < m) x[q] = HVL ? hv[v0 + (i - j - 1)] : A[v0 + (i - j - 1)];
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

// NTH = 512: m <= 128, all in registers and LDS.  NTH = 1024: the leading rows of a larger T are
// reduced in global memory by all 16 waves until the trailing block fits.
// scratch (doubles): A[m*m] | d[m] | e[m] | beta[m] | work of the inverse iteration when LDS is short
template <int NTH>
__global__ __launch_bounds__(NTH) void k_sym_eig(int m, int nw, const double* __restrict__ S, int64_t lds,
                                                 double* __restrict__ wout, double* __restrict__ V, int64_t ldv,
                                                 double* __restrict__ scr) {
  constexpr bool HEAD = NTH > 512;
  constexpr int LDV = HEAD ? EIG_MAX : EIG_T;
  __shared__ double buf[EIG_BUF];
  __shared__ double vec[(HEAD ? 7 : 6) * LDV];
  __shared__ double sc;
  const int t = threadIdx.x, w = t >> 6, ln = t & 63;
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

  // ---- the trailing block, rows o.. of T, in the registers of waves 0..7
  const int L = m - o;
  double* const hv = buf;                   // packed v_j, j = 0..L-3
  double* const pp = buf + EIG_HV;          // [2][8][128] partial sums of A v by step parity
  double* const rowb = pp + 2 * 8 * EIG_T;  // [2][128] the next row, by step parity
  double* const own = rowb + 2 * EIG_T;     // [8][3][16] per wave: v, v', w at its own rows
  double a[16][2], u[2] = {0.0, 0.0}, wr[2] = {0.0, 0.0};
  if (w < 8) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int l = w + 8 * r, i = ln + 64 * c;
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
      rowb[64 + ln] = a[0][1];
    }
    double* ow = own + w * 48;
    if (ln < 48) ow[ln] = 0.0;
  }
  __syncthreads();
  if constexpr (HEAD) {
    for (int i = t; i < o; i += NTH) {
      dl[i] = dg[i];
      el[i] = eg[i];
      bl[i] = bg[i];
    }
  }
  const bool two = L > 64;
  for (int j = 0; j + 2 < L; ++j) {
    double v[2] = {0.0, 0.0}, b = 0.0;
    if (w < 8) {
      const double* rb = rowb + (j & 1) * EIG_T;
      const double uj = lane_get(j < 64 ? u[0] : u[1], j & 63), wj = lane_get(j < 64 ? wr[0] : wr[1], j & 63);
      double x[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) x[c] = rb[ln + 64 * c] - (uj * wr[c] + wj * u[c]);
      double sg = 0.0;
      if (ln > j + 1) sg = x[0] * x[0];
      if (two && ln + 64 > j + 1) sg = fma(x[1], x[1], sg);
      sg = wave_sum(sg);
      const double alpha = lane_get(j + 1 < 64 ? x[0] : x[1], (j + 1) & 63);
      double e, rv;
      reflector(alpha, sg, e, b, rv);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
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
      if (w == (j & 7)) {
        double* dst = hv + j * (L - 1) - j * (j - 1) / 2 - (j + 1);
        if (ln > j && ln < L) dst[ln] = v[0];
        if (two && ln + 64 > j && ln + 64 < L) dst[ln + 64] = v[1];
      }
      double* ow = own + w * 48;
      double* const ov = ow + 16 * (j & 1);
      const double* const ou = ow + 16 * ((j & 1) ^ 1);
      const double* const owr = ow + 32;
      if ((ln & 7) == w) {
        ov[ln >> 3] = v[0];
        ov[8 + (ln >> 3)] = v[1];
      }
      wave_lds_fence();
      // apply the pending update of step j - 1 to the rows below j and form this wave's part of A v
      double s0 = 0.0, s1 = 0.0;
      double* nrow = rowb + ((j + 1) & 1) * EIG_T;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int l = w + 8 * r;
        if (l > j && l < L) {
          const double ul = ou[r], wl = owr[r], vl = ov[r];
          a[r][0] -= ul * wr[0] + wl * u[0];
          s0 = fma(a[r][0], vl, s0);
          if (two) {
            a[r][1] -= ul * wr[1] + wl * u[1];
            s1 = fma(a[r][1], vl, s1);
          }
          if (l == j + 1) {
            nrow[ln] = a[r][0];
            nrow[64 + ln] = a[r][1];
          }
        }
      }
      double* pj = pp + ((j & 1) * 8 + w) * EIG_T;
      pj[ln] = s0;
      if (two) pj[64 + ln] = s1;
    }
    __syncthreads();
    if (w < 8) {
      const double* pj = pp + (j & 1) * 8 * EIG_T;
      double p[2] = {0.0, 0.0};
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        p[0] += pj[g * EIG_T + ln];
        if (two) p[1] += pj[g * EIG_T + 64 + ln];
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) p[c] = ln + 64 * c > j && ln + 64 * c < L ? p[c] * b : 0.0;
      const double K = 0.5 * b * wave_sum(fma(p[0], v[0], p[1] * v[1]));
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        wr[c] = fma(-K, v[c], p[c]);
        u[c] = v[c];
      }
      double* owr = own + w * 48 + 32;
      if ((ln & 7) == w) {
        owr[ln >> 3] = wr[0];
        owr[8 + (ln >> 3)] = wr[1];
      }
      wave_lds_fence();
    }
  }
  // the last two rows, with the pending update of the last step
  if (w < 8) {
    if (w == 0 && L >= 2) {
      const int j = L - 2;
      const double* rb = rowb + (j & 1) * EIG_T;
      const double uj = lane_get(j < 64 ? u[0] : u[1], j & 63), wj = lane_get(j < 64 ? wr[0] : wr[1], j & 63);
      const double x0 = rb[ln] - (uj * wr[0] + wj * u[0]), x1 = rb[64 + ln] - (uj * wr[1] + wj * u[1]);
      const double dj = lane_get(j < 64 ? x0 : x1, j & 63), ej = lane_get(j + 1 < 64 ? x0 : x1, (j + 1) & 63);
      if (ln == 0) {
        dl[o + j] = dj;
        el[o + j] = ej;
        bl[o + j] = 0.0;
      }
    }
    if (w == ((L - 1) & 7)) {
      double x = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (w + 8 * r == L - 1) x = L - 1 < 64 ? a[r][0] - 2.0 * u[0] * wr[0] : a[r][1] - 2.0 * u[1] * wr[1];
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
  for (int i = t; i < m; i += NTH) {
    const double e = ldexp(el[i], -ex);
    dl[i] = ldexp(dl[i], -ex);
    el[i] = e;
    e2l[i] = fmax(e * e, 1e-60);
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
  // at 128 interior points of the current interval, which shrinks 129-fold (counts are monotone in x,
  // so the crossing is found by ballots)
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
        const double h = (x1 - x0) / 129.0;
        const double xa = x0 + (2 * ln + 1) * h, xb = x0 + (2 * ln + 2) * h;
        const int2 cnt = sturm_pair(m, dl, e2l, xa, xb);
        // the lowest P points have count <= idx (monotone); the eigenvalue lies between points P and P + 1
        const int P = __popcll(__ballot(xa < x1 && cnt.x <= idx)) + __popcll(__ballot(xb < x1 && cnt.y <= idx));
        const double na = P > 0 ? x0 + P * h : x0;
        const double nb = P < 128 ? x0 + (P + 1) * h : x1;
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
      inverse_iteration(m, nw, dl, el, lam[t] + 10.0 * epsp * rep, epsp, 0x9E3779B9u * (uint32_t)(t + 1), u1 + t,
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
  else if (m <= EIG_T)
    k_sym_eig<512><<<1, 512, 0, s>>>(m, nwant, S, lds, w, V, ldv, scratch);
  else
    k_sym_eig<1024><<<1, 1024, 0, s>>>(m, nwant, S, lds, w, V, ldv, scratch);
  SPPC_LAUNCH_CHECK();
}

}  // namespace sppc
