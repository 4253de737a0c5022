// kernels_eigblock.hip - every eigenpair of the Rayleigh-Ritz matrix of the small space's block iteration
// (m <= 32 columns, eq. EP_small): one workgroup, all in LDS.
//
// Apart from kernels_eig.hip on purpose.  The block iteration stops its deflation-only pairs at a
// residual of 1e-9 in the mixed form, and what is left of their error follows the rounding of every step
// of the iteration (its filtered columns are nearly parallel): another rounding here moves the vectors
// of a mixed solve by up to 1e-8 (n = 1.17M, k = 8), ten times what the order of the products' sums does.
// So this solver keeps its order of operations; 4 waves (one per SIMD) instead of 16 shorten its barriers.
#include "common.h"
#include "wave.h"

namespace sppc {

namespace {

constexpr int EB = 32;            // columns at most
constexpr int EB_THREADS = 256;   // column i = t % 32, row group t / 32 (8 groups)

// a / b from the hardware reciprocal refined by one Newton-Raphson step, a few ulp from the
// rounded quotient: the Sturm counts and the shifted solves of inverse iteration sit on long
// chains of dependent divisions and do not need the correctly rounded one.  b is nonzero and
// finite at every call (both callers clamp their pivots away from zero); below 1e-290 the
// reciprocal could overflow, and the plain division is taken.
__device__ inline double quick_div(double a, double b) {
  if (fabs(b) < 1e-290) return a / b;
  double r = __builtin_amdgcn_rcp(b);
  r = fma(r, fma(-b, r, 1.0), r);
  return a * r;
}

// Sturm count: number of eigenvalues of the tridiagonal (d, e) smaller than x.  The pivots are
// kept at least 1e-290 in magnitude, so the reciprocal needs no guard.
__device__ inline double rcp_div(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(r, fma(-b, r, 1.0), r);
  return a * r;
}
__device__ int sturm_count(int m, const double* d, const double* e2, double x, double pivmin) {
  pivmin = fmax(pivmin, 1e-290);
  int cnt = 0;
  double q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  cnt += q < 0.0;
  int i = 1;
  // the operands of 8 steps are loaded ahead of the dependent chain
  for (; i + 8 <= m; i += 8) {
    double dd[8], ee[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      dd[u] = d[i + u] - x;
      ee[u] = e2[i + u - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      q = dd[u] - rcp_div(ee[u], q);
      if (fabs(q) < pivmin) q = -pivmin;
      cnt += q < 0.0;
    }
  }
  for (; i < m; ++i) {
    q = d[i] - x - rcp_div(e2[i - 1], q);
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
  }
  return cnt;
}

// Solve (Tri - lam I) y = y in place by Gaussian elimination with partial pivoting on the
// tridiagonal (two superdiagonals appear after interchanges).  Work arrays u0,u1,u2,l [m], piv [m].
__device__ void tri_shifted_solve(int m, const double* d, const double* e, double lam, double epsp,
                                  double* u0, double* u1, double* u2, double* l, unsigned char* piv,
                                  double* y, bool factor) {
  if (factor) {
    double ca = d[0] - lam;
    double cb = m > 1 ? e[0] : 0.0;
    for (int k = 0; k < m - 1; ++k) {
      const double sub = e[k];
      const double na = d[k + 1] - lam;
      const double nb = (k + 1 < m - 1) ? e[k + 1] : 0.0;
      if (fabs(ca) >= fabs(sub)) {
        if (ca == 0.0) ca = epsp;
        const double mult = quick_div(sub, ca);
        u0[k] = ca; u1[k] = cb; u2[k] = 0.0; l[k] = mult; piv[k] = 0;
        ca = na - mult * cb;
        cb = nb;
      } else {
        const double mult = quick_div(ca, sub);
        u0[k] = sub; u1[k] = na; u2[k] = nb; l[k] = mult; piv[k] = 1;
        ca = cb - mult * na;
        cb = -mult * nb;
      }
    }
    if (fabs(ca) < epsp) ca = ca >= 0.0 ? epsp : -epsp;
    u0[m - 1] = ca;
    for (int k = 0; k < m - 1; ++k)
      if (fabs(u0[k]) < epsp) u0[k] = u0[k] >= 0.0 ? epsp : -epsp;
  }
  for (int k = 0; k < m - 1; ++k) {
    if (piv[k]) {
      const double t = y[k];
      y[k] = y[k + 1];
      y[k + 1] = t;
    }
    y[k + 1] -= l[k] * y[k];
  }
  y[m - 1] = quick_div(y[m - 1], u0[m - 1]);
  if (m >= 2) y[m - 2] = quick_div(y[m - 2] - u1[m - 2] * y[m - 1], u0[m - 2]);
  for (int k = m - 3; k >= 0; --k) y[k] = quick_div(y[k] - u1[k] * y[k + 1] - u2[k] * y[k + 2], u0[k]);
}

__device__ void normalize(int m, double* y) {
  double s = 0.0, mx = 0.0;
  for (int i = 0; i < m; ++i) mx = fmax(mx, fabs(y[i]));
  if (mx == 0.0) return;
  const double rmx = 1.0 / mx;
  for (int i = 0; i < m; ++i) { y[i] *= rmx; s += y[i] * y[i]; }
  s = 1.0 / sqrt(s);
  for (int i = 0; i < m; ++i) y[i] *= s;
}


__global__ __launch_bounds__(EB_THREADS) void k_sym_eig_block(int m, const double* __restrict__ S, int64_t lds,
                                                              double* __restrict__ wout, double* __restrict__ V,
                                                              int64_t ldv) {
  __shared__ double vsh[EB], vsh2[EB], wsh[EB], pp[8 * EB];
  __shared__ double A[EB * EB], hv[EB * EB];
  __shared__ double d[EB], e[EB], e2[EB], beta[EB];
  __shared__ double Y[EB * EB], u0[EB * EB], u1[EB * EB], u2[EB * EB], lm[EB * EB];
  __shared__ unsigned char piv[EB * EB];
  __shared__ double sc[4];
  const int t = threadIdx.x;
  const int wv = t >> 6, ln = t & 63;
  const int nw = m;
  for (int q = t; q < m * m; q += EB_THREADS) A[(q / m) * EB + q % m] = S[(int64_t)(q / m) * lds + q % m];
  __syncthreads();

  // ---- Householder tridiagonalisation (the lower part; A stays symmetric).  The rank-2 update of step
  // j - 1 is applied in step j: to row j as it forms its vector, and to the rest of the trailing block
  // in the pass that forms A v.  up/wsh hold v and w of step j - 1 (index 0 = row j).
  bool pend = false;
  for (int j = 0; j + 2 < m; ++j) {
    double* const vc = (j & 1) ? vsh2 : vsh;
    const double* const up = (j & 1) ? vsh : vsh2;
    const int len = m - 1 - j;
    const double* xr = A + j * EB + j + 1;
    if (t < 64) {
      const double u0 = pend ? up[0] : 0.0, w0 = pend ? wsh[0] : 0.0;
      double part = 0.0;
      for (int i = 1 + t; i < len; i += 64) {
        const double x = xr[i] - (u0 * wsh[1 + i] + w0 * up[1 + i]);
        part += x * x;
      }
      part = wave_sum(part);
      const double sigma = part;
      const double alpha = xr[0] - (u0 * wsh[1] + w0 * up[1]);
      double b = 0.0, v0 = 1.0, ej = alpha;
      if (sigma > 0.0) {
        const double mu = sqrt(alpha * alpha + sigma);
        v0 = alpha <= 0.0 ? alpha - mu : -sigma / (alpha + mu);
        b = 2.0 * v0 * v0 / (sigma + v0 * v0);
        ej = mu;
      }
      if (t == 0) {
        d[j] = A[j * EB + j] - 2.0 * u0 * w0;
        e[j] = ej;
        beta[j] = b;
        sc[0] = b;
      }
      const double rv0 = 1.0 / v0;
      for (int i = t; i < len; i += 64) {
        const double x = i == 0 ? alpha : xr[i] - (u0 * wsh[1 + i] + w0 * up[1 + i]);
        vc[i] = i == 0 ? 1.0 : (b == 0.0 ? 0.0 : x * rv0);
      }
    }
    __syncthreads();
    const double b = sc[0];
    for (int i = t; i < len; i += EB_THREADS) hv[j * EB + i] = vc[i];  // for the back-transformation
    {
      const int i = t & 31, lg = t >> 5;
      double* ci = A + (j + 1) * EB + (j + 1) + i;
      if (i < len) {
        double s0 = 0.0;
        if (pend) {
          const double ui = up[1 + i], wi = wsh[1 + i];
          for (int l = lg; l < len; l += 8) {
            const double a0 = ci[l * EB] - (up[1 + l] * wi + wsh[1 + l] * ui);
            ci[l * EB] = a0;
            s0 += a0 * vc[l];
          }
        } else {
          for (int l = lg; l < len; l += 8) s0 += ci[l * EB] * vc[l];
        }
        pp[lg * EB + i] = s0;
      }
    }
    __syncthreads();  // every read of the previous step's w is done
    if (t < 64) {
      double kp = 0.0;
      for (int i2 = t; i2 < len; i2 += 64) {
        double pi = 0.0;
#pragma unroll
        for (int g8 = 0; g8 < 8; ++g8) pi += pp[g8 * EB + i2];
        pi *= b;
        wsh[i2] = pi;
        kp += pi * vc[i2];
      }
      kp = wave_sum(kp);
      const double K = 0.5 * b * kp;
      for (int i2 = t; i2 < len; i2 += 64) wsh[i2] -= K * vc[i2];
    }
    pend = true;
    __syncthreads();
  }
  if (t == 0) {
    // the last 2 x 2 block, with the pending update of the last step (index 0 = row m - 2)
    const double* lb = A + (m >= 2 ? m - 2 : 0) * EB + (m >= 2 ? m - 2 : 0);
    if (m >= 2) {
      const double* vl = ((m - 3) & 1) ? vsh2 : vsh;
      const double v0 = pend ? vl[0] : 0.0, v1 = pend ? vl[1] : 0.0;
      const double w0 = pend ? wsh[0] : 0.0, w1 = pend ? wsh[1] : 0.0;
      d[m - 2] = lb[0] - 2.0 * v0 * w0;
      d[m - 1] = lb[EB + 1] - 2.0 * v1 * w1;
      e[m - 2] = lb[EB] - (v1 * w0 + w1 * v0);
      beta[m - 2] = 0.0;
    } else {
      d[0] = lb[0];
    }
    e[m - 1] = 0.0;
    beta[m - 1] = 0.0;
    double tn = 0.0;
    for (int i = 0; i < m; ++i)
      tn = fmax(tn, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i < m - 1 ? fabs(e[i]) : 0.0));
    sc[2] = fmax(tn, 1e-300);
  }
  __syncthreads();
  for (int i = t; i < m; i += EB_THREADS) e2[i] = e[i] * e[i];
  __syncthreads();
  const double tn = sc[2];

  // ---- eigenvalues by multisection: one wave per eigenvalue; in each round the 64 lanes evaluate the
  // Sturm count at 64 interior points of the current interval, which shrinks 65-fold (counts are
  // monotone in x, so the crossing is found by a ballot).
  {
    double lo = d[0], hi = d[0], maxe2 = 0.0;
    for (int i = 0; i < m; ++i) {
      const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i < m - 1 ? fabs(e[i]) : 0.0);
      lo = fmin(lo, d[i] - r);
      hi = fmax(hi, d[i] + r);
      if (i < m - 1) maxe2 = fmax(maxe2, e2[i]);
    }
    const double pivmin = 2.2250738585072014e-308 * fmax(1.0, maxe2);
    for (int idx = wv; idx < nw; idx += EB_THREADS / 64) {
      double a = lo - 1e-14 * tn - 1e-300, bb = hi + 1e-14 * tn + 1e-300;
      for (int it = 0; it < 40; ++it) {
        if (bb - a <= 2.220446049250313e-16 * fmax(fabs(a), fabs(bb)) + pivmin) break;
        const double h = (bb - a) / 65.0;
        const double x = a + (ln + 1) * h;
        const bool le = x < bb && sturm_count(m, d, e2, x, pivmin) <= idx;
        const unsigned long long bal = __ballot(le);
        // lanes 0..L-1 have count <= idx (monotone); the eigenvalue lies in [x_{L-1}, x_L]
        const int L = __popcll(bal);
        const double na = L > 0 ? a + L * h : a;
        const double nbv = L < 64 ? a + (L + 1) * h : bb;
        if (!(na < nbv) || (na == a && nbv == bb)) break;
        a = na;
        bb = fmin(nbv, bb);
      }
      if (ln == 0) wsh[idx] = 0.5 * (a + bb);
    }
  }
  __syncthreads();

  // ---- eigenvectors of the tridiagonal by inverse iteration, one thread per vector
  const double epsp = 2.220446049250313e-16 * tn;
  if (t < nw) {
    double* y = Y + t * m;
    double lam = wsh[t];
    // repeated eigenvalues: separate the shifts slightly so the vectors differ
    int rep = 0;
    for (int c2 = t - 1; c2 >= 0 && wsh[t] - wsh[c2] < 10.0 * epsp; --c2) ++rep;
    lam += 10.0 * epsp * rep;
    uint32_t h = 0x9E3779B9u * (uint32_t)(t + 1);
    for (int i = 0; i < m; ++i) {
      h ^= h << 13; h ^= h >> 17; h ^= h << 5;
      y[i] = 0.5 + (double)(h & 0xFFFFFF) / (double)0x1000000;
    }
    for (int it = 0; it < 2; ++it) {  // the shift is the eigenvalue to a few ulp: two solves suffice
      tri_shifted_solve(m, d, e, lam, epsp, u0 + t * m, u1 + t * m, u2 + t * m, lm + t * m, piv + t * m, y, it == 0);
      normalize(m, y);
    }
  }
  __syncthreads();
  // vectors of close eigenvalues: classical Gram-Schmidt twice against the earlier members of their
  // cluster (dots by all waves, the update by wave 0)
  {
    const double ctol = 1e-3 * tn;
    for (int c = 1; c < nw; ++c) {
      int c0 = c;
      while (c0 > 0 && wsh[c0] - wsh[c0 - 1] <= ctol) --c0;
      if (c0 == c) continue;  // uniform across the block
      double* y = Y + c * m;
      for (int pass = 0; pass < 2; ++pass) {
        for (int c2 = c0 + wv; c2 < c; c2 += EB_THREADS / 64) {
          const double* y2 = Y + c2 * m;
          double sdot = 0.0;
          for (int i = ln; i < m; i += 64) sdot += y[i] * y2[i];
          for (int o = 32; o > 0; o >>= 1) sdot += __shfl_xor(sdot, o);
          if (ln == 0) vsh[c2] = sdot;
        }
        __syncthreads();
        if (wv == 0) {
          double v = 0.0, part = 0.0;
          if (ln < m) {
            v = y[ln];
            for (int c2 = c0; c2 < c; ++c2) v -= vsh[c2] * Y[c2 * m + ln];
            part += v * v;
          }
          for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
          const double nrm = sqrt(part);
          if (ln < m) y[ln] = nrm > 0.0 ? v / nrm : 0.0;
        }
        __syncthreads();
      }
    }
  }

  // ---- back-transformation V = H_0 H_1 ... H_{m-3} Y, one wave per column (entry ln in lane ln)
  for (int c = wv; c < nw; c += EB_THREADS / 64) {
    double y = ln < m ? Y[c * m + ln] : 0.0;
    for (int j = m - 3; j >= 0; --j) {
      const double b = beta[j];
      if (b == 0.0) continue;
      const bool in = ln > j && ln < m;
      const double v = in ? hv[j * EB + (ln - j - 1)] : 0.0;
      // (0 + v y: a bare product would be contracted into the first addition of the wave's sum)
      const double s = wave_sum(fma(v, y, 0.0)) * b;
      if (in) y -= s * v;
    }
    // sign convention (largest-magnitude entry positive) and output
    double best = ln < m ? fabs(y) : -1.0, val = y;
    int bi = ln;
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
    if (ln < m) V[(int64_t)ln * ldv + c] = sgn * y;
    if (ln == 0) wout[c] = wsh[c];
  }
}

}  // namespace

void sym_eig_block(int m, const double* S, int64_t lds, double* w, double* V, int64_t ldv, hipStream_t s) {
  if (m < 1 || m > EB) throw Error(1, "sym_eig_block: need 1 <= m <= 32");
  k_sym_eig_block<<<1, EB_THREADS, 0, s>>>(m, S, lds, w, V, ldv);
  SPPC_LAUNCH_CHECK();
}

}  // namespace sppc
