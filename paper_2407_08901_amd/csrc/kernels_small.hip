// kernels_small.hip - single-workgroup kernels on the small matrices of the method:
// the Cholesky factors of the block QR (eq. QR), the projected matrix T = Q^T H Q, and the
// coefficient bookkeeping of the perturbative recursion (eq. exp_seq, eq. exp_seq2).
#include "common.h"
#include "wave.h"

namespace sppc {

namespace {

// ---------------------------------------------------------------- Cholesky-QR factors
constexpr int KB = 32;

// Pivoted Cholesky of G restricted to the columns whose angle exceeds tau (one wave, LDS).
// rel > 0: a column whose Schur complement (what remains of it after the pivots taken) has fallen
// to rel times its own Gram diagonal is dropped as dependent on those pivots.  The complement of a
// Gram matrix carries rounding of about b eps times that diagonal (b <= 32), so below ~1e-14 it is
// noise; normalised, it becomes a direction that is not orthogonal to the basis the block was
// projected against (the second pass orthonormalises the block only within itself).
//
// One wave; lanes j and j + 32 hold column j (rows 0..15 and 16..31 of the updates).  The chain of b
// dependent pivots is the time, so a step stays within the wave: the pivot by DPP maxima and a ballot,
// no serial scan (b = 32: 200 us with a scan by one lane; see k_cholqr_second for the second factor).
__device__ inline double wave_max_nonneg(double v) {
  v = fmax(v, dpp_move<0x111, 0xF>(v));
  v = fmax(v, dpp_move<0x112, 0xF>(v));
  v = fmax(v, dpp_move<0x114, 0xF>(v));
  v = fmax(v, dpp_move<0x118, 0xF>(v));
  v = fmax(v, dpp_move<0x142, 0xA>(v));
  v = fmax(v, dpp_move<0x143, 0xC>(v));
  return lane_get(v, 63);
}

// W[i][j] -= l_i l_j for the column j of this lane and its half of the rows (b <= 32); l in LDS
__device__ inline void rank1_update(int b, double (*W)[KB + 1], const double* l, double lj, int j, int half) {
  const int i0 = half * 16;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int i = i0 + q;
    if (i < b && j < b) W[i][j] -= l[i] * lj;
  }
}

// Ri = R^-1 for the upper triangular R (s x s, rows in LDS): column c by lane c, back substitution.
__device__ inline void upper_inverse(int s, const double (*R)[KB + 1], double (*Ri)[KB + 1], int t) {
  if (t < s)
    for (int a = 0; a < s; ++a) Ri[a][t] = 0.0;
  wave_lds_fence();
  if (t < s) {
    Ri[t][t] = 1.0 / R[t][t];
    for (int a = s - 2; a >= 0; --a) {
      double acc = 0.0;
#pragma unroll 4
      for (int q = a + 1; q < s; ++q) acc = fma(R[a][q], Ri[q][t], acc);
      if (a < t) Ri[a][t] = -acc / R[a][a];
    }
  }
  wave_lds_fence();
}

__global__ __launch_bounds__(64) void k_cholqr_first(int b, const double* __restrict__ G,
                                                     const double* __restrict__ psi2, double tau, double rel,
                                                     double* __restrict__ M, double* __restrict__ Rfac,
                                                     double* __restrict__ angles, int* __restrict__ info) {
  __shared__ double W[KB][KB + 1];
  __shared__ double L[KB][KB + 1];   // L[s][i]: the factor's column s, entry of column i of the block
  __shared__ double R[KB][KB + 1];
  __shared__ double Ri[KB][KB + 1];
  __shared__ int perm[KB];
  const int t = threadIdx.x, j = t & 31, half = t >> 5;
  for (int e = t; e < b * b; e += 64) {
    W[e / b][e % b] = G[e];
    M[e] = 0.0;
  }
  double gd = 0.0, pn = 1.0;
  bool cand = false;
  if (j < b) {
    gd = G[j * b + j];
    pn = psi2[j] > 0.0 ? psi2[j] : 1.0;
    const double a = sqrt(fmax(gd, 0.0) / pn);
    if (t < b) angles[t] = a;
    cand = a > tau;
  }
  double wd = gd;  // the Schur complement's diagonal
  wave_lds_fence();
  int s = 0;
  while (s < b) {
    if (cand && !(wd > rel * gd)) cand = false;  // dependent on the pivots
    const double bv = wave_max_nonneg(cand && wd > 0.0 ? wd : 0.0);
    if (!(bv > 0.0)) break;
    const int best = __builtin_ctzll(__ballot(cand && wd == bv));
    if (!(bv > tau * tau * lane_get(pn, best))) break;
    const double r = sqrt(bv);
    const double lj = cand ? W[j][best] / r : 0.0;
    if (t < b) L[s][t] = lj;
    if (t == 0) perm[s] = best;
    wave_lds_fence();
    rank1_update(b, W, L[s], lj, j, half);
    wd -= lj * lj;
    if (j == best) cand = false;
    wave_lds_fence();
    ++s;
  }
  // R1[a][c] = L[a][perm[c]]
  for (int e = t; e < s * s; e += 64) {
    const int a = e / s, c = e % s;
    R[a][c] = L[a][perm[c]];
  }
  wave_lds_fence();
  upper_inverse(s, R, Ri, t);
  for (int e = t; e < s * s; e += 64) {
    const int a = e / s, c = e % s;
    M[perm[a] * b + c] = Ri[a][c];
  }
  // Rfac (b x b, rows >= s zero): Phi[:, j] ~= Phi1 Rfac[:, j]
  for (int e = t; e < b * b; e += 64) {
    const int a = e / b, c = e % b;
    Rfac[e] = (a < s) ? L[a][c] : 0.0;
  }
  if (t == 0) {
    info[0] = s;
    info[1] = 0;
  }
}

// Cholesky of G2 (s x s, leading dim b), M2 = R2^-1 (ld b), Rfac <- R2 * Rfac (s x b).  One wave, as
// k_cholqr_first without pivoting.
__global__ __launch_bounds__(64) void k_cholqr_second(int b, const double* __restrict__ G2,
                                                      double* __restrict__ M2, double* __restrict__ Rfac,
                                                      int* __restrict__ info) {
  __shared__ double W[KB][KB + 1];
  __shared__ double R[KB][KB + 1];
  __shared__ double Ri[KB][KB + 1];
  __shared__ double F[KB][KB + 1];
  const int t = threadIdx.x, j = t & 31, half = t >> 5;
  const int s = info[0];
  for (int e = t; e < s * s; e += 64) W[e / s][e % s] = G2[(e / s) * b + e % s];
  for (int e = t; e < s * b; e += 64) F[e / b][e % b] = Rfac[e];
  wave_lds_fence();
  int fail = 0;
  for (int q = 0; q < s; ++q) {
    double d = W[q][q];
    if (!(d > 0.0)) {
      fail = 1;
      d = 1e-300;
    }
    const double r = sqrt(d);
    const double lj = j < s ? (j > q ? W[q][j] / r : j == q ? r : 0.0) : 0.0;
    if (t < s) R[q][t] = lj;
    wave_lds_fence();
    rank1_update(s, W, R[q], lj, j, half);
    wave_lds_fence();
  }
  upper_inverse(s, R, Ri, t);
  for (int e = t; e < s * s; e += 64) M2[(e / s) * b + (e % s)] = Ri[e / s][e % s];
  for (int e = t; e < s * b; e += 64) {
    const int a = e / b, c = e % b;
    double acc = 0.0;
    for (int q = a; q < s; ++q) acc = fma(R[a][q], F[q][c], acc);
    Rfac[e] = acc;
  }
  if (t == 0) info[1] = fail;
}

// ---------------------------------------------------------------- T bookkeeping
__global__ void k_t_extend(int m_old, int kn, const double* __restrict__ X, int64_t ldx,
                           double* __restrict__ T, int64_t ldt) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int mt = m_old + kn;
  if (e >= (int64_t)mt * kn) return;
  const int i = (int)(e / kn), j = (int)(e % kn);
  const int cj = m_old + j;
  if (i < m_old) {
    const double v = X[(int64_t)i * ldx + j];
    T[(int64_t)i * ldt + cj] = v;
    T[(int64_t)cj * ldt + i] = v;
  } else {
    const int a = i - m_old;
    T[(int64_t)i * ldt + cj] = 0.5 * (X[(int64_t)i * ldx + j] + X[(int64_t)(m_old + j) * ldx + a]);
  }
}

__global__ void k_t_full(int m, const double* __restrict__ X, int64_t ldx, double* __restrict__ T,
                         int64_t ldt) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)m * m) return;
  const int i = (int)(e / m), j = (int)(e % m);
  T[(int64_t)i * ldt + j] = 0.5 * (X[(int64_t)i * ldx + j] + X[(int64_t)j * ldx + i]);
}

__global__ void k_t_diag(int m, const double* __restrict__ th, double* __restrict__ T, int64_t ldt) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)m * m) return;
  const int i = (int)(e / m), j = (int)(e % m);
  T[(int64_t)i * ldt + j] = i == j ? th[i] : 0.0;
}

__global__ void k_store_coef(int m_old, int kn, int k, const double* __restrict__ C, int64_t ldc,
                             const double* __restrict__ Rt, double* __restrict__ G, int64_t ldg) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)(m_old + kn) * k) return;
  const int i = (int)(e / k), j = (int)(e % k);
  G[(int64_t)i * ldg + j] = i < m_old ? C[(int64_t)i * ldc + j] : Rt[(int64_t)(i - m_old) * ldc + j];
}

// E^(p)_j = G^(p-1)[:, j]^T (T[:, j] - E0_j e_j)  (eq. exp_seq, first line: Psi^(p-1)^T V Psi^(0)
// with Psi^(l) = Q G^(l), Q^T H Psi^(0) = T[:, 0:k] and Q^T H0 Psi^(0) = E0 on the first k rows);
// A = G^(p-1), B = sum_{l=0}^{p-2} G^(l) diag(E^(p-l)), both m x k (zero-padded rows).
__global__ void k_corr_coefs(int p, int k, int m, const double* __restrict__ Gh, int64_t gstride,
                             int64_t ldg, const int* __restrict__ mh, double* __restrict__ Et,
                             const double* __restrict__ T, int64_t ldt, const double* __restrict__ E0,
                             double* __restrict__ A, double* __restrict__ B) {
  __shared__ double Ep[32];
  const int t = threadIdx.x;
  const double* Gp = Gh + (int64_t)(p - 1) * gstride;
  const int mp = mh[p - 1];
  if (t < k) {
    double s = 0.0;
#pragma unroll 8  // the sum is a chain of loads otherwise: 32 -> 13 us at k = 8, m = 128
    for (int i = 0; i < mp; ++i) s += Gp[(int64_t)i * ldg + t] * T[(int64_t)i * ldt + t];
    s -= E0[t] * Gp[(int64_t)t * ldg + t];
    Ep[t] = s;
    Et[(int64_t)p * k + t] = s;
  }
  __syncthreads();
  for (int64_t e = t; e < (int64_t)m * k; e += blockDim.x) {
    const int i = (int)(e / k), j = (int)(e % k);
    A[e] = i < mp ? Gp[(int64_t)i * ldg + j] : 0.0;
    double s = 0.0;
    for (int l = 0; l + 2 <= p; ++l) {
      const double El = (l == 0) ? Ep[j] : Et[(int64_t)(p - l) * k + j];
      if (i < mh[l]) s += El * Gh[(int64_t)l * gstride + (int64_t)i * ldg + j];
    }
    B[e] = s;
  }
}

// out[j][kk] = c[j][kk] / (w[j] - sigma_kk) for the deflated j != kk (psi_kk is projected out),
// sigma_kk = shift[kk] when given, else E_kk^(0) = w[kk]
__global__ void k_deflate_coefs(int D, int k, const double* __restrict__ w, const double* __restrict__ shift,
                                const double* __restrict__ c, int64_t ldc, double* __restrict__ out, int64_t ldo) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= D * k) return;
  const int j = e / k, kk = e % k;
  const double Ek = shift ? shift[kk] : w[kk];
  const double dj = w[j] - Ek;
  double v = 0.0;
  if (j != kk && fabs(dj) > 1e-12 * fmax(1.0, fabs(Ek))) v = c[(int64_t)j * ldc + kk] / dj;
  out[(int64_t)j * ldo + kk] = v;
}

// out[j][a] = c[j][a] / (w[j] - theta[a]) for every deflated j (shifted small-space solve)
__global__ void k_deflate_shift(int D, int na, const double* __restrict__ w, const double* __restrict__ theta,
                                const double* __restrict__ c, int64_t ldc, double* __restrict__ out,
                                int64_t ldo) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= D * na) return;
  const int j = e / na, a = e % na;
  const double th = theta[a];
  const double dj = w[j] - th;
  double v = 0.0;
  if (fabs(dj) > 1e-12 * fmax(1.0, fabs(th))) v = c[(int64_t)j * ldc + a] / dj;
  out[(int64_t)j * ldo + a] = v;
}

__global__ void k_add(int count, const double* __restrict__ a, double* __restrict__ b) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) b[e] += a[e];
}

// per-chunk max |x| (first index on ties) for each column
__global__ __launch_bounds__(256) void k_colargmax(int64_t n, int b, const double* __restrict__ X,
                                                   int64_t ldx, double* __restrict__ pv,
                                                   int64_t* __restrict__ pi) {
  __shared__ double sv[256];
  __shared__ int64_t si[256];
  const int c = blockIdx.y;
  const int64_t r0 = (int64_t)blockIdx.x * 4096;
  const int64_t r1 = min<int64_t>(n, r0 + 4096);
  double best = -1.0;
  int64_t bi = r0;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const double a = fabs(X[r * ldx + c]);
    if (a > best) { best = a; bi = r; }
  }
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < (unsigned)o) {
      const double ov = sv[threadIdx.x + o];
      const int64_t oi = si[threadIdx.x + o];
      if (ov > sv[threadIdx.x] || (ov == sv[threadIdx.x] && oi < si[threadIdx.x])) {
        sv[threadIdx.x] = ov;
        si[threadIdx.x] = oi;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    pv[(int64_t)c * gridDim.x + blockIdx.x] = sv[0];
    pi[(int64_t)c * gridDim.x + blockIdx.x] = si[0];
  }
}

__global__ void k_colsign(int64_t nch, int b, const double* __restrict__ X, int64_t ldx,
                          const double* __restrict__ pv, const int64_t* __restrict__ pi,
                          double* __restrict__ sgn) {
  const int c = threadIdx.x;
  if (c >= b) return;
  double best = -1.0;
  int64_t bi = 0;
  for (int64_t q = 0; q < nch; ++q) {
    const double v = pv[(int64_t)c * nch + q];
    const int64_t i = pi[(int64_t)c * nch + q];
    if (v > best || (v == best && i < bi)) { best = v; bi = i; }
  }
  sgn[c] = X[bi * ldx + c] < 0.0 ? -1.0 : 1.0;
}

__global__ void k_colscale(int64_t n, int b, double* __restrict__ X, int64_t ldx,
                           const double* __restrict__ sgn) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * b) return;
  const int64_t r = e / b;
  const int c = (int)(e % b);
  X[r * ldx + c] *= sgn[c];
}

__global__ void k_select_smallest(int64_t n, const double* __restrict__ d, int nsel, int* __restrict__ idx) {
  __shared__ double sv[1024];
  __shared__ int si[1024];
  // pass q takes the smallest (value, index) pair above the one taken by pass q - 1
  double pv = -INFINITY;
  int pi = -1;
  for (int q = 0; q < nsel; ++q) {
    double best = INFINITY;
    int bi = 0x7fffffff;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
      const double v = d[i];
      const bool above = v > pv || (v == pv && (int)i > pi);
      if (above && (v < best || (v == best && (int)i < bi))) { best = v; bi = (int)i; }
    }
    sv[threadIdx.x] = best;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
      if (threadIdx.x < (unsigned)o) {
        const double ov = sv[threadIdx.x + o];
        const int oi = si[threadIdx.x + o];
        if (ov < sv[threadIdx.x] || (ov == sv[threadIdx.x] && oi < si[threadIdx.x])) {
          sv[threadIdx.x] = ov;
          si[threadIdx.x] = oi;
        }
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) idx[q] = si[0];
    pv = sv[0];
    pi = si[0];
    __syncthreads();
  }
}

__global__ void k_unit_block(int64_t n, int b, const int* __restrict__ idx, double* __restrict__ X,
                             int64_t ldx) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * b) return;
  const int64_t r = e / b;
  const int c = (int)(e % b);
  X[r * ldx + c] = (r == idx[c]) ? 1.0 : 0.0;
}

inline int64_t g1(int64_t count) { return cdiv(count > 0 ? count : 1, 256); }

}  // namespace

void cholqr_first(int b, const double* G, const double* psi_sumsq, double tau, double rel, double* M,
                  double* Rfac, double* angles, int* info, hipStream_t s) {
  if (b < 1 || b > KB) throw Error(1, "cholqr: block width must be 1..32");
  k_cholqr_first<<<1, 64, 0, s>>>(b, G, psi_sumsq, tau, rel, M, Rfac, angles, info);
  SPPC_LAUNCH_CHECK();
}

void cholqr_second(int b, const double* G2, double* M2, double* Rfac, int* info, hipStream_t s) {
  k_cholqr_second<<<1, 64, 0, s>>>(b, G2, M2, Rfac, info);
  SPPC_LAUNCH_CHECK();
}

void t_extend(int m_old, int kn, const double* X, int64_t ldx, double* T, int64_t ldt, hipStream_t s) {
  k_t_extend<<<g1((int64_t)(m_old + kn) * kn), 256, 0, s>>>(m_old, kn, X, ldx, T, ldt);
  SPPC_LAUNCH_CHECK();
}

void t_from_full(int m, const double* X, int64_t ldx, double* T, int64_t ldt, hipStream_t s) {
  k_t_full<<<g1((int64_t)m * m), 256, 0, s>>>(m, X, ldx, T, ldt);
  SPPC_LAUNCH_CHECK();
}

void t_set_diag(int m, const double* theta, double* T, int64_t ldt, hipStream_t s) {
  k_t_diag<<<g1((int64_t)m * m), 256, 0, s>>>(m, theta, T, ldt);
  SPPC_LAUNCH_CHECK();
}

void store_coef(int m_old, int kn, int k, const double* C, int64_t ldc, const double* Rtot, double* G,
                int64_t ldg, hipStream_t s) {
  k_store_coef<<<g1((int64_t)(m_old + kn) * k), 256, 0, s>>>(m_old, kn, k, C, ldc, Rtot, G, ldg);
  SPPC_LAUNCH_CHECK();
}

void build_correction_coefs(int p, int k, int m, const double* Ghist, int64_t gstride, int64_t ldg,
                            const int* m_hist, double* Etab, const double* T, int64_t ldt,
                            const double* E0, double* A, double* B, hipStream_t s) {
  k_corr_coefs<<<1, 256, 0, s>>>(p, k, m, Ghist, gstride, ldg, m_hist, Etab, T, ldt, E0, A, B);
  SPPC_LAUNCH_CHECK();
}

void deflate_coefs(int D, int k, const double* w, const double* shift, const double* c, int64_t ldc, double* out,
                   int64_t ldo, hipStream_t s) {
  k_deflate_coefs<<<g1((int64_t)D * k), 256, 0, s>>>(D, k, w, shift, c, ldc, out, ldo);
  SPPC_LAUNCH_CHECK();
}

void deflate_shift(int D, int na, const double* w, const double* theta, const double* c, int64_t ldc, double* out,
                   int64_t ldo, hipStream_t s) {
  k_deflate_shift<<<g1((int64_t)D * na), 256, 0, s>>>(D, na, w, theta, c, ldc, out, ldo);
  SPPC_LAUNCH_CHECK();
}

void add_small(int count, const double* a, double* b, hipStream_t s) {
  if (count <= 0) return;
  k_add<<<g1(count), 256, 0, s>>>(count, a, b);
  SPPC_LAUNCH_CHECK();
}

void sign_fix_columns(int64_t n, int b, double* X, int64_t ldx, double* work, hipStream_t s) {
  const int64_t nch = cdiv(n > 0 ? n : 1, 4096);
  double* pv = work;
  int64_t* pi = (int64_t*)(work + nch * b);
  double* sg = work + 2 * nch * b;
  k_colargmax<<<dim3((unsigned)nch, (unsigned)b), 256, 0, s>>>(n, b, X, ldx, pv, pi);
  k_colsign<<<1, 64, 0, s>>>(nch, b, X, ldx, pv, pi, sg);
  k_colscale<<<g1(n * b), 256, 0, s>>>(n, b, X, ldx, sg);
  SPPC_LAUNCH_CHECK();
}

void select_smallest(int64_t n, const double* d, int nsel, int* idx, hipStream_t s) {
  k_select_smallest<<<1, 1024, 0, s>>>(n, d, nsel, idx);
  SPPC_LAUNCH_CHECK();
}

void unit_block(int64_t n, int b, const int* idx, double* X, int64_t ldx, hipStream_t s) {
  k_unit_block<<<g1(n * b), 256, 0, s>>>(n, b, idx, X, ldx);
  SPPC_LAUNCH_CHECK();
}

}  // namespace sppc
