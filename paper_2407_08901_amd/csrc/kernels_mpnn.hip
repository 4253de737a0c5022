// kernels_mpnn.hip - learned preconditioner for the continuation: a 2-layer message-passing
// network over the graph of H that corrects the diagonal (Jacobi) step for each Ritz pair.
//
//   f = [r / rms(r), (d - theta)/(1 + |theta|), lambda(level)],  g = A f,  A = H - diag(d)
//   lambda = min(max(level - n_small_levels + 1, 0), 2) / 2 (0 in the small space, 1/2 next to it, 1 beyond)
//   h = tanh(Ws f + Wn g + b1)   (32 hidden units, per row, in registers; never written to HBM)
//   o = ws.h + A (wn.h) + b2 ;   t = tJ (1 + o),  tJ = r / (d - theta) (clamped) ;  t~ = t - x (x.t)
//
// The messages g reduce to one block product per application: A (r / rms(r)) -- the other two
// feature columns are affine in theta and use A d, A 1 and A level, computed once.  Layer 2
// needs A u with u = wn.h.  Training adds one more product, A dL/do (A is symmetric).  All
// row sums over samples are deterministic per-block partials added in a fixed order.
// Parameters: Ws[32x3] | Wn[32x3] | b1[32] | ws[32] | wn[32] | b2  (289).
#include "common.h"
#include "partials.h"

namespace sppc {

namespace {

constexpr int HID = 32;
constexpr int NPAR = MPNN_NPAR;

__device__ inline double clamp_den(double den, double theta) {
  const double fl = 1e-2 * fmax(1.0, fabs(theta));
  return fabs(den) < fl ? (den >= 0.0 ? fl : -fl) : den;
}

// static per-row inputs of the network
struct Static {
  const double* d;    // diag(H)
  const double* lev;  // level / (L-1)
  const double* Ad;   // A d
  const double* A1;   // A 1
  const double* Al;   // A lev
};

// Y[r][s] = X[r][s] / scale[s], with Y32 also its float32 copy (the next product's input)
__global__ void k_scale_cols(int64_t n, int S, const double* __restrict__ X, int64_t ldx,
                             const double* __restrict__ sumsq, double* __restrict__ Y, float* __restrict__ Y32) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * S) return;
  const int64_t r = e / S;
  const int s = (int)(e % S);
  double sr = sqrt(sumsq[s] / (double)n);
  if (!(sr > 0.0)) sr = 1.0;
  const double y = X[r * ldx + s] / sr;
  Y[e] = y;
  if (Y32) Y32[e] = (float)y;
}

// layer 1 + the row parts of layer 2: u = wn.h, hs = ws.h   (HF = H fr, the full product); with u32 also the
// float32 copy of u
template <typename T>
__global__ __launch_bounds__(256) void k_mpnn_layer1(int64_t n, int S, Static st, const T* __restrict__ w,
                                                     const double* __restrict__ fr,
                                                     const double* __restrict__ HF,
                                                     const double* __restrict__ theta, double* __restrict__ u,
                                                     float* __restrict__ u32, double* __restrict__ hs) {
  __shared__ T wsh[NPAR];
  for (int i = threadIdx.x; i < NPAR; i += blockDim.x) wsh[i] = w[i];
  __syncthreads();
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * S) return;
  const int64_t r = e / S;
  const int s = (int)(e % S);
  const double th = theta[s], sth = 1.0 + fabs(th);
  const double d = st.d[r];
  const T f0 = (T)fr[e], f1 = (T)((d - th) / sth), f2 = (T)st.lev[r];
  const T g0 = (T)(HF[e] - d * fr[e]), g1 = (T)((st.Ad[r] - th * st.A1[r]) / sth), g2 = (T)st.Al[r];
  T su = 0, sh = 0;
#pragma unroll 8
  for (int j = 0; j < HID; ++j) {
    const T pre = wsh[j * 3] * f0 + wsh[j * 3 + 1] * f1 + wsh[j * 3 + 2] * f2 + wsh[96 + j * 3] * g0 +
                  wsh[96 + j * 3 + 1] * g1 + wsh[96 + j * 3 + 2] * g2 + wsh[192 + j];
    const T h = tanh(pre);
    su += wsh[256 + j] * h;
    sh += wsh[224 + j] * h;
  }
  u[e] = (double)su;
  if (u32) u32[e] = (float)su;
  hs[e] = (double)sh;
}

// t = tJ (1 + o), o = hs + (H u - d u) + b2 ; also tJ for the backward pass
template <typename T>
__global__ void k_mpnn_out(int64_t n, int S, const double* __restrict__ d, const T* __restrict__ w,
                           const double* __restrict__ R, int64_t ldr, const double* __restrict__ theta,
                           const double* __restrict__ hs, const double* __restrict__ u,
                           const double* __restrict__ Hu, double* __restrict__ t, double* __restrict__ tJ) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * S) return;
  const int64_t r = e / S;
  const int s = (int)(e % S);
  const double th = theta[s];
  const double o = hs[e] + (Hu[e] - d[r] * u[e]) + (double)w[288];
  const double tj = R[r * ldr + s] / clamp_den(d[r] - th, th);
  t[e] = tj * (1.0 + o);
  if (tJ) tJ[e] = tj;
}

// Y[r][s] = a[s] * X[r][s] + b[s] * Z[r][s]   (per-column coefficients, device)
__global__ void k_comb_cols(int64_t n, int S, const double* __restrict__ a, const double* __restrict__ X,
                            int64_t ldx, const double* __restrict__ b, const double* __restrict__ Z, int64_t ldz,
                            double* __restrict__ Y, int64_t ldy) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * S) return;
  const int64_t r = e / S;
  const int s = (int)(e % S);
  Y[r * ldy + s] = a[s] * X[r * ldx + s] + b[s] * Z[r * ldz + s];
}

// t -= x (x.t) with the dots of the columns on the device, and with f also t *= f
__global__ void k_project_x(int64_t n, int S, const double* __restrict__ xdt, const double* __restrict__ X,
                            int64_t ldx, double* __restrict__ t, const double* __restrict__ f) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * S) return;
  const int64_t r = e / S;
  const int s = (int)(e % S);
  const double v = fma(-xdt[s], X[r * ldx + s], t[e]);
  t[e] = f ? v * f[e] : v;
}

// Partials over a chunk of rows of t.e, t.t and e.e per sample, one pass over both (three passes of two
// operands each cost 110 us at n = 386k, S = 16; this one 17 us).  Column q S + s of part: dot q of sample s.
__global__ __launch_bounds__(256) void k_loss_dots(int64_t n, int S, const double* __restrict__ t,
                                                   const double* __restrict__ E, double* __restrict__ part,
                                                   int64_t chunk) {
  __shared__ double sh[3][256];
  const int i = threadIdx.x;
  const int B2 = S <= 1 ? 1 : S <= 2 ? 2 : S <= 4 ? 4 : S <= 8 ? 8 : S <= 16 ? 16 : 32;
  const int tc = i % B2, tr = i / B2, nrt = 256 / B2;
  const int64_t r0 = (int64_t)blockIdx.x * chunk;
  const int64_t r1 = min<int64_t>(n, r0 + chunk);
  double a = 0.0, b = 0.0, c = 0.0;
  if (tc < S) {
#pragma unroll 4
    for (int64_t r = r0 + tr; r < r1; r += nrt) {
      const double x = t[r * S + tc], y = E[r * S + tc];
      a = fma(x, y, a);
      b = fma(x, x, b);
      c = fma(y, y, c);
    }
  }
  sh[0][i] = a;
  sh[1][i] = b;
  sh[2][i] = c;
  __syncthreads();
  for (int o = 128; o >= B2; o >>= 1) {
    if (i < o)
#pragma unroll
      for (int q = 0; q < 3; ++q) sh[q][i] += sh[q][i + o];
    __syncthreads();
  }
  if (i < S)
#pragma unroll
    for (int q = 0; q < 3; ++q) part[((int64_t)blockIdx.x * 3 + q) * S + i] = sh[q][i];
}

// their sums (the threads of a group over the columns, the groups over the chunks, then the groups in
// order), the loss per sample and the coefficients of dL/dt~ = ca e + cb t~; one workgroup
__global__ __launch_bounds__(1024) void k_loss_coef(int64_t nch, int S, const double* __restrict__ part,
                                                    double* __restrict__ ca, double* __restrict__ cb,
                                                    double* __restrict__ lossv, double inv_scale) {
  __shared__ double sh[1024], dot[96];
  const int t = threadIdx.x, W = 3 * S, G = 1024 / W;
  double v = 0.0;
  if (t < G * W) {
#pragma unroll 8
    for (int64_t c = t / W; c < nch; c += G) v += part[c * W + t % W];
  }
  sh[t] = v;
  __syncthreads();
  if (t < W) {
    double d = 0.0;
    for (int g = 0; g < G; ++g) d += sh[g * W + t];
    dot[t] = d;
  }
  __syncthreads();
  const int s = t;
  if (s >= S) return;
  const double c1 = dot[s], c2 = dot[S + s], q = c2 * dot[2 * S + s];
  if (lossv) lossv[s] = 1.0 - c1 * c1 / q;
  ca[s] = -2.0 * c1 / q * inv_scale;
  cb[s] = 2.0 * c1 * c1 / (c2 * q) * inv_scale;
}

// Gradient partials over a run of (row, sample) items.  The values of an item that do not depend on the
// hidden unit are computed once per item, by one thread (a thread per item of a tile of 256), and go
// through LDS to the 32 threads that hold the hidden units; when each of those formed them for itself, an
// item cost 32 64-bit divisions by S and 64 float64 divisions, and the blocks of 512 items left most of the
// chip idle on small inputs.  n = 4900, S = 4: 51 -> 6.6 us; n = 386k, S = 16: 970 -> 336 us, bound by the
// issue of the ten conversions and float64 sums per item and unit.
constexpr int GT = 256;  // items per tile

template <typename T>
__global__ __launch_bounds__(GT) void k_mpnn_grad(int64_t n, int S, Static st, const T* __restrict__ w,
                                                  const double* __restrict__ fr, const double* __restrict__ HF,
                                                  const double* __restrict__ theta,
                                                  const double* __restrict__ dO, const double* __restrict__ HdO,
                                                  double* __restrict__ part, int64_t items_per_block) {
  struct alignas(16) Item {
    T v[8];  // the six inputs, dL/do, dL/du
  };
  __shared__ Item it[GT];
  __shared__ double red[8][HID][10];
  const int t = threadIdx.x, j = t & 31, slot = t >> 5;
  T ws[6];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    ws[q] = w[j * 3 + q];
    ws[3 + q] = w[96 + j * 3 + q];
  }
  const T wb = w[192 + j], wo = w[224 + j], wu = w[256 + j];
  double acc[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) acc[q] = 0.0;
  const int64_t i0 = (int64_t)blockIdx.x * items_per_block;
  const int64_t i1 = min<int64_t>(n * S, i0 + items_per_block);
  for (int64_t base = i0; base < i1; base += GT) {
    const int cnt = (int)min<int64_t>(GT, i1 - base);
    if (t < cnt) {
      const int64_t rb = base / S;
      const uint32_t x = (uint32_t)(base - rb * S) + (uint32_t)t;
      const int64_t e = base + t, r = rb + x / (uint32_t)S;
      const int s = (int)(x % (uint32_t)S);
      const double th = theta[s], sth = 1.0 + fabs(th);
      const double d = st.d[r];
      Item& o = it[t];
      o.v[0] = (T)fr[e];
      o.v[1] = (T)((d - th) / sth);
      o.v[2] = (T)st.lev[r];
      o.v[3] = (T)(HF[e] - d * fr[e]);
      o.v[4] = (T)((st.Ad[r] - th * st.A1[r]) / sth);
      o.v[5] = (T)st.Al[r];
      o.v[6] = (T)dO[e];
      o.v[7] = (T)(HdO[e] - d * dO[e]);  // dL/du = A dL/do
    }
    __syncthreads();
    for (int i = slot; i < cnt; i += 8) {
      const Item& o = it[i];
      const T f0 = o.v[0], f1 = o.v[1], f2 = o.v[2], g0 = o.v[3], g1 = o.v[4], g2 = o.v[5];
      const T dov = o.v[6], duv = o.v[7];
      const T pre = ws[0] * f0 + ws[1] * f1 + ws[2] * f2 + ws[3] * g0 + ws[4] * g1 + ws[5] * g2 + wb;
      const T h = tanh(pre);
      const T dpre = (dov * wo + duv * wu) * ((T)1 - h * h);
      acc[0] += (double)(dpre * f0);
      acc[1] += (double)(dpre * f1);
      acc[2] += (double)(dpre * f2);
      acc[3] += (double)(dpre * g0);
      acc[4] += (double)(dpre * g1);
      acc[5] += (double)(dpre * g2);
      acc[6] += (double)dpre;
      acc[7] += (double)(dov * h);
      acc[8] += (double)(duv * h);
      acc[9] += (double)dov;  // db2 (only lane 0's copy is used)
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 10; ++q) red[slot][j][q] = acc[q];
  __syncthreads();
  // part is parameter-major, so that the sums over the blocks read whole lines
  const int64_t nb = gridDim.x;
  for (int p = t; p < NPAR; p += GT) {
    int jj, q;
    if (p < 96) {
      jj = p / 3;
      q = p % 3;
    } else if (p < 192) {
      jj = (p - 96) / 3;
      q = 3 + (p - 96) % 3;
    } else if (p < 288) {
      jj = (p - 192) & 31;
      q = 6 + ((p - 192) >> 5);
    } else {
      jj = 0;
      q = 9;
    }
    double v = 0.0;
#pragma unroll
    for (int sl = 0; sl < 8; ++sl) v += red[sl][jj][q];
    part[(int64_t)p * nb + blockIdx.x] = v;
  }
}

__global__ void k_sum_parts(int64_t nb, const double* __restrict__ part, double* __restrict__ g) {
  const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= NPAR) return;
  double s = 0.0;
  for (int64_t b = lane; b < nb; b += 64) s += part[i * nb + b];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) g[i] = s;
}

// rounded to bfloat16 (nearest even) and back
__device__ inline float round_bf16(float w) {
  uint32_t bits = __float_as_uint(w);
  bits += 0x7FFFu + ((bits >> 16) & 1u);
  return __uint_as_float(bits & 0xFFFF0000u);
}

// Adam on the float32 master weights; the network uses their bfloat16 rounding
__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const double* __restrict__ g, float lr, float b1, float b2, float eps, int step,
                       float* __restrict__ wq) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= NPAR) return;
  const float gi = (float)g[i];
  m[i] = b1 * m[i] + (1.f - b1) * gi;
  v[i] = b2 * v[i] + (1.f - b2) * gi * gi;
  const float mh = m[i] / (1.f - powf(b1, (float)step));
  const float vh = v[i] / (1.f - powf(b2, (float)step));
  w[i] -= lr * mh / (sqrtf(vh) + eps);
  if (wq) wq[i] = round_bf16(w[i]);
}

__global__ void k_round_bf16(int cnt, const float* __restrict__ w, float* __restrict__ wq) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) wq[i] = round_bf16(w[i]);
}

// Weights and theta of one evaluation from the caller's pinned host copy (1.2 KB: two copies and their
// synchronisations cost more than reading it over the link), the weights rounded to bfloat16 (T = float).
template <typename T>
__global__ __launch_bounds__(320) void k_mpnn_inputs(int S, const float* __restrict__ w_host,
                                                     const double* __restrict__ th_host, T* __restrict__ w,
                                                     double* __restrict__ th) {
  const int i = threadIdx.x;
  if (i < NPAR) {
    if constexpr (sizeof(T) == 4) w[i] = round_bf16(w_host[i]);
    else w[i] = (double)w_host[i];
  }
  if (i < S) th[i] = th_host[i];
}

// static inputs: lev, and the row sums A d, A 1, A lev from full products
__global__ void k_static(int64_t n, const double* __restrict__ d, const double* __restrict__ lev,
                         const double* __restrict__ P, double* __restrict__ Ad, double* __restrict__ A1,
                         double* __restrict__ Al) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  // P = H [d, 1, lev] row-major n x 3
  Ad[r] = P[r * 3] - d[r] * d[r];
  A1[r] = P[r * 3 + 1] - d[r];
  Al[r] = P[r * 3 + 2] - d[r] * lev[r];
}

__global__ void k_pack3(int64_t n, const double* __restrict__ d, const double* __restrict__ lev,
                        double* __restrict__ P) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  P[r * 3] = d[r];
  P[r * 3 + 1] = 1.0;
  P[r * 3 + 2] = lev[r];
}

// level feature: the level counted from the small space, clipped: 0 on the small-space levels, 1/2
// on the first level outside it, 1 beyond (the same values for any number of levels)
__global__ void k_levels(int64_t n, int L, int nsmall, const int64_t* __restrict__ off, double* __restrict__ lev) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  int l = 0;
  while (l + 1 < L && off[l + 1] <= r) ++l;
  const int rel = l - nsmall + 1;
  lev[r] = 0.5 * (double)(rel < 0 ? 0 : rel > 2 ? 2 : rel);
}

__global__ void k_mul(int64_t cnt, const double* __restrict__ a, double* __restrict__ b) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < cnt) b[e] *= a[e];
}

inline int64_t gg(int64_t c) { return cdiv(c > 0 ? c : 1, 256); }

}  // namespace

int mpnn_nparam() { return NPAR; }

// Static inputs: lev[n], Ad[n], A1[n], Al[n]; tmp >= 6n doubles.
void mpnn_prepare(const DevCSR& H, const double* diag, const int64_t* level_off_dev, int L, int nsmall, double* lev,
                  double* Ad, double* A1, double* Al, double* tmp, hipStream_t s) {
  const int64_t n = H.n;
  k_levels<<<gg(n), 256, 0, s>>>(n, L, nsmall, level_off_dev, lev);
  k_pack3<<<gg(n), 256, 0, s>>>(n, diag, lev, tmp);
  spmm_f64(H, tmp, 3, tmp + 3 * n, 3, 3, nullptr, s);
  k_static<<<gg(n), 256, 0, s>>>(n, diag, lev, tmp + 3 * n, Ad, A1, Al);
  SPPC_LAUNCH_CHECK();
}

// Forward (and, with E, the loss gradient) for S samples.  R, X: n x S (leading dims ldr, ldx),
// theta_dev[S].  T_out (n x S, ld S): the projected output t~ (or nullptr).  grad_out (device,
// 289 doubles, mean over samples) and loss_dev (S doubles) when E != nullptr.
// Y := Y - Q (Q^T Y) for Y n x S (ld S) and a basis Q n x m (ld ldq) with orthonormal columns.
static void project_basis(int64_t n, int S, const MpnnBasis& B, double* Y, hipStream_t s) {
  double* C = B.work;
  double* gw = B.work + (int64_t)B.m * 32;
  for (int c0 = 0; c0 < S; c0 += 32) {
    const int bs = S - c0 < 32 ? S - c0 : 32;
    gemm_tn(n, B.m, bs, B.Q, B.ldq, Y + c0, S, C, bs, 1.0, 0.0, gw, s);
    gemm_nn(n, B.m, bs, B.Q, B.ldq, C, bs, Y + c0, S, -1.0, 1.0, s);
  }
}

int64_t mpnn_basis_work_doubles(int64_t n, int m) { return (int64_t)m * 32 + gemm_tn_work(n, m, 32); }

template <typename T>
void mpnn_run(const DevCSR& H, const double* diag, const double* lev, const double* Ad, const double* A1,
              const double* Al, const T* w, int S, const double* R, int64_t ldr, const double* X, int64_t ldx,
              const double* theta_dev, const double* E, double* T_out, double* grad_out, double* loss_dev,
              double* work, const MpnnBasis* basis, hipStream_t s, bool project) {
  const int64_t n = H.n;
  const int64_t items = n * S;
  if (!project && E) throw Error(1, "mpnn_run: the loss needs the projected output");
  double* fr = work;
  double* HF = fr + items;
  double* u = HF + items;
  double* hs = u + items;
  double* Hu = hs + items;
  double* t = Hu + items;
  double* tJ = t + items;
  double* dO = tJ + items;
  double* HdO = dO + items;
  double* sm = HdO + items;
  double* sumsq = sm;
  double* ca = sm + 64;
  double* cb = sm + 128;
  double* xdt = sm + 192;
  double* part = sm + MPNN_SMALL;
  Static st{diag, lev, Ad, A1, Al};
  // t~ is built in the caller's output where that does not overlap an operand that is still to be read
  auto apart = [&](const double* p, int64_t ld, int64_t cols) {
    const uintptr_t a0 = (uintptr_t)T_out, a1 = (uintptr_t)(T_out + items);
    return !p || (uintptr_t)(p + ((n - 1) * ld + cols)) <= a0 || (uintptr_t)p >= a1;
  };
  if (T_out && apart(R, ldr, S) && apart(X, ldx, S) && apart(E, S, S) && (!basis || apart(basis->Q, basis->ldq, basis->m)))
    t = T_out;
  // the two aggregations: with the bfloat16 weights (T = float) their products take float32 X when
  // float32 values are stored (float32 products, float64 sums; the network's inputs need no more),
  // the float32 copy of X in tJ's space, which k_mpnn_out fills only after both
  float* x32 = sizeof(T) == 4 && H.val32 ? (float*)tJ : nullptr;
  auto hprod = [&](const double* Xd, double* Yd) {
    if (x32) spmm_f32(H, x32, S, Yd, S, S, nullptr, s);
    else spmm_f64(H, Xd, S, Yd, S, S, nullptr, s);
  };
  colsumsq(n, S, R, ldr, sumsq, part, s);
  k_scale_cols<<<gg(items), 256, 0, s>>>(n, S, R, ldr, sumsq, fr, x32);
  hprod(fr, HF);
  k_mpnn_layer1<T><<<gg(items), 256, 0, s>>>(n, S, st, w, fr, HF, theta_dev, u, x32, hs);
  hprod(u, Hu);
  k_mpnn_out<T><<<gg(items), 256, 0, s>>>(n, S, diag, w, R, ldr, theta_dev, hs, u, Hu, t, tJ);
  // t~ = t - x (x.t), or t - Q (Q^T t) with a basis
  if (!project) {
    // unprojected t = tJ (1 + o) (the step of a single-vector refinement)
  } else if (basis) {
    project_basis(n, S, *basis, t, s);
  } else {
    coldots(n, S, X, ldx, t, S, xdt, part, s);
    k_project_x<<<gg(items), 256, 0, s>>>(n, S, xdt, X, ldx, t, nullptr);
  }
  if (T_out && t != T_out) copy_block(n, S, t, S, T_out, S, s);
  if (E) {
    const int64_t lch = ld_chunk(n), lnc = ld_chunks(n);
    k_loss_dots<<<lnc, 256, 0, s>>>(n, S, t, E, part, lch);
    k_loss_coef<<<1, 1024, 0, s>>>(lnc, S, part, ca, cb, loss_dev, 1.0 / S);
    // dL/dt~ = ca e + cb t~ -> dO ; then through the projection and t = tJ (1 + o)
    k_comb_cols<<<gg(items), 256, 0, s>>>(n, S, ca, E, S, cb, t, S, dO, S);
    if (basis) {
      project_basis(n, S, *basis, dO, s);
      k_mul<<<gg(items), 256, 0, s>>>(items, tJ, dO);
    } else {
      coldots(n, S, X, ldx, dO, S, xdt, part, s);
      k_project_x<<<gg(items), 256, 0, s>>>(n, S, xdt, X, ldx, dO, tJ);
    }
    spmm_f64(H, dO, S, HdO, S, S, nullptr, s);
    const int64_t ipb = grad_items(items), nblk = grad_blocks(items);
    k_mpnn_grad<T><<<nblk, GT, 0, s>>>(n, S, st, w, fr, HF, theta_dev, dO, HdO, part, ipb);
    k_sum_parts<<<cdiv(NPAR, 4), 256, 0, s>>>(nblk, part, grad_out);
  }
  SPPC_LAUNCH_CHECK();
}

template void mpnn_run<float>(const DevCSR&, const double*, const double*, const double*, const double*,
                              const double*, const float*, int, const double*, int64_t, const double*, int64_t,
                              const double*, const double*, double*, double*, double*, double*,
                              const MpnnBasis*, hipStream_t, bool);
template void mpnn_run<double>(const DevCSR&, const double*, const double*, const double*, const double*,
                               const double*, const double*, int, const double*, int64_t, const double*,
                               int64_t, const double*, const double*, double*, double*, double*, double*,
                               const MpnnBasis*, hipStream_t, bool);

void mpnn_adam(float* w, float* m, float* v, const double* g, float lr, int step, float* wq, hipStream_t s) {
  k_adam<<<cdiv(NPAR, 256), 256, 0, s>>>(w, m, v, g, lr, 0.9f, 0.999f, 1e-8f, step, wq);
  SPPC_LAUNCH_CHECK();
}

void mpnn_inputs(int S, const float* w_host, const double* th_host, float* w32, double* w64, double* th,
                 hipStream_t s) {
  if (w64) k_mpnn_inputs<double><<<1, 320, 0, s>>>(S, w_host, th_host, w64, th);
  else k_mpnn_inputs<float><<<1, 320, 0, s>>>(S, w_host, th_host, w32, th);
  SPPC_LAUNCH_CHECK();
}

void mpnn_round_bf16(int cnt, const float* w, float* wq, hipStream_t s) {
  k_round_bf16<<<cdiv(cnt, 256), 256, 0, s>>>(cnt, w, wq);
  SPPC_LAUNCH_CHECK();
}

// E = (I - Q Q^T) Psi  (n x S, ld S): the part of each exact eigenvector outside the basis.
void mpnn_target(int64_t n, int S, const MpnnBasis& B, const double* Psi, double* E, hipStream_t s) {
  const auto apart = [&](const double* p, int64_t cnt) { return p + cnt <= E || E + n * S <= p; };
  if (S <= 32 && apart(Psi, n * S) && apart(B.Q, (n - 1) * B.ldq + B.m)) {
    // E from Psi in the second pass (copying it first: 30 of 560 us at n = 1.17M, S = 8, m = 128)
    gemm_tn(n, B.m, S, B.Q, B.ldq, Psi, S, B.work, S, 1.0, 0.0, B.work + (int64_t)B.m * 32, s);
    gemm_nn_from(n, B.m, S, B.Q, B.ldq, B.work, S, Psi, S, E, S, -1.0, 1.0, s);
    return;
  }
  copy_block(n, S, Psi, S, E, S, s);
  project_basis(n, S, B, E, s);
}

}  // namespace sppc
