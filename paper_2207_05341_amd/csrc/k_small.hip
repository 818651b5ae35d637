// The likelihood of a small state (N <= kSmallMaxQubits) in one launch: tau,
// rho = T T^dagger / tau, the product-POVM map over all qubits, the NLL
// terms, the cotangent, the adjoint map and G', by one workgroup with
// everything in LDS (T and the 4^N values: 33 KB in FP64 at N = 5).
//
// Bound by launches and latency: as seven launches of 3 to 7 us each (40 us
// at N = 4, FP64), most of it their fixed cost; here the block sums, the N
// contraction rounds each way and two passes over T are about 20 barriers.
// At N = 6 the product alone (64^3 complex multiply-adds, 8 MB of LDS reads
// by one workgroup) costs more than the launches saved.
//
// Values are indexed by interleaved digits, k = sum_i (2 r_i + c_i) 4^(N-i)
// for an entry (r, c), which is also the outcome index once every digit is
// contracted: contracting qubit i replaces its digit in place.
#include <hip/hip_runtime.h>

#include "qst_device.h"
#include "qst_kernels.h"
#include "qst_plan.h"
#include "qst_povm_ops.h"

namespace qst {

namespace {

constexpr int kMaxD = 1 << kSmallMaxQubits;
constexpr int kMaxOut = kMaxD * kMaxD;
constexpr int kPer = kMaxOut / 256;  // values per thread

__device__ __forceinline__ void row_col(int k, int n, int& r, int& c) {
  r = c = 0;
#pragma unroll
  for (int i = 0; i < kSmallMaxQubits; ++i)
    if (i < n) {
      c |= ((k >> (2 * i)) & 1) << i;
      r |= ((k >> (2 * i + 1)) & 1) << i;
    }
}

// NV sums over the workgroup, valid in every thread.
template <int NV>
__device__ __forceinline__ void block_sums(double (&v)[NV], double (*red)[4]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i] = wave_sum(v[i]);
    if ((threadIdx.x & 63) == 0) red[i][threadIdx.x >> 6] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = ((red[i][0] + red[i][1]) + red[i][2]) + red[i][3];
  __syncthreads();
}

template <typename R, bool ADJ, bool TETRA>
__device__ __forceinline__ void contract_all(Cx<R>* X, int n, const ModeMatrix& A) {
  const int groups = 1 << (2 * (n - 1));
  for (int s = 0; s < n; ++s) {
    const int sh = 2 * (ADJ ? n - 1 - s : s);
    for (int g = threadIdx.x; g < groups; g += 256) {
      const int k0 = ((g >> sh) << (sh + 2)) | (g & ((1 << sh) - 1));
      Cx<R> v[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) v[m] = X[k0 + (m << sh)];
      apply4<R, ADJ, TETRA>(v, A);
#pragma unroll
      for (int m = 0; m < 4; ++m) X[k0 + (m << sh)] = v[m];
    }
    __syncthreads();
  }
}

template <typename R, bool TETRA>
__global__ __launch_bounds__(256) void small_likelihood_kernel(int n, const Cx<R>* __restrict__ T, int64_t ldT,
                                                               const R* __restrict__ f, ModeMatrix Af, ModeMatrix Aa,
                                                               double* __restrict__ tau_out, double* __restrict__ nll,
                                                               unsigned long long* __restrict__ bad,
                                                               Cx<R>* __restrict__ G, int64_t ldG,
                                                               const R* __restrict__ pt, double* __restrict__ fc) {
  __shared__ Cx<R> Tm[kMaxD][kMaxD + 1];
  __shared__ Cx<R> X[kMaxOut];
  __shared__ double red[4][4];
  const int t = threadIdx.x, d = 1 << n, D = d * d;
  R fv[kPer];
  double s2[2] = {0.0, 0.0};  // tau, F
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = t + 256 * u;
    fv[u] = R(0);
    if (e < D) {
      const Cx<R> v = T[int64_t(e >> n) * ldT + (e & (d - 1))];
      fv[u] = f[e];
      Tm[e >> n][e & (d - 1)] = v;
      s2[0] += double(v.re) * double(v.re) + double(v.im) * double(v.im);
      s2[1] += double(fv[u]);
    }
  }
  block_sums(s2, red);  // its barriers also publish T
  const double tau = s2[0], F = s2[1], inv = 1.0 / tau;
  // rho: lower triangle, mirrored
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int k = t + 256 * u;
    int r, c;
    row_col(k, n, r, c);
    if (k >= D || r < c) continue;
    R sr = 0, si = 0;
    for (int j = 0; j < d; ++j) {
      const Cx<R> a = Tm[r][j], b = Tm[c][j];
      sr += a.re * b.re + a.im * b.im;
      si += a.im * b.re - a.re * b.im;
    }
    const Cx<R> x{R(sr * inv), R(si * inv)};
    X[k] = x;
    if (r > c) X[((k & 0x155) << 1) | ((k >> 1) & 0x155)] = Cx<R>{x.re, -x.im};  // (c, r): digits' bits swapped
  }
  __syncthreads();
  contract_all<R, false, TETRA>(X, n, Af);
  double s3[4] = {0.0, 0.0, 0.0, 0.0};  // L, f > 0 with p <= 0, NaN, F_c's sum
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int k = t + 256 * u;
    if (k >= D) continue;
    const R p = X[k].re;
    const double fk = double(fv[u]), pk = double(p);
    if (fk != 0.0) {
      if (pk > 0.0) s3[0] -= fk * ln_prob(p);
      else s3[1] += 1.0;
    }
    if (pk != pk || fk != fk) s3[2] += 1.0;
    if (pt) s3[3] += sqrt(fmax(pk, 0.0) * fmax(double(pt[k]), 0.0));
    X[k] = Cx<R>{cotangent(F, fv[u], p), R(0)};
  }
  block_sums(s3, red);  // its barriers also publish the cotangents
  if (t == 0) {
    double L = s3[0];
    if (F != F || s3[2] > 0.0) L = __builtin_nan("");
    else if (s3[1] > 0.0) L = __builtin_inf();
    *tau_out = tau;
    nll[0] = L;
    nll[1] = F;
    if (pt) *fc = s3[3] * s3[3];
    if (bad) {
      bad[0] = (unsigned long long)s3[1];
      bad[1] = (unsigned long long)s3[2];
    }
  }
  if (!G) return;
  contract_all<R, true, TETRA>(X, n, Aa);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int k = t + 256 * u;
    int r, c;
    row_col(k, n, r, c);
    if (k >= D || r < c) continue;
    const Cx<R> x = X[k];
    G[int64_t(r) * ldG + c] = x;
    if (r > c) G[int64_t(c) * ldG + r] = Cx<R>{x.re, -x.im};
  }
}

}  // namespace

hipError_t launch_small_likelihood(qst_prec prec, int n, bool tetra, const void* T, int64_t ldT, const void* f,
                                   const double* W, const double* V, double* tau_dev, double* nll_dev,
                                   unsigned long long* bad_dev, void* G, int64_t ldG, const void* pt, double* fc_dev,
                                   hipStream_t s) {
  if (n < 1 || n > kSmallMaxQubits) return hipErrorInvalidValue;
  ModeMatrix Af, Aa;
  for (int i = 0; i < 32; ++i) {
    Af.a[i] = W[i];
    Aa.a[i] = V[i];
  }
  ProfScope prof("likelihood_small", s);
#define QST_SMALL(R, TET)                                                                                            \
  small_likelihood_kernel<R, TET><<<1, 256, 0, s>>>(n, static_cast<const Cx<R>*>(T), ldT, static_cast<const R*>(f), Af, \
                                                    Aa, tau_dev, nll_dev, bad_dev, static_cast<Cx<R>*>(G), ldG,            \
                                                    static_cast<const R*>(pt), fc_dev)
  if (prec == QST_F64) {
    if (tetra) QST_SMALL(double, true);
    else QST_SMALL(double, false);
  } else {
    if (tetra) QST_SMALL(float, true);
    else QST_SMALL(float, false);
  }
#undef QST_SMALL
  return hipGetLastError();
}

}  // namespace qst
