// Direct Hermitian eigensolver (FP64) behind the P-order absolute map of
// Sec. 3.2 (Eq. abs_P) and the general fidelity (Eq. F_QF through one
// eigendecomposition, as Eq. fq_decom does).
//
// H = Q T Q^dagger with T real symmetric tridiagonal (Householder), then
// T = Z Lambda Z^T, and the eigenvectors of H are the columns of Q Z:
//
// 1. Reduction.  Step k forms the reflector I - tau_k v_k v_k^dagger that
//    maps column k below the diagonal onto beta_k e_1 (beta_k real, so T is
//    real), and the Hermitian rank-2 update of the trailing matrix,
//    A22 -= v w^dagger + w v^dagger with w = tau A22 v + alpha v,
//    alpha = -|tau|^2 (v^dagger A22 v) / 2.  One launch per column: step k
//    applies the update of step k-1 on the fly to row k (which every
//    workgroup reads: row k holds column k conjugated, H being Hermitian),
//    forms reflector k from it (redundantly in every workgroup, identically
//    since the data and the order are the same), and then updates its own
//    rows of the trailing matrix while forming their entries of A22 v_k.
//    The trailing matrix is thus read and written once per column.
// 2. Splitting.  Off-diagonal entries below 4 eps sqrt(d) ||T|| are set to
//    zero (a perturbation of the size of the reduction's own rounding); the
//    unreduced blocks are then independent.
// 3. Eigenvalues by multisection: a wave per eigenvalue evaluates the Sturm
//    count (sign changes of the leading minors of T - x I) of its block at 64
//    points of the current interval and keeps the sub-interval that holds
//    the eigenvalue: about 6 bits per round, full precision in 9 or 10.
// 4. Eigenvectors by twisted factorizations, two threads per eigenvalue:
//    T - lambda I = L+ D+ L+^T (top down) = U- D- U-^T (bottom up); the twist
//    index r minimises |gamma_k| = |D+_k + D-_k - (a_k - lambda)|, and the
//    vector follows from z_r = 1 by z_k = -L+_k z_{k+1} above r and
//    z_{k+1} = -U-_k z_k below it.
// 5. Clusters (eigenvalues of a block closer than 1e-7 ||T||): inverse
//    iteration with Gaussian elimination with partial pivoting on
//    T - sigma I, each member orthogonalised against the members before it
//    (the classical treatment of clusters), one workgroup per cluster.
// 6. One Newton-Schulz step Z <- Z (3 I - Z^T Z) / 2 restores orthogonality
//    to rounding level (the twisted vectors of eigenvalues with a relative
//    gap g are orthogonal to about eps / g).
// 7. Back-transformation Q Z with the reflectors in blocks of 64 in the
//    compact form I - V T_B V^dagger (T_B upper triangular from the Gram
//    matrix of the block's reflectors, W_B = V T_B formed once), applied
//    from the last block to the first: X = V^dagger Z (row-chunk partial
//    sums, then their sum), Z -= W_B X.
//
// The eigenvalues of every block come out in ascending order; across blocks
// there is no particular order.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <cstddef>

#include "qst_device.h"
#include "qst_kernels.h"

namespace qst {

namespace {

using C64 = Cx<double>;

__device__ __forceinline__ C64 cmul(C64 a, C64 b) { return C64{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
// conj(a) * b
__device__ __forceinline__ C64 cmulc(C64 a, C64 b) { return C64{a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re}; }
__device__ __forceinline__ C64 conjg(C64 a) { return C64{a.re, -a.im}; }

constexpr double kEps = DBL_EPSILON;
constexpr double kClusterTol = 1e-7;  // relative gap below which eigenvalues form a cluster

// Sum over a workgroup of NW waves, the result returned to every thread.
template <int NW>
__device__ __forceinline__ double block_sum_allN(double v, double* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) s += red[w];
  return s;
}

__device__ __forceinline__ double wave_max(double v) {
  return wave_fold(v, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ double wave_min(double v) {
  return wave_fold(v, [](double a, double b) { return fmin(a, b); });
}

// ---------------------------------------------------------------------------
// 1. Reduction to tridiagonal form
// ---------------------------------------------------------------------------

struct TrdArgs {
  C64* A;            // d x d working matrix, row-major, Hermitian (both triangles)
  C64* V;            // d x d: row k holds v_k in columns k+1 .. d-1 (v_k[k+1] = 1)
  double* diag;      // d: diagonal of T
  double* off;       // d - 1: off-diagonal of T (beta_k)
  C64* tau;          // d - 1 reflector scalars
  int d, groups;
};

// What step k needs of row k once the previous update is in: the reflector
// H_k = I - t v v^dagger from the column's leading entry al = x[k + 1] and
// nrm = sum of |x[c]|^2 over c >= k + 2; v[c] = sc x[c], v[k + 1] = 1.
struct Reflector {
  double beta;
  C64 t, sc;
};
__device__ __forceinline__ Reflector reflector(C64 al, double nrm) {
  Reflector h{al.re, C64{0.0, 0.0}, C64{0.0, 0.0}};
  if (nrm == 0.0 && al.im == 0.0) return h;
  h.beta = -copysign(sqrt(al.re * al.re + al.im * al.im + nrm), al.re);
  // two divisions, side by side: 1 / beta and 1 / |alpha - beta|^2, both
  // scaled by beta's exponent so that neither reciprocal overflows (the second
  // did below |beta| = 7e-155, where the squares still have bits)
  const int ex = __builtin_amdgcn_frexp_exp(h.beta);
  const C64 den{ldexp(al.re - h.beta, -ex), ldexp(al.im, -ex)};
  const double ib = 1.0 / ldexp(h.beta, -ex), id = 1.0 / (den.re * den.re + den.im * den.im);
  h.t = C64{-den.re * ib, -den.im * ib};
  h.sc = C64{ldexp(den.re * id, -ex), ldexp(-den.im * id, -ex)};
  return h;
}

// Sums of eight values over a wave: lane l returns the sum of v[l / 8].  Each
// exchange halves the number of values instead of repeating the sum.
__device__ __forceinline__ double wave_sum8(const double (&v)[8]) {
  auto pair = [](double lo, double hi, auto swap) {
    const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
    const uint2 x = swap(a.x, b.x), y = swap(a.y, b.y);
    return __builtin_bit_cast(double, make_uint2(x.x, y.x)) + __builtin_bit_cast(double, make_uint2(x.y, y.y));
  };
  auto swap32 = [](uint32_t a, uint32_t b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return make_uint2(r[0], r[1]);
  };
  auto swap16 = [](uint32_t a, uint32_t b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    return make_uint2(r[0], r[1]);
  };
  double h[4], q[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) h[i] = pair(v[i], v[i + 4], swap32);
#pragma unroll
  for (int i = 0; i < 2; ++i) q[i] = pair(h[i], h[i + 2], swap16);
  const bool up = threadIdx.x & 8;
  double x = (up ? q[1] : q[0]) + dpp_lane<0x128>(up ? q[0] : q[1]);
  x += dpp_lane<0x141>(x);  // the mirror image in the eight lanes
  x += dpp_lane<0x4e>(x);   // lane ^ 2
  x += dpp_lane<0xb1>(x);   // lane ^ 1
  return x;
}

// Step k (0 <= k <= d - 2), d <= DMAX <= 2048, NT threads per workgroup.
// yprev / pprev: A22 v_{k-1} (entries k .. d-1) and its partial sums from
// step k - 1; ynext / pnext are this step's.  Rows r >= k + 1 belong to
// workgroup r % groups, at most RB of them to one, and thread t of it takes
// the columns k + t + NT j of all its rows: the entries of v_{k-1}, w_{k-1}
// and v_k that it needs stay in its registers.  Bound by latency (the
// operands of d = 1024 are in the caches and take 0.5 us to compute with; a
// step 7.6 -> 6.7 us against vectors in LDS, eight barriers and sums through
// LDS; with 256 threads 7.0):
// every load is issued at the start, the partial sums of the previous step
// are added by each wave for itself, and the workgroup meets at two barriers
// only, for the norm of the column and for its rows' sums.
template <int DMAX, int NT, int RB>
__global__ __launch_bounds__(NT) void trd_step_kernel(TrdArgs g, int k, const C64* __restrict__ yprev,
                                                      C64* __restrict__ ynext, const double* __restrict__ pprev,
                                                      double* __restrict__ pnext) {
  constexpr int NW = NT / 64, J = DMAX / NT;
  static_assert(RB % 4 == 0 && J * NT == DMAX, "rows are summed four at a time");
  __shared__ double red[NW];
  __shared__ C64 head[2];             // x[k], x[k + 1]
  __shared__ double ysum[2 * RB][NW];  // the waves' parts of y, rows' re then im in fours
  __shared__ C64 vown[RB];            // v_k at the workgroup's rows
  const int d = g.d, P = g.groups, wg = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int r1 = k + 1;
  const int first = r1 + ((wg - r1 % P) + P) % P;  // first owned row >= k + 1
  if (first >= d && wg != 0) {
    if (tid == 0) pnext[wg] = 0.0;
    return;
  }
  const bool prev = k > 0;
  const C64* vprow = g.V + int64_t(k - 1) * d;  // v_{k-1}; used only when prev
  const C64* rowk = g.A + int64_t(k) * d;
  // ---- loads
  double pp = 0.0;
  C64 tp{0.0, 0.0}, vpk{0.0, 0.0}, ypk{0.0, 0.0};
  C64 vpr[RB], ypr[RB];
  if (prev) {
    tp = g.tau[k - 1];
    vpk = vprow[k];
    ypk = yprev[k];
    for (int p = lane; p < P; p += 64) pp += pprev[p];
  }
  C64 x[J], vp[J], w[J], a[RB][J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = k + tid + NT * j;
    x[j] = vp[j] = w[j] = C64{0.0, 0.0};
    if (c < d) {
      x[j] = rowk[c];
      if (prev) {
        vp[j] = vprow[c];
        w[j] = yprev[c];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int r = first + i * P;
    vpr[i] = ypr[i] = C64{0.0, 0.0};
    if (r < d && prev) {
      vpr[i] = vprow[r];
      ypr[i] = yprev[r];
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = k + tid + NT * j;
      a[i][j] = (r < d && c > k && c < d) ? g.A[int64_t(r) * d + c] : C64{0.0, 0.0};
    }
  }
  // ---- the previous step's alpha and w; row k with its update applied
  // (x_c = conj(row_c) is column k)
  double ap = 0.0;
  if (prev) ap = -0.5 * (tp.re * tp.re + tp.im * tp.im) * wave_sum(pp);
  auto wfrom = [&](C64 v, C64 y) -> C64 {
    const C64 ty = cmul(tp, y);
    return C64{ty.re + ap * v.re, ty.im + ap * v.im};
  };
  const C64 wpk = wfrom(vpk, ypk);
  double nrm = 0.0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = k + tid + NT * j;
    w[j] = wfrom(vp[j], w[j]);
    const C64 t1 = cmulc(w[j], vpk);   // v[k] conj(w[c])
    const C64 t2 = cmulc(vp[j], wpk);  // w[k] conj(v[c])
    x[j] = C64{x[j].re - (t1.re + t2.re), -(x[j].im - (t1.im + t2.im))};
    if (c >= k + 2 && c < d) nrm += x[j].re * x[j].re + x[j].im * x[j].im;
  }
  if (tid < 2) head[tid] = x[0];
  nrm = wave_sum(nrm);
  if (lane == 0) red[wave] = nrm;
  __syncthreads();
  nrm = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) nrm += red[i];
  const Reflector h = reflector(head[1], nrm);
  C64* vrow = g.V + int64_t(k) * d;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = k + tid + NT * j;
    C64 v = cmul(x[j], h.sc);
    if (c == k + 1) v = C64{1.0, 0.0};
    if (c <= k || c >= d) v = C64{0.0, 0.0};
    x[j] = v;
    if (wg == 0 && c > k && c < d) vrow[c] = v;
  }
  if (wg == 0 && tid == 0) {
    g.diag[k] = head[0].re;
    g.off[k] = h.beta;
    g.tau[k] = h.t;
  }
  // ---- own rows: update with (v_{k-1}, w_{k-1}) on columns >= k + 1, and
  // y_k[r] = sum_c A22[r][c] v_k[c]
#pragma unroll
  for (int b = 0; b < RB; b += 4) {
    double y[8];
#pragma unroll
    for (int i = b; i < b + 4; ++i) {
      const int r = first + i * P;
      double yr = 0.0, yi = 0.0;
      if (r < d) {
        C64* row = g.A + int64_t(r) * d;
        const C64 wpr = wfrom(vpr[i], ypr[i]);
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int c = k + tid + NT * j;
          C64 e = a[i][j];
          if (prev) {
            const C64 t1 = cmulc(w[j], vpr[i]), t2 = cmulc(vp[j], wpr);
            e.re -= t1.re + t2.re;
            e.im -= t1.im + t2.im;
            if (c > k && c < d) row[c] = e;
          }
          yr += e.re * x[j].re - e.im * x[j].im;
          yi += e.re * x[j].im + e.im * x[j].re;
          if (c == r) vown[i] = x[j];
        }
      }
      y[i - b] = yr;
      y[4 + i - b] = yi;
    }
    const double sum = wave_sum8(y);
    if ((lane & 7) == 0) ysum[2 * b + (lane >> 3)][wave] = sum;
  }
  __syncthreads();
  if (wave != 0) return;
  double part = 0.0;
  const int r = first + lane * P;
  if (lane < RB && r < d) {
    const int q = 2 * (lane & ~3) + (lane & 3);
    double yr = 0.0, yi = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      yr += ysum[q][i];
      yi += ysum[q + 4][i];
    }
    ynext[r] = C64{yr, yi};
    const C64 v = vown[lane];
    part = v.re * yr + v.im * yi;  // Re(conj(v_r) y_r)
  }
  part = wave_sum(part);
  if (lane == 0) pnext[wg] = part;
}

// The same step for d > 2048 (d <= DMAX), where a thread's columns no longer
// fit its registers: v_k in LDS, w_{k-1} formed from global memory where it
// is used, and wave w of a workgroup takes its rows first + (w + i NT/64)
// groups.
template <int DMAX, int NT>
__global__ __launch_bounds__(NT) void trd_step_wide_kernel(TrdArgs g, int k, const C64* __restrict__ yprev,
                                                      C64* __restrict__ ynext, const double* __restrict__ pprev,
                                                      double* __restrict__ pnext) {
  constexpr int NW = NT / 64;
  constexpr int J2 = (DMAX + NT - 1) / NT;  // row-k slots per thread
  __shared__ C64 vs[DMAX];  // v_k (column index), with x_k before scaling
  __shared__ double red[NW];
  const int d = g.d, P = g.groups, wg = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int r1 = k + 1;
  const int first = r1 + ((wg - r1 % P) + P) % P;  // first owned row >= k + 1
  if (first >= d && wg != 0) {
    if (tid == 0) pnext[wg] = 0.0;
    return;
  }
  const bool prev = k > 0;
  const C64* vprow = g.V + int64_t(k - 1) * d;  // v_{k-1}; used only when prev
  const C64* rowk = g.A + int64_t(k) * d;
  // ---- independent loads
  double pp = 0.0;
  if (prev)
    for (int p = tid; p < P; p += NT) pp += pprev[p];
  C64 rk[J2], vl[J2], yl[J2];
#pragma unroll
  for (int j = 0; j < J2; ++j) {
    const int c = k + tid + NT * j;
    rk[j] = vl[j] = yl[j] = C64{0.0, 0.0};
    if (c < d) {
      rk[j] = rowk[c];
      if (prev) {
        vl[j] = vprow[c];
        yl[j] = yprev[c];
      }
    }
  }
  C64 vpk{0.0, 0.0}, ypk{0.0, 0.0};
  const int r0 = first + wave * P;
  C64 vr0{0.0, 0.0}, yr0{0.0, 0.0};
  if (prev) {
    vpk = vprow[k];
    ypk = yprev[k];
    if (r0 < d) {
      vr0 = vprow[r0];
      yr0 = yprev[r0];
    }
  }
  // ---- the previous step's alpha and w
  C64 tp{0.0, 0.0};
  double ap = 0.0;
  if (prev) {
    tp = g.tau[k - 1];
    const double s = block_sum_allN<NW>(pp, red);
    ap = -0.5 * (tp.re * tp.re + tp.im * tp.im) * s;
  }
  auto wfrom = [&](C64 v, C64 y) -> C64 {
    const C64 ty = cmul(tp, y);
    return C64{ty.re + ap * v.re, ty.im + ap * v.im};
  };
  const C64 wpk = wfrom(vpk, ypk);
  // row k with the previous update applied; x_c = conj(row_c) is column k
  double nrm = 0.0;
#pragma unroll
  for (int j = 0; j < J2; ++j) {
    const int c = k + tid + NT * j;
    if (c < d) {
      C64 r = rk[j];
      if (prev) {
        const C64 wc = wfrom(vl[j], yl[j]);
        const C64 t1 = cmulc(wc, vpk);     // v[k] conj(w[c])
        const C64 t2 = cmulc(vl[j], wpk);  // w[k] conj(v[c])
        r.re -= t1.re + t2.re;
        r.im -= t1.im + t2.im;
      }
      rk[j] = conjg(r);
      vs[c] = rk[j];
      if (c >= k + 2) nrm += r.re * r.re + r.im * r.im;
    }
  }
  nrm = block_sum_allN<NW>(nrm, red);  // its barriers also publish vs
  const C64 al = vs[k + 1];
  const double dk = vs[k].re;
  const Reflector h = reflector(al, nrm);
  __syncthreads();  // everyone has read vs[k], vs[k + 1]
  C64* vrow = g.V + int64_t(k) * d;
#pragma unroll
  for (int j = 0; j < J2; ++j) {
    const int c = k + tid + NT * j;
    if (c > k && c < d) {
      const C64 v = c == k + 1 ? C64{1.0, 0.0} : cmul(rk[j], h.sc);
      vs[c] = v;
      if (wg == 0) vrow[c] = v;
    }
  }
  if (wg == 0 && tid == 0) {
    g.diag[k] = dk;
    g.off[k] = h.beta;
    g.tau[k] = h.t;
  }
  __syncthreads();
  // own rows: update with (v_{k-1}, w_{k-1}) on columns >= k + 1, and
  // y_k[r] = sum_c A22[r][c] v_k[c]
  double part = 0.0;
  for (int r = r0, i = 0; r < d; r += NW * P, ++i) {
    C64* row = g.A + int64_t(r) * d;
    C64 vpr{0.0, 0.0}, wpr{0.0, 0.0};
    if (prev) {
      vpr = i == 0 ? vr0 : vprow[r];
      wpr = wfrom(vpr, i == 0 ? yr0 : yprev[r]);
    }
    double yr = 0.0, yi = 0.0;
    auto visit = [&](int c, C64 a) {
      if (prev) {
        const C64 vc = vprow[c], wc = wfrom(vc, yprev[c]);
        const C64 t1 = cmulc(wc, vpr), t2 = cmulc(vc, wpr);
        a.re -= t1.re + t2.re;
        a.im -= t1.im + t2.im;
        row[c] = a;
      }
      const C64 v = vs[c];
      yr += a.re * v.re - a.im * v.im;
      yi += a.re * v.im + a.im * v.re;
    };
    for (int c = k + 1 + lane; c < d; c += 64) visit(c, row[c]);
    yr = wave_sum(yr);
    yi = wave_sum(yi);
    if (lane == 0) {
      ynext[r] = C64{yr, yi};
      const C64 v = vs[r];
      part += v.re * yr + v.im * yi;  // Re(conj(v_r) y_r)
    }
  }
  part = block_sum_allN<NW>(part, red);
  if (tid == 0) pnext[wg] = part;
}

// A lane's value, the same lane for the whole wave.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint2 u = __builtin_bit_cast(uint2, v);
  return __builtin_bit_cast(double,
                            make_uint2(__builtin_amdgcn_readlane(u.x, lane), __builtin_amdgcn_readlane(u.y, lane)));
}

// The last steps, k0 = max(0, d - kTrdTail) on, by one workgroup with the
// trailing matrix in LDS (144 KiB): a step in a launch of its own costs 5.5
// us at any size, of which more than half is the launch; here it takes 3.6 us
// on average (d = 1024, 8 waves; 4.1 with 16, whose common work shares the
// SIMDs, 3.8 with 4).  Every wave holds the vectors in its lanes (column lane + 64 j), so a step
// has one barrier, for y = A22 v; wave w updates and multiplies the rows
// k + 1 + w + 8 i, four at a time.  The same steps in the same arithmetic
// as trd_step_kernel, the update of step k0 - 1 included (yprev its A22 v).
constexpr int kTrdTail = 96, kTailWaves = 8;

__global__ __launch_bounds__(64 * kTailWaves) void trd_tail_kernel(TrdArgs g, int k0,
                                                                   const C64* __restrict__ yprev) {
  constexpr int J = (kTrdTail + 63) / 64;
  __shared__ C64 S[kTrdTail * kTrdTail];
  __shared__ C64 ys[2][kTrdTail];
  const int d = g.d, m = d - k0, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  C64 vp[J], y[J], w[J], x[J];
  C64 tp{0.0, 0.0};
  if (k0 > 0) tp = g.tau[k0 - 1];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = lane + 64 * j;
    vp[j] = y[j] = C64{0.0, 0.0};
    if (k0 > 0 && c < m) {
      vp[j] = g.V[int64_t(k0 - 1) * d + k0 + c];
      y[j] = yprev[k0 + c];
    }
  }
  for (int r = wave; r < m; r += kTailWaves)
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      if (c < m) S[r * kTrdTail + c] = g.A[int64_t(k0 + r) * d + k0 + c];
    }
  __syncthreads();
  auto at = [&](const C64(&u)[J], int c) -> C64 {  // c uniform
    const C64 v = c < 64 ? u[0] : u[J - 1];
    return C64{lane_value(v.re, c & 63), lane_value(v.im, c & 63)};
  };
  for (int k = 0;; ++k) {
    // the previous step's w
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      if (k > 0) y[j] = c >= k && c < m ? ys[(k - 1) & 1][c] : C64{0.0, 0.0};
      s += vp[j].re * y[j].re + vp[j].im * y[j].im;
    }
    const double ap = -0.5 * (tp.re * tp.re + tp.im * tp.im) * wave_sum(s);
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const C64 ty = cmul(tp, y[j]);
      w[j] = C64{ty.re + ap * vp[j].re, ty.im + ap * vp[j].im};
    }
    // row k with the update applied; x_c = conj(row_c) is column k
    const C64 vpk = at(vp, k), wpk = at(w, k);
    double nrm = 0.0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      x[j] = C64{0.0, 0.0};
      if (c >= k && c < m) {
        const C64 a = S[k * kTrdTail + c];
        const C64 t1 = cmulc(w[j], vpk), t2 = cmulc(vp[j], wpk);
        x[j] = C64{a.re - (t1.re + t2.re), -(a.im - (t1.im + t2.im))};
        if (c >= k + 2) nrm += x[j].re * x[j].re + x[j].im * x[j].im;
      }
    }
    const double dk = at(x, k).re;
    if (threadIdx.x == 0) g.diag[k0 + k] = dk;
    if (k == m - 1) break;
    const Reflector h = reflector(at(x, k + 1), wave_sum(nrm));
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      C64 v = cmul(x[j], h.sc);
      if (c == k + 1) v = C64{1.0, 0.0};
      if (c <= k || c >= m) v = C64{0.0, 0.0};
      x[j] = v;
      if (wave == 0 && c > k && c < m) g.V[int64_t(k0 + k) * d + k0 + c] = v;
    }
    if (threadIdx.x == 0) {
      g.off[k0 + k] = h.beta;
      g.tau[k0 + k] = h.t;
    }
    for (int r0 = k + 1 + wave; r0 < m; r0 += 4 * kTailWaves) {
      double yv[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = r0 + i * kTailWaves;
        double yr = 0.0, yi = 0.0;
        if (r < m) {
          const C64 vpr = at(vp, r), wpr = at(w, r);
#pragma unroll
          for (int j = 0; j < J; ++j) {
            if (64 * (j + 1) <= k + 1 || 64 * j >= m) continue;  // no column of this slot is left
            const int c = lane + 64 * j;
            if (c > k && c < m) {
              C64 e = S[r * kTrdTail + c];
              const C64 t1 = cmulc(w[j], vpr), t2 = cmulc(vp[j], wpr);
              e.re -= t1.re + t2.re;
              e.im -= t1.im + t2.im;
              S[r * kTrdTail + c] = e;
              yr += e.re * x[j].re - e.im * x[j].im;
              yi += e.re * x[j].im + e.im * x[j].re;
            }
          }
        }
        yv[i] = yr;
        yv[4 + i] = yi;
      }
      const double sum = wave_sum8(yv);
      const int q = lane >> 3, r = r0 + (q & 3) * kTailWaves;
      if ((lane & 7) == 0 && r < m) (q < 4 ? ys[k & 1][r].re : ys[k & 1][r].im) = sum;
    }
#pragma unroll
    for (int j = 0; j < J; ++j) vp[j] = x[j];
    tp = h.t;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// 2. Splitting, norms, status
// ---------------------------------------------------------------------------

struct TriScal {
  double tnorm, pivmin;
  int status;  // 0 finite, -1 not finite
  int pad;
};

// One workgroup of 256 threads: ||T|| (largest Gershgorin bound), zeroes
// negligible off-diagonal entries, the unreduced block [bstart[i], bend[i])
// of every index (each thread scans a contiguous range, then a scan over the
// threads' results), the pivot floor, and whether everything is finite.
__global__ __launch_bounds__(256) void tri_split_kernel(const double* __restrict__ a, double* __restrict__ e, int d,
                                                        int* __restrict__ bstart, int* __restrict__ bend,
                                                        TriScal* __restrict__ ts) {
  __shared__ double mx[3][4];
  __shared__ double bc[2];
  __shared__ int lo_s[256], hi_s[256];
  const int tid = threadIdx.x;
  double tn = 0.0, e2 = 0.0, bad = 0.0;
  for (int k = tid; k < d; k += 256) {
    const double ek = k < d - 1 ? fabs(e[k]) : 0.0, el = k > 0 ? fabs(e[k - 1]) : 0.0;
    const double v = fabs(a[k]) + ek + el;
    if (!isfinite(v)) bad = 1.0;
    tn = fmax(tn, v);
    e2 = fmax(e2, ek * ek);
  }
  tn = wave_max(tn);
  e2 = wave_max(e2);
  bad = wave_max(bad);
  const int w = tid >> 6, l = tid & 63;
  if (l == 0) {
    mx[0][w] = tn;
    mx[1][w] = e2;
    mx[2][w] = bad;
  }
  __syncthreads();
  if (tid == 0) {
    bc[0] = fmax(fmax(mx[0][0], mx[0][1]), fmax(mx[0][2], mx[0][3]));
    bc[1] = fmax(fmax(mx[1][0], mx[1][1]), fmax(mx[1][2], mx[1][3]));
    const double b = fmax(fmax(mx[2][0], mx[2][1]), fmax(mx[2][2], mx[2][3]));
    ts->tnorm = bc[0];
    ts->pivmin = DBL_MIN * fmax(1.0, bc[1]);
    ts->status = b != 0.0 ? -1 : 0;
  }
  __syncthreads();
  const double stol = 4.0 * kEps * sqrt(double(d)) * bc[0];
  // thread tid owns indices [i0, i1); a block starts at 0 and after every
  // zero off-diagonal entry e[k] (at k + 1), and ends after it (at k + 1)
  const int per = (d + 255) / 256, i0 = min(d, tid * per), i1 = min(d, i0 + per);
  int last_start = -1, first_end = d;
  for (int k = i0; k < i1; ++k)
    if (k < d - 1 && fabs(e[k]) <= stol) e[k] = 0.0;
  __syncthreads();  // e[i0 - 1] belongs to the previous thread
  for (int k = i0; k < i1; ++k) {
    const bool starts = k == 0 || e[k - 1] == 0.0;
    if (starts) last_start = k;
  }
  for (int k = i1 - 1; k >= i0; --k) {
    const bool ends = k == d - 1 || e[k] == 0.0;
    if (ends) first_end = k + 1;
  }
  lo_s[tid] = last_start;
  hi_s[tid] = first_end;
  __syncthreads();
  // inclusive max-scan of lo_s (from the left) and min-scan of hi_s (from the right)
  for (int o = 1; o < 256; o <<= 1) {
    const int lv = tid >= o ? lo_s[tid - o] : -1;
    const int hv = tid + o < 256 ? hi_s[tid + o] : d;
    __syncthreads();
    lo_s[tid] = max(lo_s[tid], lv);
    hi_s[tid] = min(hi_s[tid], hv);
    __syncthreads();
  }
  int st = tid > 0 ? lo_s[tid - 1] : -1;
  for (int k = i0; k < i1; ++k) {
    if (k == 0 || e[k - 1] == 0.0) st = k;
    bstart[k] = st;
  }
  int en = tid < 255 ? hi_s[tid + 1] : d;
  for (int k = i1 - 1; k >= i0; --k) {
    if (k == d - 1 || e[k] == 0.0) en = k + 1;
    bend[k] = en;
  }
}

// ---------------------------------------------------------------------------
// 3. Eigenvalues by multisection of Sturm counts
// ---------------------------------------------------------------------------

// Number of eigenvalues of the block [s, t) below x: the sign changes of
// p_k = (a_k - x) p_{k-1} - e_{k-1}^2 p_{k-2}, a and e2 = e^2 in LDS scaled to
// ||T|| in [1, 2).  A p that is zero counts with its neighbours (the next one
// has the sign opposite to the one before it).  No division: the chain from
// one p to the next is one fused multiply-add where the pivots
// q_k = p_k / p_{k-1} take a division each, and the count belongs to a matrix
// as close to T.  In 8 steps p grows by less than 2^24 and, unreduced as the
// block is, shrinks by less than 2^-500, so it is rescaled every 8.
__device__ __forceinline__ int sturm_count(const double* a, const double* e2, int s, int t, double x) {
  double p0 = 1.0, p = a[s] - x;
  auto top = [](double v) { return uint32_t(__double2hiint(v)); };
  uint32_t c = top(p) >> 31;
  int k = s + 1;
  for (; k + 8 <= t; k += 8) {  // the LDS reads of 8 steps ahead of their use
    double ak[8], ek[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      ak[u] = a[k + u] - x;
      ek[u] = e2[k + u - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double q = fma(ak[u], p, -(ek[u] * p0));
      c += (top(q) ^ top(p)) >> 31;
      p0 = p;
      p = q;
    }
    const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p0)));
    p = ldexp(p, -ex);
    p0 = ldexp(p0, -ex);
  }
  for (; k < t; ++k) {
    const double q = fma(a[k] - x, p, -(e2[k - 1] * p0));
    c += (top(q) ^ top(p)) >> 31;
    p0 = p;
    p = q;
  }
  return int(c);
}

// A wave per index i: the (i - s)-th smallest eigenvalue of its block; the
// diagonal and the squared off-diagonal staged in LDS (d <= DMAX).
template <int DMAX>
__global__ __launch_bounds__(256) void tri_eigvals_kernel(const double* __restrict__ a, const double* __restrict__ e,
                                                          int d, const int* __restrict__ bstart,
                                                          const int* __restrict__ bend,
                                                          const TriScal* __restrict__ ts, double* __restrict__ lam) {
  __shared__ double sa[DMAX], se2[DMAX];
  const int scale = ts->tnorm > 0.0 ? ilogb(ts->tnorm) : 0;  // ||T|| 2^-scale in [1, 2)
  for (int k = threadIdx.x; k < d; k += 256) {
    sa[k] = ldexp(a[k], -scale);
    const double ek = k < d - 1 ? ldexp(e[k], -scale) : 0.0;
    se2[k] = ek * ek;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= d) return;
  const int s = bstart[i], t = bend[i], j = i - s, n = t - s;
  if (n == 1) {
    if (lane == 0) lam[i] = a[s];
    return;
  }
  const double pivmin = DBL_MIN;
  double gl = HUGE_VAL, gu = -HUGE_VAL;
  for (int k = s + lane; k < t; k += 64) {
    const double r = (k > s ? sqrt(se2[k - 1]) : 0.0) + (k < t - 1 ? sqrt(se2[k]) : 0.0);
    gl = fmin(gl, sa[k] - r);
    gu = fmax(gu, sa[k] + r);
  }
  gl = wave_min(gl);
  gu = wave_max(gu);
  const double tn = fmax(fabs(gl), fabs(gu));
  gl -= 2.0 * kEps * tn * n + 2.0 * pivmin;
  gu += 2.0 * kEps * tn * n + 2.0 * pivmin;
  double lo = gl, hi = gu;
  for (int it = 0; it < 64; ++it) {
    const double x = lo + (hi - lo) * (double(lane + 1) / 65.0);
    const int cnt = sturm_count(sa, se2, s, t, x);
    const unsigned long long above = __ballot(cnt > j);  // lanes whose point lies above the eigenvalue
    const int f = above ? __ffsll(above) - 1 : 64;
    const double xl = __shfl(x, f > 0 ? f - 1 : 0, 64), xh = __shfl(x, f < 64 ? f : 63, 64);
    const double nlo = f > 0 ? xl : lo, nhi = f < 64 ? xh : hi;
    lo = nlo;
    hi = nhi;
    if (hi - lo <= 2.0 * kEps * fmax(fabs(lo), fabs(hi)) + pivmin) break;
  }
  if (lane == 0) lam[i] = ldexp(0.5 * (lo + hi), scale);
}

// ---------------------------------------------------------------------------
// 4. Eigenvectors by twisted factorizations
// ---------------------------------------------------------------------------

// Column i of Z (d x d complex, zero outside the block, written as real
// values) by lane i % 64 of the two waves of a workgroup: wave 0 takes the
// factorization from the top and the vector above the twist index, wave 1
// the one from the bottom and the vector below it, each half of the search
// for the index and of the scaling.  Scratch: D+ at W[k d + i] and U- at
// W[d^2 + k d + i]; the diagonal and off-diagonal staged in LDS (d <= DMAX).
// Bound by latency (d = 1024: 1024 dependent divisions per wave, then the
// scratch in batches of kVecBatch whose loads overlap): d = 1024 633 -> 472 us.
constexpr int kVecBatch = 32;

template <int DMAX>
__global__ __launch_bounds__(128) void tri_vectors_kernel(const double* __restrict__ a_g,
                                                          const double* __restrict__ e_g, int d,
                                                          const int* __restrict__ bstart,
                                                          const int* __restrict__ bend, const TriScal* __restrict__ ts,
                                                          const double* __restrict__ lam, double* __restrict__ W,
                                                          C64* __restrict__ Z) {
  constexpr int B = kVecBatch;
  __shared__ double a[DMAX], e[DMAX];
  __shared__ double val[2][64];  // the waves' smallest |gamma|, then their parts of the norm
  __shared__ int idx[2][64];
  for (int k = threadIdx.x; k < d; k += 128) {
    a[k] = a_g[k];
    e[k] = k < d - 1 ? e_g[k] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, half = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  int s = 0, t = 0;  // no rows: nothing to do (past the end, or a block of one)
  double l = 0.0;
  if (i < d) {
    s = bstart[i];
    t = bend[i];
    l = lam[i];
    if (t - s == 1) {
      if (half == 0) Z[int64_t(s) * d + i] = C64{1.0, 0.0};
      t = s;
    }
  }
  const double pivmin = ts->pivmin;
  double* Dp = W + i;
  double* Um = W + int64_t(d) * d + i;
  C64* z_i = Z + i;
  if (half == 0) {
    // top down: D+_{k+1} = (a_{k+1} - l) - e_k^2 / D+_k
    double dp = 1.0;
    for (int k = s; k < t; ++k) {
      dp = k == s ? a[k] - l : (a[k] - l) - e[k - 1] * (e[k - 1] / dp);
      if (fabs(dp) < pivmin) dp = -pivmin;
      Dp[int64_t(k) * d] = dp;
    }
  } else if (t > s) {
    // bottom up: U-_k = e_k / D-_{k+1}, D-_k = (a_k - l) - U-_k e_k
    double dm = a[t - 1] - l;
    if (fabs(dm) < pivmin) dm = -pivmin;
    for (int k = t - 2; k >= s; --k) {
      const double ek = e[k], u = ek / dm;
      Um[int64_t(k) * d] = u;
      dm = (a[k] - l) - u * ek;
      if (fabs(dm) < pivmin) dm = -pivmin;
    }
  }
  __syncthreads();
  // the twist index: gamma_k = D+_k + D-_k - (a_k - l) = D+_k - U-_k e_k,
  // gamma_{t-1} = D+_{t-1}; the largest k of the smallest |gamma_k|
  const int mid = s + (t - s) / 2, lo = half == 0 ? s : mid, hi = half == 0 ? mid : t;
  double best = HUGE_VAL;
  int r = hi - 1;
  for (int k0 = hi - 1; k0 >= lo; k0 -= B) {
    double dpb[B], ub[B];
#pragma unroll
    for (int q = 0; q < B; ++q) {
      const int k = k0 - q;
      dpb[q] = k >= lo ? Dp[int64_t(k) * d] : 0.0;
      ub[q] = k >= lo && k < t - 1 ? Um[int64_t(k) * d] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < B; ++q) {
      const int k = k0 - q;
      if (k >= lo) {
        const double gam = fabs(dpb[q] - ub[q] * e[k]);  // e[t - 1] only with ub = 0
        if (gam < best) {
          best = gam;
          r = k;
        }
      }
    }
  }
  val[half][lane] = best;
  idx[half][lane] = r;
  __syncthreads();
  r = val[0][lane] < val[1][lane] ? idx[0][lane] : idx[1][lane];
  __syncthreads();  // val is used again
  // z_r = 1; z_k = -(e_k / D+_k) z_{k+1} above r, z_{k+1} = -U-_k z_k below
  double nrm = 0.0, z = 1.0;
  if (half == 0) {
    if (t > s) {
      z_i[int64_t(r) * d] = C64{1.0, 0.0};
      nrm = 1.0;
    }
    for (int k0 = r - 1; k0 >= s && t > s; k0 -= B) {
      double b[B];
#pragma unroll
      for (int q = 0; q < B; ++q) b[q] = k0 - q >= s ? Dp[int64_t(k0 - q) * d] : 1.0;
#pragma unroll
      for (int q = 0; q < B; ++q) {
        const int k = k0 - q;
        if (k >= s) {
          z = -(e[k] / b[q]) * z;
          z_i[int64_t(k) * d] = C64{z, 0.0};
          nrm += z * z;
        }
      }
    }
  } else {
    for (int k0 = r; k0 < t - 1; k0 += B) {
      double b[B];
#pragma unroll
      for (int q = 0; q < B; ++q) b[q] = k0 + q < t - 1 ? Um[int64_t(k0 + q) * d] : 0.0;
#pragma unroll
      for (int q = 0; q < B; ++q) {
        const int k = k0 + q;
        if (k < t - 1) {
          z = -b[q] * z;
          z_i[int64_t(k + 1) * d] = C64{z, 0.0};
          nrm += z * z;
        }
      }
    }
  }
  val[half][lane] = nrm;
  __syncthreads();
  if (t == s) return;
  const double inv = 1.0 / sqrt(val[0][lane] + val[1][lane]);
  const int z0 = half == 0 ? s : r + 1, z1 = half == 0 ? r + 1 : t;  // the rows this wave wrote
  for (int k0 = z0; k0 < z1; k0 += B) {
    double b[B];
#pragma unroll
    for (int q = 0; q < B; ++q) b[q] = k0 + q < z1 ? z_i[int64_t(k0 + q) * d].re : 0.0;
#pragma unroll
    for (int q = 0; q < B; ++q)
      if (k0 + q < z1) z_i[int64_t(k0 + q) * d].re = b[q] * inv;
  }
}

// ---------------------------------------------------------------------------
// 5. Clusters
// ---------------------------------------------------------------------------

// A deterministic value in [-1, 1) from (i, k) (a 64-bit integer hash).
__device__ __forceinline__ double hash_unit(uint64_t i, uint64_t k) {
  uint64_t x = i * 0x9E3779B97F4A7C15ull + k * 0xBF58476D1CE4E5B9ull;
  x ^= x >> 31;
  x *= 0x94D049BB133111EBull;
  x ^= x >> 29;
  return double(x >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// Solves (T_b - sig I) x = y in place (y: n values), T_b the block of
// (a, e) starting at s, by Gaussian elimination with partial pivoting; dd,
// du, du2: n values each of scratch.  One thread.
__device__ void tri_solve(const double* __restrict__ a, const double* __restrict__ e, int s, int n, double sig,
                          double tiny, double* __restrict__ dd, double* __restrict__ du, double* __restrict__ du2,
                          double* __restrict__ y) {
  for (int k = 0; k < n; ++k) {
    dd[k] = a[s + k] - sig;
    du[k] = k < n - 1 ? e[s + k] : 0.0;
    du2[k] = 0.0;
  }
  for (int k = 0; k < n - 1; ++k) {
    const double ek = e[s + k];
    if (fabs(dd[k]) >= fabs(ek)) {
      if (dd[k] == 0.0) dd[k] = tiny;
      const double m = ek / dd[k];
      dd[k + 1] -= m * du[k];
      y[k + 1] -= m * y[k];
    } else {
      const double m = dd[k] / ek;
      dd[k] = ek;
      const double t = dd[k + 1];
      dd[k + 1] = du[k] - m * t;
      if (k < n - 2) {
        du2[k] = du[k + 1];
        du[k + 1] = -m * du[k + 1];
      }
      du[k] = t;
      const double yk = y[k];
      y[k] = y[k + 1];
      y[k + 1] = yk - m * y[k + 1];
    }
  }
  if (dd[n - 1] == 0.0) dd[n - 1] = tiny;
  y[n - 1] /= dd[n - 1];
  if (n > 1) y[n - 2] = (y[n - 2] - du[n - 2] * y[n - 1]) / dd[n - 2];
  for (int k = n - 3; k >= 0; --k) y[k] = (y[k] - du[k] * y[k + 1] - du2[k] * y[k + 2]) / dd[k];
}

// Workgroup i (64 threads) treats the cluster that starts at index i, if
// one does; 4 n values of scratch at W + 2 d i (clusters start at least two
// indices apart, so the areas do not overlap).
__global__ __launch_bounds__(64) void tri_cluster_kernel(const double* __restrict__ a, const double* __restrict__ e,
                                                         int d, const int* __restrict__ bstart,
                                                         const int* __restrict__ bend, const TriScal* __restrict__ ts,
                                                         const double* __restrict__ lam, double* __restrict__ W,
                                                         C64* __restrict__ Z) {
  const int i = blockIdx.x, lane = threadIdx.x;
  const int s = bstart[i], t = bend[i], n = t - s;
  if (n < 2) return;
  const double tn = ts->tnorm, gap = kClusterTol * tn;
  const bool starts = (i == s || lam[i] - lam[i - 1] > gap) && i + 1 < t && lam[i + 1] - lam[i] <= gap;
  if (!starts) return;
  int c = 1;
  while (i + c < t && lam[i + c] - lam[i + c - 1] <= gap) ++c;
  double* dd = W + int64_t(2) * d * i;
  double* du = dd + n;
  double* du2 = du + n;
  double* y = du2 + n;
  const double pert = 10.0 * kEps * tn, tiny = kEps * tn;
  double prev = -HUGE_VAL;
  for (int m = 0; m < c; ++m) {
    double sig = lam[i + m];
    if (m > 0 && sig - prev < pert) sig = prev + pert;
    prev = sig;
    for (int k = lane; k < n; k += 64) y[k] = hash_unit(uint64_t(i + m), uint64_t(k));
    for (int it = 0; it < 3; ++it) {
      __syncthreads();
      if (lane == 0) tri_solve(a, e, s, n, sig, tiny, dd, du, du2, y);
      __syncthreads();
      for (int q = 0; q < m; ++q) {  // orthogonalise against the earlier members
        const C64* zq = Z + int64_t(s) * d + (i + q);
        double dot = 0.0;
        for (int k = lane; k < n; k += 64) dot += zq[int64_t(k) * d].re * y[k];
        dot = wave_sum(dot);
        for (int k = lane; k < n; k += 64) y[k] -= dot * zq[int64_t(k) * d].re;
      }
      double nrm = 0.0;
      for (int k = lane; k < n; k += 64) nrm += y[k] * y[k];
      nrm = wave_sum(nrm);
      const double inv = 1.0 / sqrt(nrm);
      for (int k = lane; k < n; k += 64) y[k] *= inv;
    }
    C64* zm = Z + int64_t(s) * d + (i + m);
    for (int k = lane; k < n; k += 64) zm[int64_t(k) * d] = C64{y[k], 0.0};
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// 6. Newton-Schulz matrix, fills
// ---------------------------------------------------------------------------

// M = 1.5 I - 0.5 G (d x d contiguous).
__global__ __launch_bounds__(256) void ns_matrix_kernel(const C64* __restrict__ G, C64* __restrict__ M, int n) {
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= (int64_t(1) << (2 * n))) return;
  const int64_t r = e >> n, c = e & ((int64_t(1) << n) - 1);
  const C64 g = G[e];
  M[e] = C64{(r == c ? 1.5 : 0.0) - 0.5 * g.re, -0.5 * g.im};
}

__global__ __launch_bounds__(256) void zero_kernel(C64* __restrict__ X, int64_t count) {
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e < count) X[e] = C64{0.0, 0.0};
}

// ---------------------------------------------------------------------------
// 7. Back-transformation
// ---------------------------------------------------------------------------

constexpr int kNb = kEighBlock;  // 64
constexpr int kGramRows = kEighGramRows;

// v_{k0 + j}[r] from the reflector rows (0 at and above the diagonal).
__device__ __forceinline__ C64 refl(const C64* __restrict__ V, int d, int k0, int j, int nk, int r) {
  const int k = k0 + j;
  if (j >= nk || r <= k || r >= d) return C64{0.0, 0.0};
  return V[int64_t(k) * d + r];
}

// Partial Gram matrices of the blocks' reflectors: workgroup (b, y) sums
// conj(v_j[r]) v_l[r] over the rows r of chunk y (kGramRows rows from
// k0 + 1) into Gp[(b * gchunks + y)][j][l].
__global__ __launch_bounds__(256) void bt_gram_kernel(const C64* __restrict__ V, int d, int gchunks,
                                                      C64* __restrict__ Gp) {
  __shared__ C64 ch[32][kNb + 1];
  const int b = blockIdx.x, y = blockIdx.y, tid = threadIdx.x;
  const int k0 = b * kNb, nk = min(kNb, d - 1 - k0);
  const int rs = k0 + 1 + y * kGramRows, re = min(d, rs + kGramRows);
  const int tj = tid >> 4, tl = tid & 15;  // entries (4 tj + x, 4 tl + y)
  C64 acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int z = 0; z < 4; ++z) acc[x][z] = C64{0.0, 0.0};
  for (int r0 = rs; r0 < re; r0 += 32) {
    __syncthreads();
    for (int q = tid; q < 32 * kNb; q += 256) {
      const int j = q >> 5, rr = q & 31, r = r0 + rr;
      ch[rr][j] = r < re ? refl(V, d, k0, j, nk, r) : C64{0.0, 0.0};
    }
    __syncthreads();
#pragma unroll 4
    for (int rr = 0; rr < 32; ++rr) {
      C64 u[4], w[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        u[x] = ch[rr][4 * tj + x];
        w[x] = ch[rr][4 * tl + x];
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          const C64 p = cmulc(u[x], w[z]);
          acc[x][z].re += p.re;
          acc[x][z].im += p.im;
        }
    }
  }
  C64* G = Gp + (int64_t(b) * gchunks + y) * kNb * kNb;
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int z = 0; z < 4; ++z) G[(4 * tj + x) * kNb + 4 * tl + z] = acc[x][z];
}

// Workgroup b: G = the sum of block b's partial Gram matrices (fixed
// order), then the triangular factor column by column:
// T[j][j] = tau_j, T[0:j][j] = -tau_j T[0:j][0:j] G[0:j][j], four threads to
// a row.  Bound by the chain of columns (d = 1024: 164 -> 83 us).
__global__ __launch_bounds__(256) void bt_tmat_kernel(const C64* __restrict__ Gp, int gchunks,
                                                      const C64* __restrict__ tau, int d, C64* __restrict__ Tall) {
  __shared__ C64 gt[kNb][kNb + 1];  // G, then T in place
  const int b = blockIdx.x, tid = threadIdx.x, row = tid >> 2, quarter = tid & 3;
  const int k0 = b * kNb, nk = min(kNb, d - 1 - k0);
  for (int q = tid; q < kNb * kNb; q += 256) {
    C64 g{0.0, 0.0};
    for (int y = 0; y < gchunks; ++y) {
      const C64 v = Gp[(int64_t(b) * gchunks + y) * kNb * kNb + q];
      g.re += v.re;
      g.im += v.im;
    }
    gt[q >> 6][q & 63] = g;
  }
  __syncthreads();
  for (int j = 0; j < kNb; ++j) {
    const C64 tj_ = j < nk ? tau[k0 + j] : C64{0.0, 0.0};
    C64 sum{0.0, 0.0};
    for (int q = row + quarter; q < j; q += 4) {
      const C64 p = cmul(gt[row][q], gt[q][j]);  // T[row][q] G[q][j]
      sum.re += p.re;
      sum.im += p.im;
    }
    sum.re += dpp_lane<0x4e>(sum.re);  // lane ^ 2
    sum.im += dpp_lane<0x4e>(sum.im);
    sum.re += dpp_lane<0xb1>(sum.re);  // lane ^ 1
    sum.im += dpp_lane<0xb1>(sum.im);
    __syncthreads();
    if (quarter == 0) {
      C64 v{0.0, 0.0};
      if (row < j) {
        const C64 p = cmul(tj_, sum);
        v = C64{-p.re, -p.im};
      } else if (row == j) {
        v = tj_;
      }
      gt[row][j] = v;
    }
    __syncthreads();
  }
  C64* T = Tall + int64_t(b) * kNb * kNb;
  for (int q = tid; q < kNb * kNb; q += 256) T[q] = gt[q >> 6][q & 63];
}

// W_b = V_b T_b, stored like the reflectors: W[(k0 + j) d + r] =
// sum_{l <= j} v_{k0 + l}[r] T_b[l][j] for r in [k0 + 1, d) (workgroup (b,
// y): rows k0 + 1 + 64 y ...).
__global__ __launch_bounds__(256) void bt_wfactor_kernel(const C64* __restrict__ V, const C64* __restrict__ Tall,
                                                         int d, C64* __restrict__ W) {
  __shared__ C64 vs[64][kNb + 1];  // [row][l]
  __shared__ C64 ts[kNb][kNb + 1];  // [l][j]
  const int b = blockIdx.x, tid = threadIdx.x;
  const int k0 = b * kNb, nk = min(kNb, d - 1 - k0);
  const int r0 = k0 + 1 + blockIdx.y * 64;
  if (r0 >= d) return;
  for (int q = tid; q < 64 * kNb; q += 256) {
    const int l = q >> 6, rr = q & 63;
    vs[rr][l] = refl(V, d, k0, l, nk, r0 + rr);
    ts[q >> 6][q & 63] = Tall[int64_t(b) * kNb * kNb + q];
  }
  __syncthreads();
  const int tr = tid >> 4, tc = tid & 15;  // rows 4 tr + x, columns j = 4 tc + z
  C64 acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int z = 0; z < 4; ++z) acc[x][z] = C64{0.0, 0.0};
  for (int l = 0; l < kNb; ++l) {
    C64 u[4], w[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      u[x] = vs[4 * tr + x][l];
      w[x] = ts[l][4 * tc + x];
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        const C64 p = cmul(u[x], w[z]);
        acc[x][z].re += p.re;
        acc[x][z].im += p.im;
      }
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int r = r0 + 4 * tr + x;
    if (r >= d) continue;
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const int j = 4 * tc + z;
      if (j < nk) W[int64_t(k0 + j) * d + r] = acc[x][z];
    }
  }
}

// Partial sums of V_b^dagger Z over the row chunk y of R rows (rows from
// k0 + 1): P[y][j][c] for the 32 reflectors j of half z and the column tile x
// of 64.  The next 16 rows are loaded while 16 are summed, and half of the
// reflectors to a workgroup occupies twice the CUs (a block of d = 1024: 29.5
// -> 18.8 us).
__global__ __launch_bounds__(256) void bt_partial_kernel(const C64* __restrict__ V, const C64* __restrict__ Z, int d,
                                                         int k0, int nk, int R, C64* __restrict__ P) {
  __shared__ C64 vs[2][16][kNb / 2 + 1];
  __shared__ C64 zs[2][16][kNb + 1];
  const int tid = threadIdx.x, tj = tid >> 4, tc = tid & 15, j0 = blockIdx.z * (kNb / 2);
  const int c0 = blockIdx.x * 64, rs = k0 + 1 + blockIdx.y * R, re = min(d, rs + R);
  C64 acc[2][4];  // reflectors j0 + 2 tj + x, columns tc + 16 y
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[x][y] = C64{0.0, 0.0};
  C64 vl[2], zl[4];
  auto load = [&](int r0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int q = u * 256 + tid, r = r0 + (q & 15);
      vl[u] = r < re ? refl(V, d, k0, j0 + (q >> 4), nk, r) : C64{0.0, 0.0};
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = u * 256 + tid, r = r0 + (q >> 6), c = c0 + (q & 63);
      zl[u] = (r < re && c < d) ? Z[int64_t(r) * d + c] : C64{0.0, 0.0};
    }
  };
  load(rs);
  int buf = 0;
  for (int r0 = rs; r0 < re; r0 += 16, buf ^= 1) {
#pragma unroll
    for (int u = 0; u < 2; ++u) vs[buf][tid & 15][(u * 256 + tid) >> 4] = vl[u];
#pragma unroll
    for (int u = 0; u < 4; ++u) zs[buf][(u * 256 + tid) >> 6][tid & 63] = zl[u];
    __syncthreads();  // also: nobody is still reading the other buffer's previous rows
    load(r0 + 16);
#pragma unroll 4
    for (int rr = 0; rr < 16; ++rr) {
      C64 u[2], w[4];
#pragma unroll
      for (int x = 0; x < 2; ++x) u[x] = vs[buf][rr][2 * tj + x];
#pragma unroll
      for (int y = 0; y < 4; ++y) w[y] = zs[buf][rr][tc + 16 * y];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          const C64 p = cmulc(u[x], w[y]);
          acc[x][y].re += p.re;
          acc[x][y].im += p.im;
        }
    }
  }
  C64* out = P + int64_t(blockIdx.y) * kNb * d;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int c = c0 + tc + 16 * y;
      if (c < d) out[int64_t(j0 + 2 * tj + x) * d + c] = acc[x][y];
    }
}

// X[j][c] = sum_y P[y][j][c] (64 d entries, fixed order).
__global__ __launch_bounds__(256) void bt_sum_kernel(const C64* __restrict__ P, int chunks, int d,
                                                     C64* __restrict__ X) {
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t count = int64_t(kNb) * d;
  if (e >= count) return;
  C64 s{0.0, 0.0};
  for (int y = 0; y < chunks; ++y) {
    const C64 v = P[int64_t(y) * count + e];
    s.re += v.re;
    s.im += v.im;
  }
  X[e] = s;
}

// Z[r][c] -= sum_j w_{k0 + j}[r] X[j][c] on the tile (rows k0 + 1 + 32 y,
// columns 64 x), W = V_b T_b as bt_wfactor_kernel stores it.  Both operands
// of the tile (96 KiB) are loaded at once, so it waits on memory once, and
// 32 rows to a workgroup occupy twice the CUs (a block of d = 1024: 32 -> 26
// us).
constexpr int kUpdRows = 32;

__global__ __launch_bounds__(256) void bt_update_kernel(const C64* __restrict__ W, const C64* __restrict__ X, int d,
                                                        int k0, int nk, C64* __restrict__ Z) {
  __shared__ C64 vs[kUpdRows][kNb + 1];  // [row][j]
  __shared__ C64 xs[kNb][65];            // [j][column]
  const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15;  // rows 2 tr + x, columns tc + 16 y
  const int r0 = k0 + 1 + blockIdx.y * kUpdRows, c0 = blockIdx.x * 64;
#pragma unroll 4
  for (int q = tid; q < kUpdRows * kNb; q += 256) {
    const int j = q / kUpdRows, rr = q % kUpdRows, r = r0 + rr;
    vs[rr][j] = (j < nk && r < d) ? W[int64_t(k0 + j) * d + r] : C64{0.0, 0.0};
  }
#pragma unroll 8
  for (int q = tid; q < kNb * 64; q += 256) {
    const int j = q >> 6, c = c0 + (q & 63);
    xs[j][q & 63] = c < d ? X[int64_t(j) * d + c] : C64{0.0, 0.0};
  }
  C64 acc[2][4];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int r = r0 + 2 * tr + x, c = c0 + tc + 16 * y;
      acc[x][y] = (r < d && c < d) ? Z[int64_t(r) * d + c] : C64{0.0, 0.0};
    }
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < kNb; ++j) {
    C64 u[2], w[4];
#pragma unroll
    for (int x = 0; x < 2; ++x) u[x] = vs[2 * tr + x][j];
#pragma unroll
    for (int y = 0; y < 4; ++y) w[y] = xs[j][tc + 16 * y];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const C64 p = cmul(u[x], w[y]);
        acc[x][y].re -= p.re;
        acc[x][y].im -= p.im;
      }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int r = r0 + 2 * tr + x, c = c0 + tc + 16 * y;
      if (r < d && c < d) Z[int64_t(r) * d + c] = acc[x][y];
    }
}

__global__ void status_out_kernel(const TriScal* __restrict__ ts, int* __restrict__ out) { *out = ts->status; }

// Workgroups of a reduction step: four rows each up to d = 1024, eight at
// 2048 (the RB of the kernels), sixteen and more beyond, so at most 256.
int trd_groups(int d) {
  const int waves = d <= 1024 ? 4 : (d <= 2048 ? 8 : 16);
  const int g = (d + waves - 1) / waves;
  return g > kTrdMaxGroups ? kTrdMaxGroups : g;
}

}  // namespace

EighWork eigh_work(int n, void* eig_area) {
  const EighLayout L = eigh_layout(n);
  unsigned char* w = static_cast<unsigned char*>(eig_area);
  EighWork e;
  e.diag = reinterpret_cast<double*>(w + L.diag);
  e.off = reinterpret_cast<double*>(w + L.off);
  e.tau = w + L.tau;
  e.y0 = w + L.y0;
  e.y1 = w + L.y1;
  e.p0 = reinterpret_cast<double*>(w + L.p0);
  e.p1 = reinterpret_cast<double*>(w + L.p1);
  e.bstart = reinterpret_cast<int*>(w + L.bstart);
  e.bend = reinterpret_cast<int*>(w + L.bend);
  e.scal = w + L.scal;
  e.status = reinterpret_cast<int*>(w + L.scal + offsetof(TriScal, status));
  e.tfac = w + L.tfac;
  e.pbuf = w + L.pbuf;
  e.xbuf = w + L.xbuf;
  return e;
}

hipError_t launch_tridiagonalize(int n, void* A, void* V, const EighWork& w, hipStream_t s) {
  const int d = 1 << n, P = trd_groups(d);
  TrdArgs g{static_cast<C64*>(A), static_cast<C64*>(V), w.diag, w.off, static_cast<C64*>(w.tau), d, P};
  C64* y[2] = {static_cast<C64*>(w.y0), static_cast<C64*>(w.y1)};
  double* p[2] = {w.p0, w.p1};
  const int k0 = d > kTrdTail ? d - kTrdTail : 0;
  for (int k = 0; k < k0; ++k) {
    const int a = k & 1, b = a ^ 1;  // step k reads y[b], p[b] (step k - 1) and writes y[a], p[a]
    if (d <= 512)
      trd_step_kernel<512, 256, 4><<<P, 256, 0, s>>>(g, k, y[b], y[a], p[b], p[a]);
    else if (d <= 1024)
      trd_step_kernel<1024, 512, 4><<<P, 512, 0, s>>>(g, k, y[b], y[a], p[b], p[a]);
    else if (d <= 2048)
      trd_step_kernel<2048, 512, 8><<<P, 512, 0, s>>>(g, k, y[b], y[a], p[b], p[a]);
    else
      trd_step_wide_kernel<8192, 1024><<<P, 1024, 0, s>>>(g, k, y[b], y[a], p[b], p[a]);
  }
  trd_tail_kernel<<<1, 64 * kTailWaves, 0, s>>>(g, k0, y[(k0 & 1) ^ 1]);
  return hipGetLastError();
}

hipError_t launch_tri_eigvals(int n, const EighWork& w, double* lam, hipStream_t s) {
  const int d = 1 << n;
  TriScal* ts = static_cast<TriScal*>(w.scal);
  tri_split_kernel<<<1, 256, 0, s>>>(w.diag, w.off, d, w.bstart, w.bend, ts);
  if (d <= 2048)
    tri_eigvals_kernel<2048><<<(d + 3) / 4, 256, 0, s>>>(w.diag, w.off, d, w.bstart, w.bend, ts, lam);
  else
    tri_eigvals_kernel<8192><<<(d + 3) / 4, 256, 0, s>>>(w.diag, w.off, d, w.bstart, w.bend, ts, lam);
  return hipGetLastError();
}

hipError_t launch_tri_vectors(int n, const EighWork& w, const double* lam, void* scratch, void* Z, hipStream_t s) {
  const int d = 1 << n;
  const int64_t count = int64_t(d) * d;
  const TriScal* ts = static_cast<const TriScal*>(w.scal);
  zero_kernel<<<unsigned((count + 255) / 256), 256, 0, s>>>(static_cast<C64*>(Z), count);
  if (d <= 2048)
    tri_vectors_kernel<2048><<<(d + 63) / 64, 128, 0, s>>>(w.diag, w.off, d, w.bstart, w.bend, ts, lam,
                                                          static_cast<double*>(scratch), static_cast<C64*>(Z));
  else
    tri_vectors_kernel<8192><<<(d + 63) / 64, 128, 0, s>>>(w.diag, w.off, d, w.bstart, w.bend, ts, lam,
                                                          static_cast<double*>(scratch), static_cast<C64*>(Z));
  tri_cluster_kernel<<<d, 64, 0, s>>>(w.diag, w.off, d, w.bstart, w.bend, ts, lam, static_cast<double*>(scratch),
                                      static_cast<C64*>(Z));
  return hipGetLastError();
}

hipError_t launch_ns_matrix(int n, const void* G, void* M, hipStream_t s) {
  const int64_t count = int64_t(1) << (2 * n);
  ns_matrix_kernel<<<unsigned((count + 255) / 256), 256, 0, s>>>(static_cast<const C64*>(G), static_cast<C64*>(M), n);
  return hipGetLastError();
}

hipError_t launch_back_transform(int n, const void* V, const EighWork& w, void* Z, void* Wbuf, hipStream_t s) {
  const int d = 1 << n;
  const int blocks = (d - 1 + kNb - 1) / kNb;
  const C64* v = static_cast<const C64*>(V);
  C64* T = static_cast<C64*>(w.tfac);
  C64* Wm = static_cast<C64*>(Wbuf);
  C64* P = static_cast<C64*>(w.pbuf);
  const int gchunks = eigh_gram_chunks(d);
  bt_gram_kernel<<<dim3(blocks, gchunks), 256, 0, s>>>(v, d, gchunks, P);
  bt_tmat_kernel<<<blocks, 256, 0, s>>>(P, gchunks, static_cast<const C64*>(w.tau), d, T);
  bt_wfactor_kernel<<<dim3(blocks, unsigned((d + 63) / 64)), 256, 0, s>>>(v, T, d, Wm);
  const int R = eigh_chunk_rows(d);
  const unsigned ct = unsigned((d + 63) / 64);
  const unsigned sum_blocks = unsigned((int64_t(kNb) * d + 255) / 256);
  for (int b = blocks - 1; b >= 0; --b) {
    const int k0 = b * kNb, nk = d - 1 - k0 < kNb ? d - 1 - k0 : kNb;
    const int m = d - 1 - k0;  // rows k0 + 1 .. d - 1
    const int chunks = (m + R - 1) / R;
    bt_partial_kernel<<<dim3(ct, chunks, 2), 256, 0, s>>>(v, static_cast<const C64*>(Z), d, k0, nk, R, P);
    bt_sum_kernel<<<sum_blocks, 256, 0, s>>>(P, chunks, d, static_cast<C64*>(w.xbuf));
    bt_update_kernel<<<dim3(ct, unsigned((m + kUpdRows - 1) / kUpdRows)), 256, 0, s>>>(Wm, static_cast<const C64*>(w.xbuf), d, k0,
                                                                       nk, static_cast<C64*>(Z));
  }
  return hipGetLastError();
}

hipError_t launch_eigh_status(const EighWork& w, int* out, hipStream_t s) {
  status_out_kernel<<<1, 1, 0, s>>>(static_cast<const TriScal*>(w.scal), out);
  return hipGetLastError();
}

}  // namespace qst
