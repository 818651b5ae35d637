// Fidelity of the reconstructed state (Sec. 2.3).
//
// Quantum fidelity against a target of low rank r (Eq. F_QF):
//   F_q = (Tr sqrt(sqrt(rho_hat) rho sqrt(rho_hat)))^2,
//   rho_hat = T T^dagger / tau,  rho = W W^dagger / tw,  W d x r.
// sqrt(rho_hat) rho sqrt(rho_hat) has the nonzero eigenvalues of the r x r
// matrix C = M M^dagger / (tau tw), M = W^dagger T (r x d), so
// F_q = (sum_i sqrt(lambda_i(C)))^2.  Four launches:
//   1. fid_partial_kernel: M over row blocks of T (FP64 sums; also the
//      partial sums of |T|^2 for tau and of |W|^2 for tw) -- reads T once per
//      8 or 16 target columns;
//   2. fid_mreduce_kernel: M from the row-block sums, in order;
//   3. fid_gram_kernel: C_ab = sum_j M_aj conj(M_bj), one workgroup per pair;
//   4. fid_jacobi_kernel: tau, tw, C scaled by its trace, parallel cyclic Jacobi
//      eigenvalues of the Hermitian C (FP64, one workgroup), F_q.
// Classical fidelity (Eq. F_CF): F_c = (sum_k sqrt(p_hat_k p_k))^2 (negative
// entries read as 0), a two-stage FP64 reduction.
// Every sum has a fixed order: results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <cfloat>

#include "qst_device.h"
#include "qst_kernels.h"
#include "qst_plan.h"

namespace qst {

namespace {

constexpr int kRowChunk = 64;
constexpr int kRowGroup = 8;

struct Zd {
  double re, im;
};

// Workgroup (cb, rb): columns cb*64 .. +63 of T (fewer when d < 64), rows
// rb*RB .. (rb+1)*RB - 1.  Thread t: column c = t & 63, row quarter
// q = t >> 6 (rows i0 + q, i0 + q + 4, ... of each 64-row chunk).  For each
// chunk of AC target columns a0.., W's rows of the chunk are staged in LDS
// and every thread adds conj(W_ia) T_ij over its rows; the quarters are
// summed in order and P[rb][a][j] written.  In the first pass the thread
// also sums |T_ij|^2 (tau), written per workgroup to taup[rb * ncb + cb];
// the workgroups of column block 0 also sum |W|^2 of their rows (twp[rb]).
// AC target columns per pass over T (8 for ranks up to 8, else 16).
template <typename R, int AC>
__global__ __launch_bounds__(256) void fid_partial_kernel(const Cx<R>* __restrict__ T, int64_t ldT,
                                                          const Cx<R>* __restrict__ W, int64_t ldW, int r, int d,
                                                          int RB, Zd* __restrict__ P, double* __restrict__ taup,
                                                          double* __restrict__ twp) {
  __shared__ Zd wl[kRowChunk][AC];
  __shared__ Zd red[3][64][AC];
  __shared__ double rtau[4];
  const int ncb = d < 64 ? 1 : d / 64;
  const int cb = blockIdx.x % ncb, rb = blockIdx.x / ncb;
  const int t = threadIdx.x, c = t & 63, q = t >> 6;
  const int64_t j = int64_t(cb) * 64 + c;
  const bool col = j < d;
  const int64_t r0 = int64_t(rb) * RB;
  const int chunk = RB < kRowChunk ? RB : kRowChunk;
  double tsum = 0.0, wsum = 0.0;
  for (int a0 = 0; a0 < r; a0 += AC) {
    Zd acc[AC];
#pragma unroll
    for (int a = 0; a < AC; ++a) acc[a] = Zd{0.0, 0.0};
    for (int i0 = 0; i0 < RB; i0 += chunk) {
      __syncthreads();  // the previous chunk's W is no longer read
      for (int e = t; e < chunk * AC; e += 256) {
        const int ii = e / AC, a = e % AC;
        Cx<R> w{R(0), R(0)};
        if (a0 + a < r) w = W[(r0 + i0 + ii) * ldW + a0 + a];
        wl[ii][a] = Zd{double(w.re), double(w.im)};
        wsum += double(w.re) * double(w.re) + double(w.im) * double(w.im);
      }
      __syncthreads();
      if (col) {
        // kRowGroup rows of T loaded before any is used (one memory round
        // trip per group); rows past the chunk are clamped and dropped
        for (int g0 = q; g0 < chunk; g0 += 4 * kRowGroup) {
          Cx<R> xg[kRowGroup];
#pragma unroll
          for (int u = 0; u < kRowGroup; ++u) {
            const int ii = g0 + 4 * u < chunk ? g0 + 4 * u : q;
            xg[u] = T[(r0 + i0 + ii) * ldT + j];
          }
#pragma unroll
          for (int u = 0; u < kRowGroup; ++u) {
            const int ii = g0 + 4 * u;
            if (ii >= chunk) break;
            const double xr = double(xg[u].re), xi = double(xg[u].im);
            if (a0 == 0) tsum += xr * xr + xi * xi;
#pragma unroll
            for (int a = 0; a < AC; ++a) {
              const double wr = wl[ii][a].re, wi = wl[ii][a].im;
              // conj(w) x
              acc[a].re += wr * xr + wi * xi;
              acc[a].im += wr * xi - wi * xr;
            }
          }
        }
      }
    }
    // quarters 1..3 hand their sums to quarter 0, which adds them in order
    __syncthreads();
    if (q > 0) {
#pragma unroll
      for (int a = 0; a < AC; ++a) red[q - 1][c][a] = acc[a];
    }
    __syncthreads();
    if (q == 0 && col) {
#pragma unroll
      for (int a = 0; a < AC; ++a) {
        Zd s = acc[a];
        for (int k = 0; k < 3; ++k) {
          s.re += red[k][c][a].re;
          s.im += red[k][c][a].im;
        }
        if (a0 + a < r) P[(int64_t(rb) * r + a0 + a) * d + j] = s;
      }
    }
  }
  const double ts = block_sum256(tsum, rtau);
  if (t == 0) taup[blockIdx.x] = ts;
  if (cb == 0) {
    const double wsm = block_sum256(wsum, rtau);
    if (t == 0) twp[rb] = wsm;
  }
}

// M_aj = sum_rb P[rb][a][j] (row blocks in order), one entry per thread.
__global__ __launch_bounds__(256) void fid_mreduce_kernel(const Zd* __restrict__ P, int nrb, int r, int d,
                                                          Zd* __restrict__ M) {
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= int64_t(r) * d) return;
  double sr = 0.0, si = 0.0;
  for (int k = 0; k < nrb; ++k) {
    const Zd x = P[int64_t(k) * r * d + e];
    sr += x.re;
    si += x.im;
  }
  M[e] = Zd{sr, si};
}

// C_ab = sum_j M_aj conj(M_bj); workgroup b handles the lower pair
// (a, b) = tri_decode(b) and writes C_ab and C_ba.
__global__ __launch_bounds__(256) void fid_gram_kernel(const Zd* __restrict__ M, int r, int d, Zd* __restrict__ C) {
  __shared__ double red[4];
  int a, b;
  tri_decode(blockIdx.x, a, b);
  double sr = 0.0, si = 0.0;
  for (int j = threadIdx.x; j < d; j += 256) {
    const Zd x = M[int64_t(a) * d + j], y = M[int64_t(b) * d + j];
    sr += x.re * y.re + x.im * y.im;
    si += x.im * y.re - x.re * y.im;
  }
  sr = block_sum256(sr, red);
  si = block_sum256(si, red);
  if (threadIdx.x == 0) {
    C[a * r + b] = Zd{sr, si};
    C[b * r + a] = Zd{sr, -si};
  }
}

// tau and tw (the workgroup partials, in order), then the eigenvalues of
// C 2^-e, e the exponent of Tr C (a power of two: 1 / Tr C overflows for a
// trace below 5.6e-309), by parallel cyclic Jacobi and F_q = 2^e / (tau tw)
// (sum_i sqrt(lambda_i))^2; 0 where that sum is 0, for T or W of zeros too, or
// not finite.  A sweep takes the r(r-1)/2 pairs in r' - 1 steps of
// r'/2 disjoint pairs (round-robin order, r' = r rounded up to even; pairs
// with the padding index are not rotated).  The rotation of a pair (p, q)
// with c = C_pq, h = (C_qq - C_pp) / 2 and g = 1 / sqrt(h^2 + |c|^2):
// cs^2 = (1 + |h| g) / 2, sn e = sign(h) c g / (2 cs) with e = c / |c|, and the
// unitary G with G_pp = G_qq = cs, G_pq = sn e, G_qp = -sn conj(e):
// C <- G^dagger C G zeroes C_pq.  The rotations of one step touch disjoint
// rows and columns, so a step is the 2 x 2 blocks G_k^dagger C_kl G_l of its
// pairs (k, l), one thread each, with the two rotations formed by the thread
// itself.  Sweeps stop when the off-diagonal mass is below 1e-30 of the
// diagonal's, or after 40.
//
// Bound by the chain of each step (two reciprocal square roots and the LDS
// round trip; r <= 16 runs in one wave, whose barriers are free): 8 sweeps of
// 7 steps at r = 8.  Rotations formed by one thread per pair with divisions,
// columns and rows updated between barriers, and tw summed here: 67 us; now 38.
struct Rot {
  double cs, sr, si;  // cs, sn e
};
__device__ __forceinline__ Rot fid_rotation(Zd c, double dp, double dq) {
  const double a = c.re * c.re + c.im * c.im;
  if (!(a > 0.0)) return Rot{1.0, 0.0, 0.0};
  const double h = 0.5 * (dq - dp);
  const double g = rsqrt(h * h + a);
  const double c2 = 0.5 + 0.5 * fabs(h) * g;
  const double rc = rsqrt(c2);
  const double f = (h >= 0.0 ? 0.5 : -0.5) * g * rc;
  return Rot{c2 * rc, f * c.re, f * c.im};
}
template <int NT>
__global__ __launch_bounds__(NT) void fid_jacobi_kernel(const double* __restrict__ taup, int ntaup,
                                                        const double* __restrict__ twp, int ntw, int r,
                                                        const Zd* __restrict__ Cin, double* __restrict__ F) {
  constexpr int RM = NT == 64 ? 16 : kFidelityMaxRank;
  __shared__ Zd C[RM][RM + 1];
  __shared__ double mass[2][NT];
  const int t = threadIdx.x;
  // tau in lane order of one wave, tw and the trace by every thread
  double tau = 0.0, tw = 0.0, tr = 0.0;
  if (t < 64) {
    for (int k = t; k < ntaup; k += 64) tau += taup[k];
    tau = wave_sum(tau);
  }
  for (int k = 0; k < ntw; ++k) tw += twp[k];
  for (int k = 0; k < r; ++k) tr += Cin[k * r + k].re;
  const bool finite = tr <= DBL_MAX;
  const int ex = tr > 0.0 && finite ? __builtin_amdgcn_frexp_exp(tr) : 0;
  for (int e = t; e < r * r; e += NT) {
    const Zd v = Cin[e];
    C[e / r][e % r] = Zd{ldexp(v.re, -ex), ldexp(v.im, -ex)};
  }
  __syncthreads();
  const int rp = r + (r & 1), np = rp / 2;
  const int k = t / np, l = t % np;
  const bool act = t < np * np;
  for (int sweep = 0; sweep < 40; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int e = t; e < r * r; e += NT) {
      const Zd v = C[e / r][e % r];
      const double m = v.re * v.re + v.im * v.im;
      if (e / r == e % r) diag += m;
      else off += m;
    }
    if constexpr (NT == 64) {
      off = wave_sum(off);
      diag = wave_sum(diag);
    } else {
      mass[0][t] = off;
      mass[1][t] = diag;
      __syncthreads();
      off = diag = 0.0;
      for (int i = 0; i < NT; i += 64) {
        off += mass[0][i + (t & 63)];
        diag += mass[1][i + (t & 63)];
      }
      off = wave_sum(off);
      diag = wave_sum(diag);
    }
    if (off == 0.0 || off <= 1e-30 * diag) break;  // the same value in every thread
    for (int step = 0; step < rp - 1; ++step) {
      // round-robin positions u and rp - 1 - u; position 0 stays
      auto pair = [&](int u, int& p, int& q) {
        const int m = rp - 1, xu = u - 1 + step, xv = m - u - 1 + step;  // below 2 m
        const int iu = u == 0 ? 0 : (xu >= m ? xu - m : xu) + 1;
        const int iv = (xv >= m ? xv - m : xv) + 1;
        p = iu < iv ? iu : iv;
        q = iu < iv ? iv : iu;
      };
      int pk, qk, pl, ql;
      pair(k, pk, qk);
      pair(l, pl, ql);
      Zd a[2][2];
      Rot G{1.0, 0.0, 0.0}, H{1.0, 0.0, 0.0};
      const bool rk = act && qk < r, rl = act && ql < r;
      if (act) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int x = i ? qk : pk, y = j ? ql : pl;
            a[i][j] = (x < r && y < r) ? C[x][y] : Zd{0.0, 0.0};
          }
        if (rk) G = fid_rotation(C[pk][qk], C[pk][pk].re, C[qk][qk].re);
        if (rl) H = fid_rotation(C[pl][ql], C[pl][pl].re, C[ql][ql].re);
      }
      __syncthreads();
      if (act) {
        Zd b[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {  // columns: (cs cp - sn conj(e) cq, sn e cp + cs cq)
          const Zd cp = a[i][0], cq = a[i][1];
          b[i][0] = Zd{H.cs * cp.re - (H.sr * cq.re + H.si * cq.im), H.cs * cp.im - (H.sr * cq.im - H.si * cq.re)};
          b[i][1] = Zd{(H.sr * cp.re - H.si * cp.im) + H.cs * cq.re, (H.sr * cp.im + H.si * cp.re) + H.cs * cq.im};
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {  // rows: (cs rp - sn e rq, sn conj(e) rp + cs rq)
          const Zd x = b[0][j], y = b[1][j];
          a[0][j] = Zd{G.cs * x.re - (G.sr * y.re - G.si * y.im), G.cs * x.im - (G.sr * y.im + G.si * y.re)};
          a[1][j] = Zd{(G.sr * x.re + G.si * x.im) + G.cs * y.re, (G.sr * x.im - G.si * x.re) + G.cs * y.im};
        }
        // the rotated pair's own off-diagonal entries are zero by construction
        if (k == l && rk) a[0][1] = a[1][0] = Zd{0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int x = i ? qk : pk, y = j ? ql : pl;
            if (x < r && y < r) C[x][y] = a[i][j];
          }
      }
      __syncthreads();
    }
  }
  if (t == 0) {
    double sq = 0.0;
    for (int i = 0; i < r; ++i) sq += sqrt(fmax(C[i][i].re, 0.0));
    *F = finite && sq > 0.0 ? ldexp(sq * sq, ex) / (tau * tw) : 0.0;
  }
}

// F_c stage 1: block b sums sqrt(max(p_hat,0) max(p,0)) over its range.
template <typename R>
__global__ __launch_bounds__(256) void fid_classical_partial_kernel(const R* __restrict__ ph, const R* __restrict__ p,
                                                                    int64_t D, double* __restrict__ partials) {
  __shared__ double red[4];
  const int nb = gridDim.x;
  const int64_t chunk = (D + nb - 1) / nb;
  const int64_t beg = int64_t(blockIdx.x) * chunk;
  const int64_t end = beg + chunk < D ? beg + chunk : D;
  constexpr int U = 8;
  double s = 0.0;
  for (int64_t k0 = beg + threadIdx.x; k0 < end; k0 += U * int64_t(blockDim.x)) {
    R a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + u * int64_t(blockDim.x);
      const bool in = k < end;
      a[u] = in ? ph[k] : R(0);
      b[u] = in ? p[k] : R(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += sqrt(fmax(double(a[u]), 0.0) * fmax(double(b[u]), 0.0));
  }
  s = block_sum256(s, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void fid_classical_finish_kernel(const double* __restrict__ partials, int nb,
                                                                   double* __restrict__ F) {
  __shared__ double red[4];
  const double s = sum_partials256(partials, nb, red);
  if (threadIdx.x == 0) *F = s * s;
}

template <typename R>
hipError_t run_fidelity_lowrank(const void* T, int64_t ldT, const void* W, int64_t ldW, int r, int n, void* ws,
                                double* F, hipStream_t s) {
  const FidelityLayout fl = fidelity_layout(n);
  const int d = 1 << n;
  unsigned char* base = static_cast<unsigned char*>(ws);
  Zd* P = reinterpret_cast<Zd*>(base + fl.mpart);
  Zd* C = reinterpret_cast<Zd*>(base + fl.gram);
  double* taup = reinterpret_cast<double*>(base + fl.taup);
  double* twp = reinterpret_cast<double*>(base + fl.twp);
  const int ncb = d < 64 ? 1 : d / 64;
  if (r <= 8)
    fid_partial_kernel<R, 8><<<unsigned(ncb * fl.nrb), 256, 0, s>>>(static_cast<const Cx<R>*>(T), ldT,
                                                                    static_cast<const Cx<R>*>(W), ldW, r, d,
                                                                    d / fl.nrb, P, taup, twp);
  else
    fid_partial_kernel<R, 16><<<unsigned(ncb * fl.nrb), 256, 0, s>>>(static_cast<const Cx<R>*>(T), ldT,
                                                                     static_cast<const Cx<R>*>(W), ldW, r, d,
                                                                     d / fl.nrb, P, taup, twp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  Zd* M = reinterpret_cast<Zd*>(base + fl.mrow);
  fid_mreduce_kernel<<<unsigned((int64_t(r) * d + 255) / 256), 256, 0, s>>>(P, fl.nrb, r, d, M);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  fid_gram_kernel<<<unsigned(r * (r + 1) / 2), 256, 0, s>>>(M, r, d, C);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (r <= 16) fid_jacobi_kernel<64><<<1, 64, 0, s>>>(taup, ncb * fl.nrb, twp, fl.nrb, r, C, F);
  else fid_jacobi_kernel<256><<<1, 256, 0, s>>>(taup, ncb * fl.nrb, twp, fl.nrb, r, C, F);
  return hipGetLastError();
}

template <typename R>
hipError_t run_fidelity_classical(const void* ph, const void* p, int n, double* part, double* F, hipStream_t s) {
  fid_classical_partial_kernel<R><<<kReduceBlocks, 256, 0, s>>>(static_cast<const R*>(ph), static_cast<const R*>(p),
                                                                int64_t(1) << (2 * n), part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  fid_classical_finish_kernel<<<1, 256, 0, s>>>(part, kReduceBlocks, F);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fidelity_lowrank(qst_prec prec, const void* T, int64_t ldT, const void* W, int64_t ldW, int r,
                                   int n, void* ws, double* F, hipStream_t s) {
  if (prec == QST_F64) return run_fidelity_lowrank<double>(T, ldT, W, ldW, r, n, ws, F, s);
  return run_fidelity_lowrank<float>(T, ldT, W, ldW, r, n, ws, F, s);
}

hipError_t launch_fidelity_classical(qst_prec prec, const void* ph, const void* p, int n, void* ws, double* F,
                                     hipStream_t s) {
  double* part = reinterpret_cast<double*>(static_cast<unsigned char*>(ws) + fidelity_layout(n).cpart);
  return launch_fidelity_classical_part(prec, ph, p, n, part, F, s);
}

hipError_t launch_fidelity_classical_part(qst_prec prec, const void* ph, const void* p, int n, double* part, double* F,
                                          hipStream_t s) {
  if (prec == QST_F64) return run_fidelity_classical<double>(ph, p, n, part, F, s);
  return run_fidelity_classical<float>(ph, p, n, part, F, s);
}

}  // namespace qst
