// General product POVMs: K outcomes per qubit, a K-element POVM of its own
// on each qubit (Sec. 3.3), and several such settings whose negative
// log-likelihoods add (Sec. 2.1: one POVM {M^i_k} per measurement i).
//
// Route through the Pauli coordinates.  Every 2 x 2 Hermitian M is
// M = sum_b C[b] P_b over the Pauli basis P = (I, X, Y, Z) with real
// C[b] = Tr(M P_b) / 2, so for a product POVM
//   p_k = Tr((M^(1)_k1 (x) ... (x) M^(N)_kN) rho) = sum_b prod_i C^(i)[k_i][b_i] e_b,
//   e_b = Tr((P_b1 (x) ... (x) P_bN) rho)   (4^N real Pauli coordinates),
// i.e. p = (C^(1) (x) ... (x) C^(N)) e.  e comes from the product-POVM
// passes run with the Pauli matrices in place of POVM elements (the passes
// take any Hermitian four-element set; only the lower triangle of rho is
// read), and the real K x 4 factors are applied to a group of consecutive
// qubits per launch (factor_pass: the group's 4^Q inputs and K^Q outputs in
// registers).  The last forward group, the NLL terms, the cotangent
// F_s - f_k / p_k and the first adjoint group are one kernel (factor_fused):
// a thread holds the K^Q probabilities whose cotangents its adjoint needs,
// so p is never stored and f read once (and once more before, for F_s).
// The settings' adjoints are summed into one 4^N vector h in the last
// adjoint group, and the Pauli synthesis G' = sum_b h_b P_b is the adjoint
// passes'.
//
// Tensor layout of a real pass over a group: [A][m][B] with A = 4^(qubits
// before the group, still in Pauli coordinates), m the group's index (4^Q
// Pauli coordinates or K^Q outcomes, its first qubit most significant) and
// B = K^(qubits after it, finished); the flat outcome index is
// k = sum_i k_i K^(N-i), qubit N least significant.
//
// What bounds it: HBM for many outcomes (Pauli-6 at N = 10), the launches for
// few (two outcomes per qubit).  Pauli-6 at N = 10: the forward groups 60 us
// and the adjoint ones 59 us (267 MB each, 4.5 TB/s), F_s 63 us (242 MB,
// 3.8 TB/s), the fused group 96 us (457 MB, 4.8 TB/s); one qubit per launch
// with p stored took 593 us.  Three Pauli bases at N = 11: 21 launches, 121
// us; one qubit per launch took 69 and 290 us.
#include <algorithm>
#include <vector>

#include "qst_device.h"
#include "qst_kernels.h"
#include "qst_plan.h"

namespace qst {

namespace {

// Qubits per group, at most, as measured with three settings (two against
// three qubits).  K = 3: FP32 N = 11 628 against 606 us, FP64 N = 9 298 against
// 318, so neither way by much.  K = 4: FP64 N = 9 311 against 479 us (64 inputs
// and 64 outputs spill), FP32 N = 11 735 against 762.  K >= 5: three would be
// 125 outputs and more, past a thread's registers.
constexpr int max_group(int K) { return K == 2 ? 3 : 2; }

template <typename R, int K, int Q>
struct Factors {
  R c[Q][K][4];  // [qubit of the group, first most significant][k][b]
};

constexpr int cpow(int x, int e) { return e == 0 ? 1 : x * cpow(x, e - 1); }

// The transform of one group in registers, one qubit at a time.  Forward: x
// holds [4]^Q; qubit q turns its index from 4 to K.  Values live in buffers
// of cpow(max(4, K), Q).
template <typename R, int K, int Q>
__device__ __forceinline__ void group_fwd(const Factors<R, K, Q>& C, const R (&x)[cpow(4, Q)], R (&y)[cpow(K, Q)]) {
  if constexpr (Q == 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      R v = R(0);
#pragma unroll
      for (int b = 0; b < 4; ++b) v += C.c[0][k][b] * x[b];
      y[k] = v;
    }
  } else {
    // the first qubit's 4 slices, each transformed by the rest, then mixed
    constexpr int NI = cpow(4, Q - 1), NO = cpow(K, Q - 1);
    Factors<R, K, Q - 1> rest;
#pragma unroll
    for (int q = 1; q < Q; ++q)
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int b = 0; b < 4; ++b) rest.c[q - 1][k][b] = C.c[q][k][b];
#pragma unroll
    for (int i = 0; i < K * NO; ++i) y[i] = R(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      R xs[NI], ys[NO];
#pragma unroll
      for (int i = 0; i < NI; ++i) xs[i] = x[b * NI + i];
      group_fwd<R, K, Q - 1>(rest, xs, ys);
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < NO; ++i) y[k * NO + i] += C.c[0][k][b] * ys[i];
    }
  }
}
// Adjoint: [K]^Q -> [4]^Q with the transposed factors.
template <typename R, int K, int Q>
__device__ __forceinline__ void group_adj(const Factors<R, K, Q>& C, const R (&y)[cpow(K, Q)], R (&x)[cpow(4, Q)]) {
  if constexpr (Q == 1) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      R v = R(0);
#pragma unroll
      for (int k = 0; k < K; ++k) v += C.c[0][k][b] * y[k];
      x[b] = v;
    }
  } else {
    constexpr int NI = cpow(4, Q - 1), NO = cpow(K, Q - 1);
    Factors<R, K, Q - 1> rest;
#pragma unroll
    for (int q = 1; q < Q; ++q)
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int b = 0; b < 4; ++b) rest.c[q - 1][k][b] = C.c[q][k][b];
#pragma unroll
    for (int i = 0; i < 4 * NI; ++i) x[i] = R(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      R ys[NO], xs[NI];
#pragma unroll
      for (int i = 0; i < NO; ++i) ys[i] = y[k * NO + i];
      group_adj<R, K, Q - 1>(rest, ys, xs);
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < NI; ++i) x[b * NI + i] += C.c[0][k][b] * xs[i];
    }
  }
}

// NV values of every thread from or to NV consecutive elements each (B = 1,
// where a thread's elements are contiguous and neighbouring threads' are
// not): through LDS rows of NV | 1 elements, so that global accesses are
// coalesced and the row accesses spread over the banks.  A full block (NT
// rows) moves U elements per thread at a time, all in flight together.
template <typename R, int NV, int NT>
__device__ __forceinline__ void rows_in(const R* __restrict__ g, int rows, R* lds, R (&x)[NV]) {
  constexpr int LD = NV | 1, U = NV % 16 == 0 ? 16 : NV % 9 == 0 ? 9 : NV % 8 == 0 ? 8 : NV % 7 == 0 ? 7 : NV % 5 == 0 ? 5 : NV;
  static_assert(NV % U == 0, "whole batches");
  const int th = threadIdx.x;
  if (rows == NT) {
    for (int i0 = 0; i0 < NV; i0 += U) {
      R v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = g[(i0 + u) * NT + th];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = (i0 + u) * NT + th;
        lds[(e / NV) * LD + e % NV] = v[u];
      }
    }
  } else {
    for (int e = th; e < rows * NV; e += NT) lds[(e / NV) * LD + e % NV] = g[e];
  }
  __syncthreads();
  if (th < rows) {
#pragma unroll
    for (int i = 0; i < NV; ++i) x[i] = lds[th * LD + i];
  }
  __syncthreads();
}
template <typename R, int NV, int NT>
__device__ __forceinline__ void rows_out(R* __restrict__ g, int rows, R* lds, const R (&x)[NV], bool accumulate) {
  constexpr int LD = NV | 1, U = NV % 16 == 0 ? 16 : NV % 9 == 0 ? 9 : NV % 8 == 0 ? 8 : NV % 7 == 0 ? 7 : NV % 5 == 0 ? 5 : NV;
  const int th = threadIdx.x;
  if (th < rows) {
#pragma unroll
    for (int i = 0; i < NV; ++i) lds[th * LD + i] = x[i];
  }
  __syncthreads();
  if (rows == NT) {
    for (int i0 = 0; i0 < NV; i0 += U) {
      R v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = accumulate ? g[(i0 + u) * NT + th] : R(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = (i0 + u) * NT + th;
        g[e] = v[u] + lds[(e / NV) * LD + e % NV];
      }
    }
  } else {
    for (int e = th; e < rows * NV; e += NT) {
      R v = lds[(e / NV) * LD + e % NV];
      if (accumulate) v += g[e];
      g[e] = v;
    }
  }
  __syncthreads();
}

// Threads of a pass over a group: as many as keep the LDS rows of B = 1
// within 64 KiB.
template <typename R, int NV>
constexpr int pass_threads() {
  constexpr size_t row = sizeof(R) * (NV | 1);
  static_assert(row * 64 <= 65536, "a wave's rows fit");
  return row * 256 <= 65536 ? 256 : row * 128 <= 65536 ? 128 : 64;
}
template <typename R, int K, int Q>
constexpr int group_vals() {
  return cpow(K > 4 ? K : 4, Q);
}

// ADJ 0: [A][4^Q][B] -> [A][K^Q][B]; ADJ 1: back, out (+)= .
template <typename R, int K, int Q, bool ADJ>
__global__ __launch_bounds__((pass_threads<R, group_vals<R, K, Q>()>())) void factor_pass(
    const R* __restrict__ in, R* __restrict__ out, uint32_t total, uint32_t B, Factors<R, K, Q> C, int accumulate) {
  constexpr int NP = cpow(4, Q), NK = cpow(K, Q), MI = ADJ ? NK : NP, MO = ADJ ? NP : NK;
  constexpr int NT = pass_threads<R, group_vals<R, K, Q>()>();
  extern __shared__ __align__(16) char factor_lds[];
  R* lds = reinterpret_cast<R*>(factor_lds);
  for (uint32_t t0 = blockIdx.x * NT; t0 < total; t0 += gridDim.x * NT) {
    const uint32_t t = t0 + threadIdx.x;
    const int rows = total - t0 < uint32_t(NT) ? int(total - t0) : NT;
    const uint32_t a = t / B, b = t - a * B;
    const int64_t ib = int64_t(a) * MI * B + b, ob = int64_t(a) * MO * B + b;
    R x[MI], y[MO];
    if (B == 1) {
      rows_in<R, MI, NT>(in + int64_t(t0) * MI, rows, lds, x);
    } else if (t < total) {
#pragma unroll
      for (int m = 0; m < MI; ++m) x[m] = in[ib + int64_t(m) * B];
    }
    if constexpr (ADJ) group_adj<R, K, Q>(C, x, y);
    else group_fwd<R, K, Q>(C, x, y);
    if (B == 1) {
      rows_out<R, MO, NT>(out + int64_t(t0) * MO, rows, lds, y, accumulate != 0);
    } else if (t < total) {
#pragma unroll
      for (int o = 0; o < MO; ++o) {
        R v = y[o];
        if (accumulate) v += out[ob + int64_t(o) * B];
        out[ob + int64_t(o) * B] = v;
      }
    }
  }
}

// The last forward group (A = 1: every earlier qubit finished), the NLL
// terms of its outcomes, the cotangents and the first adjoint group:
// in [4^Q][B] -> out [4^Q][B] (NULL: the terms only; += with accumulate,
// where this group is also the last).  part: [4][gridDim.x] FP64 partials
// (L, unused, f > 0 with p <= 0, NaN); *Fs: F_s.
template <typename R, int K, int Q>
__global__ __launch_bounds__(256) void factor_fused(const R* __restrict__ in, R* __restrict__ out, uint32_t B,
                                                    Factors<R, K, Q> C, const R* __restrict__ f,
                                                    const double* __restrict__ Fs, double* __restrict__ part,
                                                    int accumulate) {
  constexpr int NP = cpow(4, Q), NK = cpow(K, Q);
  __shared__ double red[4];
  const double F = *Fs;
  double L = 0.0, bad0 = 0.0, bad1 = 0.0;
  for (uint32_t b = blockIdx.x * 256 + threadIdx.x; b < B; b += gridDim.x * 256) {
    R x[NP], y[NK], fr[NK];
#pragma unroll
    for (int m = 0; m < NP; ++m) x[m] = in[int64_t(m) * B + b];
#pragma unroll
    for (int k = 0; k < NK; ++k) fr[k] = f[int64_t(k) * B + b];
    group_fwd<R, K, Q>(C, x, y);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const double fk = double(fr[k]), pk = double(y[k]);
      if (fk != 0.0) {
        if (pk > 0.0) L -= fk * ln_prob(y[k]);
        else bad0 += 1.0;
      }
      if (pk != pk || fk != fk) bad1 += 1.0;
      y[k] = cotangent(F, fr[k], y[k]);
    }
    if (!out) continue;
    group_adj<R, K, Q>(C, y, x);
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      R v = x[m];
      if (accumulate) v += out[int64_t(m) * B + b];
      out[int64_t(m) * B + b] = v;
    }
  }
  const int nb = gridDim.x;
  double v = block_sum256(L, red);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
  v = block_sum256(bad0, red);
  if (threadIdx.x == 0) part[2 * nb + blockIdx.x] = v;
  v = block_sum256(bad1, red);
  if (threadIdx.x == 0) part[3 * nb + blockIdx.x] = v;
}

// F_s partial sums: part[s * nb + chunk], blockIdx.y the setting.  Bound by
// HBM: 16-byte loads (f needs no more than its own alignment), eight in
// flight per thread; with 4-byte ones 242 MB took 112 us.
template <typename R>
__global__ __launch_bounds__(256) void settings_f_kernel(const R* __restrict__ f, int64_t DK, double* __restrict__ part) {
  __shared__ double red[4];
  constexpr int V = 16 / sizeof(R), U = 8;
  typedef R vec __attribute__((ext_vector_type(V), aligned(sizeof(R))));
  const int nb = gridDim.x;
  const int64_t beg = DK * blockIdx.x / nb, end = DK * (blockIdx.x + 1) / nb;
  const R* fs = f + int64_t(blockIdx.y) * DK;
  const int64_t nv = (end - beg) / V;  // whole vectors, then at most V - 1 elements
  double acc = 0.0;
  for (int64_t e0 = threadIdx.x; e0 < nv; e0 += 256 * U) {
    vec v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t e = e0 + 256 * u;
      v[u] = *reinterpret_cast<const vec*>(fs + beg + V * (e < nv ? e : nv - 1));
      if (e >= nv) v[u] = vec(R(0));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < V; ++i) acc += double(v[u][i]);
  }
  const int64_t rest = beg + nv * V + threadIdx.x;
  if (rest < end) acc += double(fs[rest]);
  acc = block_sum256(acc, red);
  if (threadIdx.x == 0) part[int64_t(blockIdx.y) * nb + blockIdx.x] = acc;
}
__global__ __launch_bounds__(256) void settings_f_finish_kernel(const double* __restrict__ part, int nb,
                                                                double* __restrict__ scal) {
  __shared__ double red[4];
  const double v = sum_partials256(part + int64_t(blockIdx.x) * nb, nb, red);
  if (threadIdx.x == 0) scal[4 * blockIdx.x + 1] = v;
}

int64_t ipow(int64_t x, int e) {
  int64_t r = 1;
  for (int i = 0; i < e; ++i) r *= x;
  return r;
}

// One group over qubits j .. j + Q - 1 (1-based) of a setting's factors C.
enum GroupMode { kFwd, kAdj, kFused };
struct GroupCall {
  GroupMode mode;
  int n, j;
  const double* C;
  const void* in;
  void* out;
  bool accumulate;
  const void* f;     // kFused
  const double* Fs;  // kFused
  double* part;      // kFused
  int nb;            // kFused: workgroups
};

template <typename R, int K, int Q>
hipError_t launch_group_q(const GroupCall& g, hipStream_t s) {
  Factors<R, K, Q> C;
  for (int q = 0; q < Q; ++q)
    for (int k = 0; k < K; ++k)
      for (int b = 0; b < 4; ++b) C.c[q][k][b] = R(g.C[(int64_t(g.j - 1 + q) * K + k) * 4 + b]);
  const int64_t A = ipow(4, g.j - 1), B = ipow(K, g.n - (g.j - 1 + Q));
  const R* in = static_cast<const R*>(g.in);
  R* out = static_cast<R*>(g.out);
  if (g.mode == kFused) {
    factor_fused<R, K, Q><<<unsigned(g.nb), 256, 0, s>>>(in, out, uint32_t(B), C, static_cast<const R*>(g.f), g.Fs,
                                                         g.part, g.accumulate ? 1 : 0);
    return hipGetLastError();
  }
  constexpr int NV = group_vals<R, K, Q>(), NT = pass_threads<R, NV>();
  const int64_t total = A * B;
  const unsigned blocks = unsigned(std::min<int64_t>((total + NT - 1) / NT, 8192));
  const size_t lds = B == 1 ? sizeof(R) * NT * (NV | 1) : 0;
  if (g.mode == kAdj)
    factor_pass<R, K, Q, true><<<blocks, NT, lds, s>>>(in, out, uint32_t(total), uint32_t(B), C, g.accumulate ? 1 : 0);
  else
    factor_pass<R, K, Q, false><<<blocks, NT, lds, s>>>(in, out, uint32_t(total), uint32_t(B), C, 0);
  return hipGetLastError();
}

template <typename R, int K>
hipError_t launch_group_k(int Q, const GroupCall& g, hipStream_t s) {
  if (Q == 1) return launch_group_q<R, K, 1>(g, s);
  if (Q == 2) return launch_group_q<R, K, 2>(g, s);
  if constexpr (max_group(K) >= 3) {
    if (Q == 3) return launch_group_q<R, K, 3>(g, s);
  }
  return hipErrorInvalidValue;
}

template <typename R>
hipError_t launch_group(int K, int Q, const GroupCall& g, hipStream_t s) {
  ProfScope prof("general_factor_pass", s);
  switch (K) {
    case 2: return launch_group_k<R, 2>(Q, g, s);
    case 3: return launch_group_k<R, 3>(Q, g, s);
    case 4: return launch_group_k<R, 4>(Q, g, s);
    case 5: return launch_group_k<R, 5>(Q, g, s);
    case 6: return launch_group_k<R, 6>(Q, g, s);
    case 7: return launch_group_k<R, 7>(Q, g, s);
    case 8: return launch_group_k<R, 8>(Q, g, s);
    default: return hipErrorInvalidValue;
  }
}

// Groups in forward order (qubits N down to 1): full ones of max_group(K)
// from the end, what is left over first, where the tensors of K > 4 are
// smallest; for K < 4, where they are largest, the full groups come first.
int make_groups(int n, int K, int* size) {
  const int m = max_group(K), rem = n % m;
  int g = 0;
  if (rem && K > 4) size[g++] = rem;
  for (int i = 0; i < n / m; ++i) size[g++] = m;
  if (rem && K <= 4) size[g++] = rem;
  return g;
}

// Stage 2 of one setting's NLL: scal[0], [2], [3] = (L_s, bad0_s, bad1_s)
// from the [4][nb] partials, in a fixed order (scal[1] holds F_s already).
__global__ __launch_bounds__(256) void setting_sums_kernel(const double* __restrict__ part, int nb,
                                                           double* __restrict__ scal) {
  __shared__ double red[4];
  for (int i = 0; i < 4; ++i) {
    if (i == 1) continue;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) acc += part[int64_t(i) * nb + b];
    const double v = block_sum256(acc, red);
    if (threadIdx.x == 0) scal[i] = v;
  }
}

// Totals over the settings, in setting order: nll = (L, F) with L = +inf
// after a term f_k > 0 with p_k <= 0 and NaN after a NaN, and the counters.
__global__ void settings_total_kernel(const double* __restrict__ scal, int settings, double* __restrict__ nll,
                                      unsigned long long* __restrict__ bad) {
  if (threadIdx.x != 0) return;
  double L = 0.0, F = 0.0, b0 = 0.0, b1 = 0.0;
  for (int s = 0; s < settings; ++s) {
    L += scal[4 * s];
    F += scal[4 * s + 1];
    b0 += scal[4 * s + 2];
    b1 += scal[4 * s + 3];
  }
  if (F != F || b1 > 0.0) L = __builtin_nan("");
  else if (b0 > 0.0) L = __builtin_inf();
  nll[0] = L;
  nll[1] = F;
  if (bad) {
    bad[0] = (unsigned long long)b0;
    bad[1] = (unsigned long long)b1;
  }
}

// Forward groups 0 .. stop - 1 of one setting from the Pauli coordinates e
// (ping-pong through bufA / bufB, the last of all groups into p); returns
// where the output of the last one run is.
template <typename R>
hipError_t forward_groups(int n, int K, const double* C, const int* size, int groups, int stop, const void* e, void* p,
                          void* const* bufs, const void** at, hipStream_t s) {
  const void* in = e;
  int end = n;  // the group covers qubits end - size + 1 .. end
  for (int g = 0; g < stop; ++g) {
    void* out = g == groups - 1 ? p : bufs[g & 1];
    const hipError_t err = launch_group<R>(
        K, size[g], GroupCall{kFwd, n, end - size[g] + 1, C, in, out, false, nullptr, nullptr, nullptr, 0}, s);
    if (err != hipSuccess) return err;
    in = out;
    end -= size[g];
  }
  *at = in;
  return hipSuccess;
}

// One setting: the forward groups, the fused last group (NLL partials) and,
// with h, the adjoint groups into h (+= for a later setting).
template <typename R>
hipError_t setting_likelihood(int n, int K, const double* C, const void* e, const void* f, double* sc, void* h,
                              bool accumulate, const GeneralBufs& b, hipStream_t s) {
  int size[QST_MAX_QUBITS];
  const int groups = make_groups(n, K, size);
  void* bufs[2] = {b.bufA, b.bufB};
  const void* in = nullptr;
  hipError_t err = forward_groups<R>(n, K, C, size, groups, groups - 1, e, nullptr, bufs, &in, s);
  if (err != hipSuccess) return err;
  // the fused group reads one buffer (or e) and writes the other, or h
  const int last = size[groups - 1];
  const int64_t B = ipow(K, n - last);
  const int nb = int(std::min<int64_t>((B + 255) / 256, kReduceBlocks));
  void* out = !h ? nullptr : groups == 1 ? h : bufs[(groups - 1) & 1];
  err = launch_group<R>(K, last, GroupCall{kFused, n, 1, C, in, out, groups == 1 && accumulate, f, sc + 1, b.partials, nb}, s);
  if (err != hipSuccess) return err;
  setting_sums_kernel<<<1, 256, 0, s>>>(b.partials, nb, sc);
  if ((err = hipGetLastError()) != hipSuccess || !h) return err;
  int first = 1 + last;
  for (int g = groups - 2; g >= 0; --g) {
    const void* from = out;
    out = g == 0 ? h : (from == bufs[0] ? bufs[1] : bufs[0]);
    err = launch_group<R>(K, size[g], GroupCall{kAdj, n, first, C, from, out, g == 0 && accumulate, nullptr, nullptr, nullptr, 0}, s);
    if (err != hipSuccess) return err;
    first += size[g];
  }
  return hipSuccess;
}

// F_s of every setting into scal[4 s + 1].
template <typename R>
hipError_t settings_f(const void* f, int settings, int64_t DK, const GeneralBufs& b, hipStream_t s) {
  // at most 4 kReduceBlocks partial sums in all, 64 per setting at least
  const int64_t nb = std::min<int64_t>(std::min<int64_t>(kReduceBlocks, 4 * kReduceBlocks / settings), (DK + 2047) / 2048);
  settings_f_kernel<R><<<dim3(unsigned(nb), unsigned(settings)), 256, 0, s>>>(static_cast<const R*>(f), DK, b.partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  settings_f_finish_kernel<<<unsigned(settings), 256, 0, s>>>(b.partials, int(nb), b.scal);
  return hipGetLastError();
}

template <typename R>
hipError_t general_probs(int n, int K, const double* C, void* p, const GeneralBufs& b, hipStream_t s) {
  int size[QST_MAX_QUBITS];
  const int groups = make_groups(n, K, size);
  void* bufs[2] = {b.bufA, b.bufB};
  const void* at;
  return forward_groups<R>(n, K, C, size, groups, groups, b.e, p, bufs, &at, s);
}

}  // namespace

hipError_t launch_general_probs(qst_prec prec, int n, int K, const double* C, const void* rho, int64_t ld_rho,
                                void* p, const GeneralBufs& b, hipStream_t s) {
  double W[32], V[32];
  pauli_mode_matrices(W, V);
  const PovmPlan pl = make_povm_plan(n, prec);
  ProfScope prof("povm_general", s);
  hipError_t e = launch_povm(false, prec, pl, W, false, rho, ld_rho, b.e, nullptr, nullptr, b.inter0, b.inter1, s);
  if (e != hipSuccess) return e;
  return prec == QST_F64 ? general_probs<double>(n, K, C, p, b, s) : general_probs<float>(n, K, C, p, b, s);
}

hipError_t launch_general_likelihood(qst_prec prec, int n, int K, int settings, const double* C, const void* rho,
                                     int64_t ld_rho, const void* f, void* G, int64_t ldG, double* nll_dev,
                                     unsigned long long* bad_dev, const GeneralBufs& b, hipStream_t s) {
  double W[32], V[32];
  pauli_mode_matrices(W, V);
  const PovmPlan pl = make_povm_plan(n, prec);
  const int64_t DK = ipow(K, n);
  const size_t rb = real_bytes(prec);
  ProfScope prof("likelihood_general", s);
  hipError_t e = launch_povm(false, prec, pl, W, false, rho, ld_rho, b.e, nullptr, nullptr, b.inter0, b.inter1, s);
  if (e != hipSuccess) return e;
  e = prec == QST_F64 ? settings_f<double>(f, settings, DK, b, s) : settings_f<float>(f, settings, DK, b, s);
  if (e != hipSuccess) return e;
  for (int st = 0; st < settings; ++st) {
    const double* Cs = C + int64_t(st) * n * K * 4;
    const void* fs = static_cast<const unsigned char*>(f) + size_t(st) * size_t(DK) * rb;
    double* sc = b.scal + 4 * st;
    void* h = G ? b.h : nullptr;
    e = prec == QST_F64 ? setting_likelihood<double>(n, K, Cs, b.e, fs, sc, h, st > 0, b, s)
                        : setting_likelihood<float>(n, K, Cs, b.e, fs, sc, h, st > 0, b, s);
    if (e != hipSuccess) return e;
  }
  settings_total_kernel<<<1, 64, 0, s>>>(b.scal, settings, nll_dev, bad_dev);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!G) return hipSuccess;
  // G' = sum_b h_b P_b: the adjoint passes with the Pauli set, fed h as is
  return launch_povm(true, prec, pl, V, false, G, ldG, nullptr, b.h, nullptr, b.inter0, b.inter1, s);
}

}  // namespace qst
