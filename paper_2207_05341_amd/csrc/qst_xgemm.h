// What the two families of split products share (k_xgemm.hip: two fp16 parts
// per value; k_xgemm3.hip: three bf16 parts): kernel arguments, the choice
// between the families, the T T^dagger schedule, partial tiles and the tile
// epilogue.
#pragma once

#include <algorithm>
#include <mutex>

#include "qst_device.h"
#include "qst_gemm_tiles.h"
#include "qst_kernels.h"
#include "qst_plan.h"
#include "qst_split.h"
#include "qst_xtile.h"

namespace qst {

constexpr int XT = kX6Tile;  // output tile (complex)
constexpr int XUNIT = kX6UnitVecs;

// When a kernel of a launch sequence runs; it reads the gate itself.
enum X6When { kX6Dense, kX6Sparse, kX6Always };

struct XArgs {
  const u16x8* A;  // planes of the row operand
  const u16x8* B;  // planes of the column operand (rows of B^T)
  X6Gate gate;
  X6When when;
  const float* sa;  // what takes A's row scales out again
  const float* sb;  // the same for B's rows (the output's columns)
  const double* rsum;  // HERK: sums of |T|^2 over 128-entry row pieces, [d / 128][d]
  void* C;          // output (HEMM, or HERK without x0)
  int64_t ldc;
  int d;
  const double* tau;       // tau, or NULL with tau_part
  const double* tau_part;  // FP64 partial sums of tau (kReduceBlocks), folded by every workgroup
  double* tau_out;         // where workgroup 0 of the T T^dagger fix-up stores the folded tau
  const double* up;        // HEMM: upstream scalar or NULL
  float* part;             // HERK partial tiles [slots][re, im][TILE] in the MFMA layout
  int ntiles, kIters;
  X6HerkSched sc;          // HERK schedule (rounds, then slices)
  void* x0;                // HERK: first POVM pass output, or NULL
  int x0g, x0up;
};

__device__ __forceinline__ bool x6_off(const XArgs& a) {
  return a.when != kX6Always && x6_sparse(a.gate) != (a.when == kX6Sparse);
}

constexpr int kXTileVals = XT * XT;  // complex values per tile

// Fold of the tau partials in a fixed order (bitwise the same in every
// workgroup), through the idle ring's first bytes.
__device__ __forceinline__ double x6_tau(const XArgs& a, char* lds) {
  double* red = reinterpret_cast<double*>(lds);
  double acc = 0.0;
  for (int b = threadIdx.x; b < kReduceBlocks; b += 256) acc += a.tau_part[b];
  const double sum = block_sum256(acc, red);
  if (threadIdx.x == 0) red[4] = sum;
  __syncthreads();
  const double tau = red[4];
  __syncthreads();
  return tau;
}

// (row, column) inside the 128 x 128 tile of accumulator value v of block
// (i, j) held by lane `lane` of wave (wr, wc).
__device__ __forceinline__ int x6_row(int wr, int i, int v, int lane) {
  return wr * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
}
__device__ __forceinline__ int x6_col(int wc, int j, int lane) { return wc * 64 + j * 32 + (lane & 31); }

// Partial of a tile segment, 16 bytes per lane and store: values
// 4 vq .. 4 vq + 3 of block ij = 2 i + j, part p (re, im) of wave w's lane l
// at floats ((((4 w + ij) 2 + p) 4 + vq) 64 + l) 4 .. + 3 (each store of a
// wave is 1 KB contiguous; wave w's 64 x 64 quadrant is floats
// [8192 w, 8192 (w + 1))).
__device__ __forceinline__ float* x6_slot(const XArgs& a, int64_t slot) {
  return a.part + slot * int64_t(2 * kXTileVals);
}
// slot of a round unit u (sk > 1), and of slice `which` (0: the first unit
// of the worker's range, 1: the last) of slice worker w
__device__ __forceinline__ int64_t x6_unit_slot(int64_t u) { return u; }
__device__ __forceinline__ int64_t x6_slice_slot(const X6HerkSched& sc, int64_t w, int which) {
  return (sc.sk > 1 ? sc.main : 0) + (sc.tq ? w : 2 * w + which);
}
__device__ __forceinline__ void x6_store_partial(float* dst, const float (&re)[2][2][16], const float (&im)[2][2][16]) {
  const int th = fresh_thread(), lane = th & 63, w = th >> 6;
  f4v* d4 = reinterpret_cast<f4v*>(dst);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int64_t o = (((w * 4 + i * 2 + j) * 2) * 4 + vq) * 64 + lane;
        d4[o] = f4v{re[i][j][4 * vq], re[i][j][4 * vq + 1], re[i][j][4 * vq + 2], re[i][j][4 * vq + 3]};
        d4[o + 256] = f4v{im[i][j][4 * vq], im[i][j][4 * vq + 1], im[i][j][4 * vq + 2], im[i][j][4 * vq + 3]};
      }
}

// Scales of the values of a wave's 64 x 64 quadrant at (r0, c0): rs[i][v]
// takes the row scale of value v of block row i out, cs[j] the column
// scale of block column j with the overall factor.  Powers of two but for
// that factor, so value * cs * rs rounds once.
__device__ __forceinline__ void x6_scales(const XArgs& a, int64_t r0, int64_t c0, double scale, float (&rs)[2][16],
                                          float (&cs)[2]) {
  const int lane = fresh_thread() & 63;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      rs[i][v] = a.sa[r0 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)];
#pragma unroll
  for (int j = 0; j < 2; ++j) cs[j] = float(scale * double(a.sb[c0 + j * 32 + (lane & 31)]));
}

// Diagonal entries r0 .. r0 + NR - 1 of T T^dagger, the rows' sums of
// |T|^2, as 256 / NR partial sums each in sums (x6_diag adds them): called
// by the whole workgroup, a barrier before the sums are read.  The product
// leaves out the ll terms, whose mean is zero except on the diagonal, where
// each is a square: there it came out 4e-8 low, as the trace did, and the
// gradient (in which the trace part cancels) took a relative error of 5e-7
// to 1e-6 from that (N = 10: 1.4e-6 with the product's diagonal).
template <int NR>
__device__ __forceinline__ void x6_diag_sums(const XArgs& a, int64_t r0, double* sums) {
  constexpr int NP = 256 / NR;
  const double* src = a.rsum + r0 + threadIdx.x % NR;
  double s = 0.0;
#pragma unroll 8
  for (int q = threadIdx.x / NR; q < a.d / XT; q += NP) s += src[int64_t(q) * a.d];
  sums[threadIdx.x] = s;
}
template <int NR>
__device__ __forceinline__ float x6_diag(const double* sums, int r, double scale) {
  double s = sums[r];
#pragma unroll
  for (int p = 1; p < 256 / NR; ++p) s += sums[p * NR + r];
  return float(s * scale);
}

// Tile epilogue.  HEMM: C = scale (re, im).  HERK without x0: rho = (re,
// im) / tau, and the conjugate transpose at the mirror position for an
// off-diagonal tile.  HERK with x0: the first POVM pass over G qubits on
// each 64 x 64 quadrant (the quadrant of wave q, q = 2 qr + qc; the upper
// quadrant of a diagonal tile is the mirror of the lower one and skipped),
// through a 64 x 64 tile in LDS.
template <bool HERK, int X0G>
__device__ __forceinline__ void x6_epilogue(const XArgs& a, int tr, int tc, const float (&re)[2][2][16],
                                            const float (&im)[2][2][16], double scale, char* lds) {
  const int th = fresh_thread(), lane = th & 63, w = th >> 6;
  const int wr = w >> 1, wc = w & 1;
  const int64_t R0 = int64_t(tr) * XT, C0 = int64_t(tc) * XT;
  // row scales of this lane's values (four rows per group of four values)
  // and column scales with the overall factor
  float rs[2][16], cs[2];
  x6_scales(a, R0 + wr * 64, C0 + wc * 64, scale, rs, cs);
  double* diag = reinterpret_cast<double*>(lds + 64 * 64 * sizeof(Cx<float>));
  if constexpr (HERK) {
    if (tr == tc) {
      x6_diag_sums<XT>(a, R0, diag);
      __syncthreads();
    }
  }
  if constexpr (X0G == 0) {
    Cx<float>* C = static_cast<Cx<float>*>(a.C);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t r = R0 + x6_row(wr, i, v, lane), c = C0 + x6_col(wc, j, lane);
          float xr = re[i][j][v] * cs[j] * rs[i][v], xi = im[i][j][v] * cs[j] * rs[i][v];
          if (HERK && i == j && r == c) {
            xr = x6_diag<XT>(diag, int(r - R0), scale);
            xi = 0.f;
          }
          C[r * a.ldc + c] = Cx<float>{xr, xi};
          if (HERK && tr != tc) C[c * a.ldc + r] = Cx<float>{xr, -xi};
        }
    if constexpr (HERK) {
      if (tr == tc) __syncthreads();  // the sums are read before the next segment's copies take their place
    }
  } else {
    constexpr int G = X0G;
    constexpr int S = 64 >> G;
    constexpr int TG = 1 << (2 * G);
    constexpr int M = (1 << G) - 1;
    Cx<float>* L = reinterpret_cast<Cx<float>*>(lds);
    gemm::GemmArgs g{};
    g.x0 = a.x0;
    g.x0g = a.x0g;
    g.x0up = a.x0up;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int qr = q >> 1, qc = q & 1;
      if (tr == tc && qr < qc) continue;  // uniform across the workgroup
      if (w == q) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const int r = i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), c = j * 32 + (lane & 31);
              Cx<float> x{re[i][j][v] * cs[j] * rs[i][v], im[i][j][v] * cs[j] * rs[i][v]};
              if (i == j && tr == tc && wr == wc && r == c) x = Cx<float>{x6_diag<XT>(diag, wr * 64 + r, scale), 0.f};
              L[((r >> G) * S + (c >> G)) * TG + swz<G>(r & M, c & M)] = x;
            }
      }
      __syncthreads();
      gemm::x0_rounds<float, G>(g, int64_t(2) * tr + qr, int64_t(2) * tc + qc, L);
      __syncthreads();
    }
  }
}

__device__ __forceinline__ void x6_zero(float (&re)[2][2][16], float (&im)[2][2][16]) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) re[i][j][v] = im[i][j][v] = 0.f;
}

// Tile of this workgroup in a ts x ts grid: blocks of 4 x 8 tiles per 32
// consecutive logical workgroups.
__device__ __forceinline__ void x6_hemm_tile(int ts, int& tr, int& tc) {
  const int lb = int(xcd_order(blockIdx.x, gridDim.x));
  if (ts % 8 == 0) {
    const int grp = lb / 32, within = lb % 32;
    tr = (grp / (ts / 8)) * 4 + within / 8;
    tc = (grp % (ts / 8)) * 8 + within % 8;
  } else {
    tr = lb / ts;
    tc = lb % ts;
  }
}

// (even, as the fp16 segments need; iters is)
__device__ __forceinline__ int64_t x6_slice_start(int64_t w, int64_t Q, int64_t iters) {
  return 2 * ((w * (iters / 2)) / Q);
}

// Unit u -> tile and K panels: u = s * ntiles + t covers panels
// [s kh, (s + 1) kh) of lower tile t (the units of a round share s, so
// its workgroups stream the same K range).
__device__ __forceinline__ void x6_unit(const X6HerkSched& sc, int64_t u, int64_t& t, int& k0) {
  t = u % sc.ntiles;
  k0 = int((u / sc.ntiles) * sc.kh);
}

// T T^dagger: logical workgroup w takes round units w, w + P, ...; a whole
// tile (sk = 1) is finished here, a part of one is stored as a partial.
// Then, as slice worker w < Q, the iterations [start(w), start(w + 1)) of
// the remaining units' (unit, panel) sequence.  One loop over both, so that
// the segment code (Seg) is there once.
template <class Seg, int X0G>
__device__ __forceinline__ void x6_herk_body(const XArgs& a, char* lds) {
  const X6HerkSched& sc = a.sc;
  const int w = int(xcd_order(blockIdx.x, gridDim.x));
  int r = 0;
  // transposed slices: one piece, slice w / left of unit w % left
  int it = 0, end = 0, first_unit = 0;
  if (w < sc.Q) {
    it = sc.tq ? 0 : int(x6_slice_start(w, sc.Q, sc.left_iters));
    end = sc.tq ? 1 : int(x6_slice_start(w + 1, sc.Q, sc.left_iters));
    first_unit = it / int(sc.kh);
  }
  while (r < sc.rounds || it < end) {
    int u, kb = 0, ke = int(sc.kh), slot;
    if (r < sc.rounds) {
      u = r * int(sc.P) + w;
      slot = int(x6_unit_slot(u));
      ++r;
    } else {
      int j;  // leftover unit
      if (sc.tq) {
        j = w % int(sc.left);
        kb = (w / int(sc.left)) * int(sc.ps);
        ke = kb + int(sc.ps);
        it = end;
      } else {
        j = it / int(sc.kh);
        kb = it % int(sc.kh);
        ke = min(int(sc.kh), kb + (end - it));
        it += ke - kb;
      }
      u = int(sc.main) + j;
      slot = int(x6_slice_slot(sc, w, j == first_unit ? 0 : 1));  // slot w with tq
    }
    int64_t t;
    int k0;
    x6_unit(sc, u, t, k0);
    int tr, tc;
    tri_decode(t, tr, tc);
    float re[2][2][16], im[2][2][16];
    x6_zero(re, im);
    Seg::run(a, lds, tr, tc, k0 + kb, k0 + ke, re, im);
    if (sc.sk == 1 && kb == 0 && ke == sc.kh) x6_epilogue<true, X0G>(a, tr, tc, re, im, 1.0 / x6_tau(a, lds), lds);
    else x6_store_partial(x6_slot(a, slot), re, im);
  }
}

// The product kernels use more LDS than the static limit: raise the
// per-kernel limit once per device before the first launch.
template <auto K, int BYTES>
hipError_t x6_allow_lds() {
  static std::mutex mu;  // one flag set per kernel
  static bool done[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!done[dev]) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(K), hipFuncAttributeMaxDynamicSharedMemorySize, BYTES);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  return hipSuccess;
}

inline int x6_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  return cus;
}

// k_xgemm.hip: adds the partial tiles of a T T^dagger (x0g: a.x0g, or 0).
hipError_t x6_launch_fixup(const XArgs& a, int x0g, hipStream_t s);
// k_xgemm3.hip: the products of a (its operands T, or G and T, as given to
// the fp16 ones) where an operand is not dense; planes of kX3HerkBytes or
// kX3HemmBytes per element; the scales rinv (ginv, tinv) are set to one.
// The caller adds T T^dagger's partial tiles.
hipError_t x3_launch_herk(XArgs a, const void* T, int64_t ldt, int x0g, void* planes, float* rinv, hipStream_t s);
hipError_t x3_launch_hemm(XArgs a, const void* G, int64_t ldg, const void* T, int64_t ldt, void* planes, float* ginv,
                          float* tinv, hipStream_t s);

}  // namespace qst
