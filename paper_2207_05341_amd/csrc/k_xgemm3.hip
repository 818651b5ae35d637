// Split products of QST_F32X6 where an operand is not dense (qst_split.h says
// what that is): every FP32 operand as three bf16 parts,
// x = h + m + l exactly, with FP32's exponent range (qst_split.h).
//
// A real product a b keeps hh + hm + mh + hl + lh + mm, each exact in FP32;
// the three dropped ones (ml, lm, ll) are below 2^-26 |a||b|.  Complex
// products use three real products (3M form): for C = A B, P1 = Ar Br,
// P2 = Ai Bi, P3 = (Ar + Ai)(Br + Bi), re = P1 - P2, im = P3 - P1 - P2; for
// S = T T^dagger, P1 = Tr Tr^T, P2 = Ti Ti^T, P3 = (Tr + Ti)(Tr - Ti)^T,
// re = P1 + P2, im = P3 - P1 + P2.  The sums are formed in FP32 before the
// split.  Eighteen MFMA products where the fp16 form takes ten, and 1.5 to
// 2.25 times its plane bytes: G' T at N = 11, Gaussian operands, 224 us against
// 150 (triangular T: 197 us).
//
// 128 x 128 tiles by four waves of 64 x 64, stream-K for T T^dagger
// (qst_xgemm.h).  The K loop runs over slabs: one real product's three splits
// of A and B for one 16-deep K panel (24 units, 24 KB), copied global -> LDS
// five slabs ahead into a ring of six (144 KB); the fragments of slab s + 1
// are read while the 24 MFMAs of slab s run.
#include <hip/hip_runtime.h>

#include "qst_xgemm.h"

namespace qst {

namespace {

constexpr int X3SLOT = 24 * 1024;          // one slab
constexpr int X3NSLOT = 6;                 // LDS ring slots
constexpr int X3DIST = 5;                  // slabs copied ahead of the one being computed
constexpr int X3LDS = X3SLOT * X3NSLOT;    // 147456 bytes of LDS

static_assert((X3DIST - 1) * 6 < 64, "vmcnt immediate");

// The planes of X (blockIdx.y 0) and, for G' T, of Y^T (1); one wave per
// unit block (32 rows x 16 k), lane u one fragment slot of each unit.  Bound
// by HBM.  The scales of the fp16 planes become one.
struct X3Split {
  const Cx<float>* X[2];
  int64_t ld[2];
  u16x8* P[2];
  float* inv[2];
  X6Gate gate;
};
template <int NG>
__global__ __launch_bounds__(256) void x3_split_kernel(X3Split p, int d) {
  if (!x6_sparse(p.gate)) return;
  const int y = blockIdx.y;
  const Cx<float>* X = p.X[y];
  const int64_t ld = p.ld[y];
  for (int e = blockIdx.x * 256 + threadIdx.x; e < d; e += gridDim.x * 256) p.inv[y][e] = 1.f;
  const int lane = threadIdx.x & 63;
  const int nkb = d / 16;
  const int64_t nblk = int64_t(d / 32) * nkb;
  for (int64_t blk = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6); blk < nblk; blk += int64_t(gridDim.x) * 4) {
    const int64_t row = (blk / nkb) * 32 + (lane & 31);
    const int64_t k0 = (blk % nkb) * 16 + 8 * (lane >> 5);
    float re[8], im[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const Cx<float> v = y ? X[(k0 + e) * ld + row] : X[row * ld + k0 + e];
      re[e] = v.re;
      im[e] = v.im;
    }
    write_unit_block3<NG>(p.P[y] + blk * (NG * 3 * XUNIT) + lane, re, im);
  }
}

// Panels per MFMA accumulation chain.  The BF16 MFMA rounds the FP32
// accumulator toward zero when it adds a product block (measured: a Gram
// diagonal accumulated over all 4096 panels of d = 4096 comes out 1.9e-6
// low, against 1.2e-7 for the FP32 MFMA), so a chain is kept short and
// folded into FP32 totals with round-to-nearest adds; a new chain starts
// from a zero accumulator operand.
constexpr int X3CHAIN = 32;

// Accumulate the panels [kb, ke) of output tile (tr, tc) into (re, im)
// (which the caller zeroes).  Every thread of the workgroup calls it (it
// contains barriers); on return the LDS ring is idle.
template <bool HERK>
__device__ __forceinline__ void x3_segment(const XArgs& a, char* lds, int tr, int tc, int kb, int ke,
                                           float (&re)[2][2][16], float (&im)[2][2][16]) {
  // groups per unit block, and the group of B in the third product
  constexpr int NGA = HERK ? 4 : 3, NGB = NGA, GB2 = HERK ? 3 : 2;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w >> 1, wc = w & 1;
  const int nkb = a.d / 16;
  const uint32_t lbase = __builtin_amdgcn_readfirstlane(lds_address(lds));
  // this wave's six units of every slab: unit q = 6 w + i, A (q < 12) or B,
  // split (q % 12) / 4, row block q % 4; all of it wave-uniform except the
  // lane's 16-byte offset.  cbase[i]: unit i's address at panel 0, group 0
  // (scalar registers: the asm operand requires them); a slab adds
  // (kp ng + g) 3 units.
  const uint32_t voff = uint32_t(lane) * 16;
  const u16x8* cbase[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const int q = 6 * w + i;
    const bool isB = q >= 12;
    const int sp = (q % 12) / 4, rb = q % 4;
    const int64_t r0 = int64_t(isB ? tc : tr) * (XT / 32) + rb;
    cbase[i] = uniform_ptr((isB ? a.B : a.A) + ((r0 * nkb * (isB ? NGB : NGA)) * 3 + sp) * XUNIT);
  }
  const int npan = ke - kb;
  // copies of slab s = 3 kp + prod of the segment (panel clamped to the
  // last); prod is a compile-time constant at every call
  auto dma_slab = [&](int s, int kp, int prod) {
    const int kpa = kb + min(kp, npan - 1);
    const int64_t offA = (int64_t(kpa) * NGA + prod) * 3 * XUNIT;
    const int64_t offB = (int64_t(kpa) * NGB + (prod < 2 ? prod : GB2)) * 3 * XUNIT;
    const uint32_t slot = lbase + uint32_t((s % X3NSLOT) * X3SLOT);
    return [=](int i) {
      const int q = 6 * w + i;
      dma16(cbase[i] + (q >= 12 ? offB : offA), voff, slot + uint32_t(q * 1024));
    };
  };
  u16x8 fa[3][3][2], fb[3][3][2];  // [product][split][block]
  f16v acc[3][2][2];
#pragma unroll
  for (int s = 0; s < X3DIST; ++s) {
    const auto copy = dma_slab(s, s / 3, s % 3);
#pragma unroll
    for (int i = 0; i < 6; ++i) copy(i);
  }
  QST_VMCNT((X3DIST - 1) * 6);
  __builtin_amdgcn_s_barrier();
  {
    const u16x8* L = reinterpret_cast<const u16x8*>(lds);
#pragma unroll
    for (int sp = 0; sp < 3; ++sp)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[0][sp][i] = L[(sp * 4 + wr * 2 + i) * XUNIT + lane];
        fb[0][sp][i] = L[(12 + sp * 4 + wc * 2 + i) * XUNIT + lane];
      }
  }
  // combination order hh, hm, hl, mh, mm, lh: the current slab's A_h dies
  // after the third pair, A_m and B_m after the fifth, so the next slab's
  // fragments, read two per step in the second half of the slab (in the
  // order that slab's first MFMAs use them), mostly take freed registers
  constexpr int SA[6] = {0, 0, 0, 1, 1, 2}, SB[6] = {0, 1, 2, 0, 1, 0};
  constexpr int RD_AB[12] = {0, 0, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0};  // 0: A, 1: B
  constexpr int RD_SP[12] = {0, 0, 0, 0, 1, 1, 2, 2, 1, 1, 2, 2};
  for (int c0 = 0; c0 < npan; c0 += X3CHAIN) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[p][i][j][v] = 0.f;
    const int cend = min(npan, c0 + X3CHAIN);
    for (int kp = c0; kp < cend; ++kp) {
#pragma unroll
      for (int prod = 0; prod < 3; ++prod) {
        const int s = 3 * kp + prod;
        // every slab issued six copies per wave, so slab s+1 is complete once
        // at most X3DIST-2 newer slabs are outstanding
        QST_VMCNT((X3DIST - 2) * 6);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int np = prod == 2 ? 0 : prod + 1;
        const u16x8* L = reinterpret_cast<const u16x8*>(lds + ((s + 1) % X3NSLOT) * X3SLOT);
        const auto copy = dma_slab(s + X3DIST, kp + (prod + X3DIST) / 3, (prod + X3DIST) % 3);
#pragma unroll
        for (int q = 0; q < 12; ++q) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int m = 2 * q + h;
            const int c = m / 4, i = (m / 2) & 1, j = m & 1;
            acc[prod][i][j] = mfma32b(fa[prod][SA[c]][i], fb[prod][SB[c]][j], acc[prod][i][j]);
          }
          if (q >= 6) {
#pragma unroll
            for (int r = 2 * (q - 6); r < 2 * (q - 6) + 2; ++r) {
              const int sp = RD_SP[r], bi = r & 1;
              if (RD_AB[r] == 0) fa[np][sp][bi] = L[(sp * 4 + wr * 2 + bi) * XUNIT + lane];
              else fb[np][sp][bi] = L[(12 + sp * 4 + wc * 2 + bi) * XUNIT + lane];
            }
          } else {
            copy(q);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // close the chain: one 32 x 32 block at a time
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float p1 = acc[0][i][j][v], p2 = acc[1][i][j][v], p3 = acc[2][i][j][v];
          if constexpr (HERK) {
            re[i][j][v] += p1 + p2;
            im[i][j][v] += (p3 - p1) + p2;
          } else {
            re[i][j][v] += p1 - p2;
            im[i][j][v] += (p3 - p1) - p2;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  // the clamped copies issued past the end land before the ring is reused
  // (or the workgroup's LDS is released), and every wave is past its reads
  QST_VMCNT(0);
  __syncthreads();
}

struct X3Seg {
  static __device__ __forceinline__ void run(const XArgs& a, char* lds, int tr, int tc, int kb, int ke,
                                             float (&re)[2][2][16], float (&im)[2][2][16]) {
    x3_segment<true>(a, lds, tr, tc, kb, ke, re, im);
  }
};

template <int X0G>
__global__ __launch_bounds__(256, 1) void x3_herk_kernel(XArgs a) {
  extern __shared__ __align__(16) char lds[];
  if (x6_off(a)) return;
  x6_herk_body<X3Seg, X0G>(a, lds);
}

// G' T: one tile per workgroup.
__global__ __launch_bounds__(256, 1) void x3_hemm_kernel(XArgs a) {
  extern __shared__ __align__(16) char lds[];
  if (x6_off(a)) return;
  int tr, tc;
  x6_hemm_tile(a.d / XT, tr, tc);
  double scale = 2.0 / *a.tau;
  if (a.up) scale *= *a.up;
  float re[2][2][16], im[2][2][16];
  x6_zero(re, im);
  x3_segment<false>(a, lds, tr, tc, 0, a.kIters, re, im);
  x6_epilogue<false, 0>(a, tr, tc, re, im, scale, lds);
}

template <int X0G>
hipError_t x3_run_herk(const XArgs& a, hipStream_t s) {
  const hipError_t e = x6_allow_lds<x3_herk_kernel<X0G>, X3LDS>();
  if (e != hipSuccess) return e;
  const int64_t grid = a.sc.rounds > 0 ? a.sc.P : a.sc.Q;
  x3_herk_kernel<X0G><<<unsigned(grid), 256, X3LDS, s>>>(a);
  return hipGetLastError();
}

unsigned x3_split_grid(int d) { return unsigned(std::min<int64_t>(1024, int64_t(d / 32) * (d / 16) / 4)); }

}  // namespace

hipError_t x3_launch_herk(XArgs a, const void* T, int64_t ldt, int x0g, void* planes, float* rinv, hipStream_t s) {
  X3Split p{};
  p.X[0] = static_cast<const Cx<float>*>(T);
  p.ld[0] = ldt;
  p.P[0] = static_cast<u16x8*>(planes);
  p.inv[0] = rinv;
  p.gate = a.gate;
  x3_split_kernel<4><<<x3_split_grid(a.d), 256, 0, s>>>(p, a.d);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  a.A = a.B = p.P[0];
  a.when = kX6Sparse;
  return x0g == 6   ? x3_run_herk<6>(a, s)
         : x0g == 5 ? x3_run_herk<5>(a, s)
         : x0g == 4 ? x3_run_herk<4>(a, s)
                    : x3_run_herk<0>(a, s);
}

hipError_t x3_launch_hemm(XArgs a, const void* G, int64_t ldg, const void* T, int64_t ldt, void* planes, float* ginv,
                          float* tinv, hipStream_t s) {
  u16x8* P = static_cast<u16x8*>(planes);
  X3Split p{{static_cast<const Cx<float>*>(G), static_cast<const Cx<float>*>(T)},
            {ldg, ldt},
            {P, P + size_t(a.d) * a.d * (kX3HemmBytes / 2) / sizeof(u16x8)},
            {ginv, tinv},
            a.gate};
  x3_split_kernel<3><<<dim3(x3_split_grid(a.d), 2), 256, 0, s>>>(p, a.d);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = x6_allow_lds<x3_hemm_kernel, X3LDS>()) != hipSuccess) return e;
  a.A = p.P[0];
  a.B = p.P[1];
  a.when = kX6Sparse;
  const int ts = a.d / XT;
  x3_hemm_kernel<<<unsigned(ts * ts), 256, X3LDS, s>>>(a);
  return hipGetLastError();
}

}  // namespace qst
