// Split complex products: FP32 operands, every real product computed on the
// 16-bit matrix cores from a two-part fp16 split of each operand.
//
//   state map  rho = T T^dagger / tau      (Eq. T_matrix; Eq. unified_DP)
//   gradient   grad = s (2 / tau) G' T     (adjoint of the state map)
//
// Split (qst_split.h): each operand row, scaled by a power of two, is
// x = h + l with h and l in fp16 (22 significand bits and the sign of l).  A
// real product a b keeps hh + hl + lh, each exact in FP32; the dropped ll is
// below 2^-22 |a||b| and of random sign (the diagonal of T T^dagger, where it
// is a square, is formed apart: x6_diag_sums).  Accumulation is in FP32
// inside the MFMA.
//
// Where it is used.  One scale per row leaves entries below 2^-15 of the
// row's largest fewer bits, and 22 bits are less than FP32's 24: the products
// are more accurate than FP32's where the accumulation of many comparable
// terms sets the error, and less where a few terms carry an entry or large
// entries of one operand meet small ones of the other.  So the split counts
// the entries near the largest of their row (column), and the indices of the
// contraction near the largest, and the fp16 products are stored only where
// both operands are dense by those counts (qst_split.h, with the reasons).
// Elsewhere QST_F32 runs its FP32 MFMA products (k_gemm.hip) and QST_F32X6 the
// exact three-part bf16 split (k_xgemm3.hip).  The counts are in device
// memory (X6Gate), and every kernel of either kind reads them first: no host
// decision, and a captured call chooses again at each replay.  Relative errors
// against FP64 at N = 10 or 11, FP32 MFMA / bf16 / fp16 products: Gaussian T,
// G' T 1.1e-6 / 5.0e-7 / 2.2e-7; one nonzero column of T, rho 7e-8 / 1.0e-7 /
// 1.3e-7; T = D^-1 X and G' = D A D with D within 2^+-12, 8e-7 / 5.0e-7 /
// 1.5e-5.  A kernel that finds itself unused takes 4.6 us, a launch and a load
// that misses: four of them in a QST_F32X6 step, three or four in a QST_F32 one.
//
// Complex products: ten MFMA products per 32 x 32 block and K panel.  The
// leading part h h takes the four real products of the definition.  Each of
// the two corrections A' B' (h l and l h) takes three (Gauss): K1 = B'r
// (A'r + A'i), K2 = A'r (B'i - B'r), K3 = -A'i (B'r + B'i), re = K1 + K3,
// im = K1 + K2, whose operand sums are formed from the fragments in fp16 --
// the corrections are 2^-11 of the product, so the sums' rounding is another
// FP32 rounding per term.  K2 and K3 go to the accumulators of im and re, K1
// has its own, added once at the end of a segment.
//
// What bounds it: power.  At N = 11 under sustained load G' T runs at 1.65 GHz
// (active cycles over its time; 2.4 nominal): 172 GFLOP in 150 us, 1.15
// PFLOP/s, what a large fp16 library product reaches on this card (1.14).
// Twelve products per block (four per correction): 162 us; all in the
// three-product form (nine, with re + im planes as operands) needs 1.5 times
// the LDS and plane bytes.  The three-part bf16 products (18): 224 us on the
// same operands, and two times the plane bytes.
//
// Operand planes.  A split pass writes each operand once per call as fp16
// planes in the order the v_mfma_f32_32x32x16_f16 fragments read them: a
// 1 KB unit holds a 32-row x 16-k block of one plane, 16 bytes per lane
// (lane u: row u % 32, k 8 (u / 32) .. + 7), and the four units (re_h,
// re_l, im_h, im_l) of one (row block, K panel) are contiguous.
//
// Product kernel: a 128 x 128 complex output tile per 256-thread workgroup
// (four waves of 64 x 64, 2 x 2 MFMA blocks of 32 x 32 each).  The K loop
// runs over slabs, one 16-deep K panel each (32 units, 32 KB, 40 MFMAs per
// wave).  Slabs are copied global -> LDS by the DMA form of the global load
// (no registers), three slabs ahead, into a ring of four LDS slots (128 KB).
// The fragments of the next slab are read while the current one's MFMAs
// run.
//
// T T^dagger computes the lower 128 x 128 tiles only (136 at d = 2048),
// which do not divide evenly over the compute units, so it runs stream-K:
// each workgroup takes an equal contiguous share of the (tile, panel)
// sequence; a tile cut between workgroups leaves partial sums (at most two
// per workgroup) that a fix-up kernel adds in K order (deterministic) before
// the tile's epilogue (rho, or the first POVM pass).  G' T has (d / 128)^2
// tiles, one per workgroup, numbered so that each XCD runs 4 x 8 blocks of
// tiles.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "qst_xgemm.h"

namespace qst {

namespace {

typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));

constexpr int XSLOT = 32 * 1024;      // one slab: 32 units, 4 row blocks of A and of B
constexpr int XNSLOT = 4;             // LDS ring slots
constexpr int XDIST = XNSLOT - 1;     // slabs copied ahead of the one being computed
constexpr int XCOPY = 8;              // units copied per wave and slab
constexpr int XLDS = XSLOT * XNSLOT;  // 131072 bytes of LDS

static_assert((XDIST - 1) * XCOPY < 64, "vmcnt immediate");
static_assert(kX6MaxBlocks >= kReduceBlocks, "one maximum per workgroup");

// ---------------------------------------------------------------------------
// Scales and split (helpers in qst_split.h)
// ---------------------------------------------------------------------------
// Largest |component| of every 64-entry piece of a row and of a column of
// X, per 64 x 64 tile: rowp[tc * d + row] and colp[tr * d + column].  With
// TAU also the FP64 partial sums of tau = sum |X_ij|^2 and, with f, of
// F = sum f_k: workgroup b of nb writes partials[b] (its tiles b, b + nb, ...)
// and partials[nb + b] (f over [b D / nb, (b + 1) D / nb), D = d^2), each
// summed in a fixed order.  The first 16 values of f per thread are loaded
// first, so that their loads are in flight together with those of X.
// Bound by HBM (X and f read once).
//
// Thread t holds rows t / 32 + 8 k, columns 2 (t % 32), + 1 of a tile.  The
// row maxima go over the half-wave in a halving exchange: three steps trade
// half of the remaining rows for the partner's values of the other half,
// after which a lane holds one row's maximum over eight lanes; two plain
// steps finish it (nine shuffles in place of forty).
template <bool TAU, bool WITH_F>
__device__ __forceinline__ void x6_absmax(const Cx<float>* __restrict__ X, int64_t ld, int d, float* __restrict__ rowp,
                                          float* __restrict__ colp, float* __restrict__ wmax, int* __restrict__ flags,
                                          double* __restrict__ partials, const float* __restrict__ f) {
  constexpr int NT = 256, U = 16;
  __shared__ double red[4];
  __shared__ float cm[8][64];
  const int nb = gridDim.x, t = threadIdx.x;
  if (blockIdx.x == 0 && t < 4) flags[t] = 0;  // the split that follows sets them
  const int64_t D = int64_t(d) * d;
  const int64_t fbeg = D * blockIdx.x / nb, fend = D * (blockIdx.x + 1) / nb;
  float fv[U];
  if constexpr (WITH_F) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t e = fbeg + t + u * NT;
      fv[u] = e < fend ? f[e] : 0.f;
    }
  }
  double acc = 0.0, accf = 0.0;
  float top = 0.f;
  const int tiles = d / 64, c2 = t & 31, rq = t >> 5;
  for (int tile = blockIdx.x; tile < tiles * tiles; tile += nb) {
    const int tr = tile / tiles, tc = tile % tiles;
    const Cx<float>* src = X + (int64_t(tr) * 64 + rq) * ld + int64_t(tc) * 64 + 2 * c2;
    f4u v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const f4u*>(src + 8 * k * ld);
    float m[8], ca = 0.f, cb = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float a = fmaxf(fabsf(v[k][0]), fabsf(v[k][1])), b = fmaxf(fabsf(v[k][2]), fabsf(v[k][3]));
      m[k] = fmaxf(a, b);
      ca = fmaxf(ca, a);
      cb = fmaxf(cb, b);
      if constexpr (TAU)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += double(v[k][e]) * double(v[k][e]);
    }
    cm[rq][2 * c2] = ca;
    cm[rq][2 * c2 + 1] = cb;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int half = 4 >> s;
      const bool up = (c2 >> s) & 1;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        const float send = up ? m[i] : m[i + half], keep = up ? m[i + half] : m[i];
        m[i] = fmaxf(keep, __shfl_xor(send, 1 << s, 64));
      }
    }
    float r = m[0];
    r = fmaxf(r, __shfl_xor(r, 8, 64));
    r = fmaxf(r, __shfl_xor(r, 16, 64));
    if (c2 < 8) {  // lane c2 holds row 4 (c2 & 1) + 2 (c2 >> 1 & 1) + (c2 >> 2) of its eight
      const int k = 4 * (c2 & 1) + (c2 & 2) + (c2 >> 2);
      rowp[int64_t(tc) * d + tr * 64 + rq + 8 * k] = r;
    }
    __syncthreads();
    if (t < 64) {
      float c = cm[0][t];
#pragma unroll
      for (int q = 1; q < 8; ++q) c = fmaxf(c, cm[q][t]);
      colp[int64_t(tr) * d + tc * 64 + t] = c;
      top = fmaxf(top, c);
    }
    __syncthreads();
  }
  if (t < 64) {  // the wave that folded the columns
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, 64));
    if (t == 0) wmax[blockIdx.x] = top;
  }
  if constexpr (WITH_F) {
#pragma unroll
    for (int u = 0; u < U; ++u) accf += double(fv[u]);
    // the rest of the range (N >= 12), U strided loads per thread at a time
    for (int64_t e0 = fbeg + t + U * NT; e0 < fend; e0 += U * NT) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t e = e0 + u * NT;
        fv[u] = e < fend ? f[e] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) accf += double(fv[u]);
    }
  }
  if constexpr (TAU) {
    const double st = block_sum256(acc, red);
    if (t == 0) partials[blockIdx.x] = st;
  }
  if constexpr (WITH_F) {
    const double sf = block_sum256(accf, red);
    if (t == 0) partials[nb + blockIdx.x] = sf;
  }
}

// T, for T T^dagger.
template <bool WITH_F>
__global__ __launch_bounds__(256) void x6_absmax_t_kernel(const Cx<float>* __restrict__ T, int64_t ld, int d,
                                                          X6Scales sc, double* __restrict__ partials,
                                                          const float* __restrict__ f) {
  x6_absmax<true, WITH_F>(T, ld, d, sc.rowp, sc.colp, sc.wmax, sc.bad, partials, f);
}

// G' (blockIdx.y 0) and T (1), for G' T: one launch for both.
struct X6Pair {
  const Cx<float>* X[2];
  int64_t ld[2];
  X6Scales sc[2];
  u16x8* P[2];
  float low;
};
__global__ __launch_bounds__(256) void x6_absmax_gt_kernel(X6Pair p, int d) {
  const int y = blockIdx.y;
  x6_absmax<false, false>(p.X[y], p.ld[y], d, p.sc[y].rowp, p.sc[y].colp, p.sc[y].wmax, p.sc[y].bad, nullptr, nullptr);
}

// The planes of X as a row operand (ROWS; row r scaled by its largest
// component) and of X^T (COLS; row = column of X, likewise), from one read
// of X, and what takes the scales out again (rinv, cinv).  A workgroup takes
// four consecutive 32 x 32 blocks of one block row, one per wave: it folds
// the maxima of its 32 rows and 128 columns, then a wave reads its block as
// the slots of two row-operand unit blocks (lane u: row u % 32, columns
// 16 h + 8 (u / 32) .. + 7, h = 0, 1); with COLS it passes the block through
// LDS (8 KB per wave, 16-byte chunks swizzled by row) and reads the two unit
// blocks of X^T (lane u: column u % 32, rows 16 h + 8 (u / 32) .. + 7).
// With SUMS also the FP64 sums of |x|^2 over the 128 columns of each row.
// Where less than three quarters of the entries of a 128-entry piece of a row
// (32-entry piece of a column) have a scaled component that reaches low, the
// flag bad[0] (bad[1]) is set: the operand is not dense.
// Bound by HBM: X read, 8 bytes per element and operand written.
__device__ __forceinline__ int split_swz(int r, int c) {  // (r, c) of a 32 x 32 block, complex index
  return r * 32 + 2 * (((c >> 1) ^ r) & 15) + (c & 1);
}

template <bool ROWS, bool COLS, bool SUMS>
__device__ __forceinline__ void x6_split(const Cx<float>* __restrict__ X, int64_t ld, int d, const X6Scales& sc6,
                                         u16x8* __restrict__ P, u16x8* __restrict__ PT, float low, int nmax) {
  const float *rowp = sc6.rowp, *colp = sc6.colp;
  __shared__ Cx<float> blkL[COLS ? 4 : 1][COLS ? 32 * 32 : 1];
  __shared__ float rm[8][32], cmx[2][128], rsc[32], csc[128];
  __shared__ double rs[SUMS ? 4 : 1][32];
  __shared__ int big[ROWS ? 4 : 1][32];
  __shared__ float tops[4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int row = lane & 31, hq = lane >> 5;
  const int nkb = d / 16, nb32 = d / 32, np = d / 64;
  const int64_t br = blockIdx.x / (nb32 / 4), bc0 = int64_t(blockIdx.x % (nb32 / 4)) * 4, bc = bc0 + wv;
  Cx<float> v[2][8];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) v[h][e] = X[(32 * br + row) * ld + 32 * bc + 16 * h + 8 * hq + e];
  // the first workgroups of either direction count the rows and columns near
  // the largest, whichever operand this is
  const bool rows = ROWS || bc0 == 0, cols = COLS || br == 0;
  if (bc0 == 0 || br == 0) {
    float m = 0.f;
    for (int k = t; k < nmax; k += 256) m = fmaxf(m, sc6.wmax[k]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane == 0) tops[wv] = m;
  }
  if (rows) {
    float m = 0.f;
    for (int k = t >> 5; k < np; k += 8) m = fmaxf(m, rowp[int64_t(k) * d + 32 * br + (t & 31)]);
    rm[t >> 5][t & 31] = m;
  }
  if (cols) {
    float m = 0.f;
    for (int k = t >> 7; k < np; k += 2) m = fmaxf(m, colp[int64_t(k) * d + 32 * bc0 + (t & 127)]);
    cmx[t >> 7][t & 127] = m;
  }
  __syncthreads();
  if (bc0 == 0 && t < 64) {
    float m = rm[0][t & 31];
#pragma unroll
    for (int q = 1; q < 8; ++q) m = fmaxf(m, rm[q][t & 31]);
    const float top = fmaxf(fmaxf(tops[0], tops[1]), fmaxf(tops[2], tops[3]));
    const int n = __popcll(__ballot(t < 32 && m >= kX6Near * top));
    if (t == 0) atomicAdd(&sc6.near[0], n);
  }
  if (br == 0 && t >= 128) {
    const float m = fmaxf(cmx[0][t - 128], cmx[1][t - 128]);
    const float top = fmaxf(fmaxf(tops[0], tops[1]), fmaxf(tops[2], tops[3]));
    const int n = __popcll(__ballot(m >= kX6Near * top));
    if (lane == 0) atomicAdd(&sc6.near[1], n);
  }
  if constexpr (ROWS) {
    if (t < 32) {
      float m = rm[0][t];
#pragma unroll
      for (int q = 1; q < 8; ++q) m = fmaxf(m, rm[q][t]);
      const int e = x6_scale_exp(m, kX6Top);
      rsc[t] = x6_pow2(e);
      if (bc0 == 0) sc6.rinv[32 * br + t] = x6_pow2(-e);
      if (!x6_finite(m)) sc6.bad[0] = 1;
    }
  }
  if constexpr (SUMS) {
    double acc = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        acc += double(v[h][e].re) * double(v[h][e].re) + double(v[h][e].im) * double(v[h][e].im);
    acc += __shfl_xor(acc, 32, 64);
    if (lane < 32) rs[wv][lane] = acc;
  }
  if constexpr (COLS) {
    if (t >= 128) {
      const int c = t - 128;
      const float m = fmaxf(cmx[0][c], cmx[1][c]);
      const int e = x6_scale_exp(m, kX6Top);
      if (!x6_finite(m)) sc6.bad[1] = 1;
      csc[c] = x6_pow2(e);
      if (br == 0) sc6.cinv[32 * bc0 + c] = x6_pow2(-e);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) blkL[wv][split_swz(row, 16 * h + 8 * hq + e)] = v[h][e];
  }
  __syncthreads();
  if constexpr (SUMS) {
    if (t < 32) sc6.rsum[(bc0 / 4) * d + 32 * br + t] = ((rs[0][t] + rs[1][t]) + rs[2][t]) + rs[3][t];
  }
  if constexpr (ROWS) {
    const float sc = rsc[row];
    int n = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float re[8], im[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        re[e] = v[h][e].re;
        im[e] = v[h][e].im;
      }
      n += write_unit_block(P + (br * nkb + 2 * bc + h) * kX6BlockVecs + lane, re, im, sc, low);
    }
    n += __shfl_xor(n, 32, 64);
    if (lane < 32) big[wv][lane] = n;
    __syncthreads();
    if (t < 32 && 4 * (big[0][t] + big[1][t] + big[2][t] + big[3][t]) < 3 * 128) sc6.bad[0] = 1;
  }
  if constexpr (COLS) {
    const float sc = csc[32 * wv + row];
    int n = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float re[8], im[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const Cx<float> x = blkL[wv][split_swz(16 * h + 8 * hq + e, row)];
        re[e] = x.re;
        im[e] = x.im;
      }
      n += write_unit_block(PT + (bc * nkb + 2 * br + h) * kX6BlockVecs + lane, re, im, sc, low);
    }
    n += __shfl_xor(n, 32, 64);
    if (4 * n < 3 * 32) sc6.bad[1] = 1;
  }
}

// T for T T^dagger, and with TT T^T for G' T of the same call.
template <bool TT>
__global__ __launch_bounds__(256) void x6_split_t_kernel(const Cx<float>* __restrict__ T, int64_t ld, int d, X6Scales sc,
                                                         u16x8* __restrict__ P, u16x8* __restrict__ PT, float low) {
  x6_split<true, TT, true>(T, ld, d, sc, P, PT, low, kReduceBlocks);
}

// G' (blockIdx.y 0) and T^T (1) for G' T.
__global__ __launch_bounds__(256) void x6_split_gt_kernel(X6Pair p, int d, int nmax) {
  if (blockIdx.y == 0) x6_split<true, false, false>(p.X[0], p.ld[0], d, p.sc[0], p.P[0], nullptr, p.low, nmax);
  else x6_split<false, true, false>(p.X[1], p.ld[1], d, p.sc[1], nullptr, p.P[1], p.low, nmax);
}

// ---------------------------------------------------------------------------
// Product kernel
// ---------------------------------------------------------------------------
// Panels per MFMA accumulation chain (even).  The MFMA rounds the FP32
// accumulator toward zero when it adds a product block, so a chain is kept
// short and folded into FP32 totals with round-to-nearest adds; a new chain
// starts from a zero accumulator operand.  16 panels are 1% faster at N = 11
// and 12, but where all terms of a sum have one sign (T of positive entries)
// their rho is less accurate than the three-part split's: largest error at
// N = 10, relative to sum |a||b|, 2.6e-7 against 2.4e-7; with 8, 2.0e-7.
constexpr int XCHAIN = 8;
static_assert(XCHAIN % 2 == 0, "the fragment buffers alternate by panel");

// Accumulate the panels [kb, ke), an even number, of output tile (tr, tc)
// into (re, im) (which the caller zeroes).  Every thread of the workgroup
// calls it (it contains barriers); on return the LDS ring is idle.
//
// A panel visits the wave's four 32 x 32 blocks as (0, f), (0, 1 - f),
// (1, 1 - f), (1, f) with f = 0, 1 in alternate panels, so that the next
// panel's first operands (A's row block 0, B's column block 1 - f) are read
// into registers that this panel has finished with, and its other two while
// its first block runs: no fragment is held twice.  At the end of a chain
// the accumulators of a block are folded into the totals during the next
// block's MFMAs.
template <bool HERK>
__device__ __forceinline__ void x6_segment(const XArgs& a, char* lds, int tr, int tc, int kb, int ke,
                                           float (&re)[2][2][16], float (&im)[2][2][16]) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w >> 1, wc = w & 1;
  const int nkb = a.d / 16;
  const uint32_t lbase = __builtin_amdgcn_readfirstlane(lds_address(lds));
  // this wave's eight units of every slab: the four planes of row blocks
  // 2 w and 2 w + 1 of the slab's eight (A's four, then B's)
  uint32_t voff[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) voff[u] = uint32_t(lane) * 16 + u * 1024;
  const u16x8* cbase[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = 2 * w + i;
    const int64_t r0 = int64_t(q >= 4 ? tc : tr) * (XT / 32) + (q & 3);
    cbase[i] = uniform_ptr((q >= 4 ? a.B : a.A) + r0 * nkb * kX6BlockVecs);
  }
  const int npan = ke - kb;
  // copy i (of XCOPY) of the segment's slab kp (clamped to the last)
  auto copy = [&](int kp, int i) {
    const int kpa = kb + min(kp, npan - 1);
    dma16(cbase[i >> 2] + int64_t(kpa) * kX6BlockVecs, voff[i & 3],
          lbase + uint32_t((kp % XNSLOT) * XSLOT) + uint32_t((2 * w + (i >> 2)) * 4096 + (i & 3) * 1024));
  };
  const h16x8* ring = reinterpret_cast<const h16x8*>(lds);
  auto slab = [&](int kp) { return ring + (kp % XNSLOT) * (XSLOT / 16) + lane; };
  auto read_a = [&](int kp, int i, int pl) { return slab(kp)[((wr * 2 + i) * 4 + pl) * XUNIT]; };
  auto read_b = [&](int kp, int j, int pl) { return slab(kp)[((4 + wc * 2 + j) * 4 + pl) * XUNIT]; };
  enum { RH, RL, IH, IL };            // planes re_h, re_l, im_h, im_l
  h16x8 fa[2][4], fb[2][4];           // [row block][plane], [column block][plane]
  f16v ar[2][2], ai[2][2], ap[2][2];  // chain accumulators of re and im; K1 of the corrections
#pragma unroll
  for (int s = 0; s < XDIST; ++s)
#pragma unroll
    for (int i = 0; i < XCOPY; ++i) copy(s, i);
  QST_VMCNT((XDIST - 1) * XCOPY);
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int pl = 0; pl < 4; ++pl) {
    fa[0][pl] = read_a(0, 0, pl);
    fb[0][pl] = read_b(0, 0, pl);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) ap[i][j][v] = 0.f;
  // the block folded by a chain's first panel: the last one of a panel with f = 1
#pragma unroll
  for (int v = 0; v < 16; ++v) ar[1][1][v] = ai[1][1][v] = 0.f;
  auto fold = [&](int i, int j, int x) {
    if (x < 16) re[i][j][x] += ar[i][j][x];
    else im[i][j][x - 16] += ai[i][j][x - 16];
  };
  // one panel; FIRST / LAST of its chain, first column block F
  auto panel = [&](auto first_c, auto last_c, auto f_c, int kp) {
    constexpr bool FIRST = decltype(first_c)::value, LAST = decltype(last_c)::value;
    constexpr int F = decltype(f_c)::value;
    // every slab is XCOPY copies per wave, so slab kp + 1 is complete once at
    // most XDIST - 2 newer slabs are outstanding
    QST_VMCNT((XDIST - 2) * XCOPY);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    h16x8 sh, sl;                  // Ar + Ai of the row block
    h16x8 dh, dl, nh, nl, nb;      // Bi - Br, -(Br + Bi) (h and l), -Bi_h of the column block
    h16x8 mr;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = b >> 1, j = (b == 0 || b == 3) ? F : 1 - F;
      const int pi = b == 0 ? 1 : (b - 1) >> 1, pj = b == 0 ? 1 - F : (b == 1 ? F : 1 - F);  // the block before
      const h16x8(&A)[4] = fa[i];
      const h16x8(&B)[4] = fb[j];
      f16v &R = ar[i][j], &I = ai[i][j], &K = ap[i][j];
      f16v z;
#pragma unroll
      for (int v = 0; v < 16; ++v) z[v] = 0.f;
      // ten steps of one MFMA each, with what later steps need formed in its
      // shadow (at most seven vector instructions fit one MFMA)
#pragma unroll
      for (int m = 0; m < 10; ++m) {
        if constexpr (HERK) {
          if (m == 0) R = mfma32(A[RH], B[RH], FIRST ? z : R);
          if (m == 1) I = mfma32(A[IH], B[RH], FIRST ? z : I);
          if (m == 2) R = mfma32(A[IH], B[IH], R);
          if (m == 3) I = mfma32(A[RH], nb, I);
          if (m == 5) R = mfma32(A[IH], dl, R);
          if (m == 6) I = mfma32(A[RH], nl, I);
          if (m == 8) R = mfma32(A[IL], dh, R);
          if (m == 9) I = mfma32(A[RL], nh, I);
        } else {
          if (m == 0) I = mfma32(A[RH], B[IH], FIRST ? z : I);
          if (m == 1) R = mfma32(A[RH], B[RH], FIRST ? z : R);
          if (m == 2) I = mfma32(A[IH], B[RH], I);
          if (m == 3) R = mfma32(A[IH], nb, R);
          if (m == 5) I = mfma32(A[RH], dl, I);
          if (m == 6) R = mfma32(A[IH], nl, R);
          if (m == 8) I = mfma32(A[RL], dh, I);
          if (m == 9) R = mfma32(A[IL], nh, R);
        }
        if (m == 4) K = mfma32(sh, B[RL], K);
        if (m == 7) K = mfma32(sl, B[RH], K);
        if (b != 2) {
          if (m == 0) nb = negated(B[IH]);
          if (m == 1) mr = negated(B[RL]);
          if (m == 2) dl = B[IL] + mr;
          if (m == 3) nl = negated(B[IL]);
          if (m == 4) nl = nl + mr;
          if (m == 5) mr = negated(B[RH]);
          if (m == 6) dh = B[IH] + mr;
          if (m == 7) nh = nb + mr;
        }
        if (b == 0 || b == 2) {
          if (m == 2) sh = A[RH] + A[IH];
          if (m == 5) sl = A[RL] + A[IL];
        }
        if (b == 0 && m < 4) fb[1 - F][m] = read_b(kp, 1 - F, m);
        if (b == 0 && m >= 4 && m < 8) fa[1][m - 4] = read_a(kp, 1, m - 4);
        if (b == 2 && m < 4) fa[0][m] = read_a(kp + 1, 0, m);
        if (b == 3 && m < 4) fb[1 - F][m] = read_b(kp + 1, 1 - F, m);
        if (b == 1 && m < XCOPY) copy(kp + XDIST, m);
        if ((b == 0 && FIRST) || (b > 0 && LAST)) {
#pragma unroll
          for (int x = 4 * m; x < 4 * m + 4; ++x)
            if (x < 32) fold(pi, pj, x);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  constexpr std::integral_constant<int, 0> f0{};
  constexpr std::integral_constant<int, 1> f1{};
  for (int c0 = 0; c0 < npan; c0 += XCHAIN) {
    const int n = min(XCHAIN, npan - c0);
    panel(yes, no, f0, c0);
    for (int k = 1; k + 1 < n; k += 2) {
      panel(no, no, f1, c0 + k);
      panel(no, no, f0, c0 + k + 1);
    }
    panel(no, yes, f1, c0 + n - 1);
  }
#pragma unroll
  for (int x = 0; x < 32; ++x) fold(1, 1, x);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        re[i][j][v] += ap[i][j][v];
        im[i][j][v] += ap[i][j][v];
      }
  // the clamped copies issued past the end land before the ring is reused
  // (or the workgroup's LDS is released), and every wave is past its reads
  QST_VMCNT(0);
  __syncthreads();
}

// G' T: one tile per workgroup.
__global__ __launch_bounds__(256, 1) void x6_hemm_kernel(XArgs a) {
  extern __shared__ __align__(16) char lds[];
  if (x6_off(a)) return;
  int tr, tc;
  x6_hemm_tile(a.d / XT, tr, tc);
  double scale = 2.0 / *a.tau;
  if (a.up) scale *= *a.up;
  float re[2][2][16], im[2][2][16];
  x6_zero(re, im);
  x6_segment<false>(a, lds, tr, tc, 0, a.kIters, re, im);
  x6_epilogue<false, 0>(a, tr, tc, re, im, scale, lds);
}

struct X6Seg {
  static __device__ __forceinline__ void run(const XArgs& a, char* lds, int tr, int tc, int kb, int ke,
                                             float (&re)[2][2][16], float (&im)[2][2][16]) {
    x6_segment<true>(a, lds, tr, tc, kb, ke, re, im);
  }
};

template <int X0G>
__global__ __launch_bounds__(256, 1) void x6_herk_kernel(XArgs a) {
  extern __shared__ __align__(16) char lds[];
  if (x6_off(a)) return;
  x6_herk_body<X6Seg, X0G>(a, lds);
}

// Slice workers holding the first and the last panel of leftover unit j.
__device__ __forceinline__ void x6_owners(const X6HerkSched& sc, int64_t j, int64_t& lo, int64_t& hi) {
  const int64_t f = j * sc.kh, l = f + sc.kh - 1, Q = sc.Q, it = sc.left_iters;
  lo = (f * Q) / it;
  while (lo + 1 < Q && x6_slice_start(lo + 1, Q, it) <= f) ++lo;
  while (lo > 0 && x6_slice_start(lo, Q, it) > f) --lo;
  hi = (l * Q) / it;
  while (hi + 1 < Q && x6_slice_start(hi + 1, Q, it) <= l) ++hi;
  while (hi > 0 && x6_slice_start(hi, Q, it) > l) --hi;
}

// The contributions to lower tile t in K order -- for each of its sk
// units, the round partial, or the slice partials in worker order -- as
// partial slots, one per next() call (-1 at the end).  finished(): a single
// workgroup wrote the tile (no contributions).
struct X6Contrib {
  const X6HerkSched& sc;
  int64_t t, s = 0, wg = 0, hi = -1, j = 0;
  __device__ X6Contrib(const X6HerkSched& sc_, int64_t t_) : sc(sc_), t(t_) {}
  __device__ bool finished() const {
    if (sc.sk != 1) return false;
    if (t < sc.main) return true;  // a round unit: the whole tile
    if (sc.tq) return sc.tq == 1;  // one transposed slice per unit: the whole tile
    int64_t lo, h;
    x6_owners(sc, t - sc.main, lo, h);
    return lo == h;  // inside one worker's slice: finished there
  }
  __device__ int64_t next() {
    while (true) {
      if (wg <= hi) {  // slice partials of leftover unit j
        if (sc.tq) return x6_slice_slot(sc, j + sc.left * wg++, 0);  // slice wg of unit j: worker j + left wg
        const int64_t first_unit = x6_slice_start(wg, sc.Q, sc.left_iters) / sc.kh;
        const int64_t slot = x6_slice_slot(sc, wg, j == first_unit ? 0 : 1);
        ++wg;
        return slot;
      }
      if (s >= sc.sk) return -1;
      const int64_t u = s * sc.ntiles + t;
      ++s;
      if (u < sc.main) return x6_unit_slot(u);
      j = u - sc.main;
      if (sc.tq) {
        wg = 0;
        hi = sc.tq - 1;
      } else {
        x6_owners(sc, j, wg, hi);
      }
    }
  }
};

// Fix-up: workgroup (t, q) adds quadrant q (64 x 64, the data of wave q of
// the product kernel) of the contributions to lower tile t in K order and
// applies the epilogue to it (rho, or the first POVM pass); the upper
// quadrant of a diagonal tile is the mirror of the lower one and skipped.
// Tiles go in reverse order: the leftover units, whose tiles carry the most
// contributions, belong to the last tiles, which thus start first.  Thread
// th holds values 4 (th + 256 m) + c, m < 8, c < 4, of the quadrant's
// 8192-float block (layout of x6_store_partial with w = q), loaded as
// 16-byte vectors; the loads of two contributions are in flight before they
// are added, in order.
template <int X0G>
__global__ __launch_bounds__(256, 3) void x6_fixup_kernel(XArgs a) {
  __shared__ __align__(16) Cx<float> L[64 * 64];
  __shared__ double red[4];
  if (x6_off(a)) return;
  const X6HerkSched& sc = a.sc;
  const int64_t t = sc.ntiles - 1 - (blockIdx.x >> 2);
  const int q = blockIdx.x & 3, qr = q >> 1, qc = q & 1;
  int tr, tc;
  tri_decode(t, tr, tc);
  const bool skip = tr == tc && qr < qc;  // mirror quadrant of a diagonal tile
  const int th = threadIdx.x;
  X6Contrib it(sc, t);
  if (blockIdx.x != 0 && (skip || it.finished())) return;
  // tau's partial sums (x6_tau's order), loaded now so that their latency
  // overlaps the contributions' loads; workgroup 0 also stores tau
  double tp[kReduceBlocks / 256];
#pragma unroll
  for (int k = 0; k < kReduceBlocks / 256; ++k) tp[k] = a.tau_part[th + 256 * k];
  if (blockIdx.x == 0 && (skip || it.finished())) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kReduceBlocks / 256; ++k) acc += tp[k];
    const double tau = block_sum256(acc, red);
    if (th == 0 && a.tau_out) *a.tau_out = tau;
    return;
  }
  __shared__ double diag[256];
  if (tr == tc && qr == qc) x6_diag_sums<64>(a, int64_t(tr) * XT + qr * 64, diag);
  f4v acc[8], v[2][8];
#pragma unroll
  for (int m = 0; m < 8; ++m) acc[m] = f4v{0.f, 0.f, 0.f, 0.f};
  // two contributions in flight (most tiles have two), then added in order
  while (true) {
    int64_t sl[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) sl[k] = it.next();
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (sl[k] >= 0) {
        const f4v* src = reinterpret_cast<const f4v*>(x6_slot(a, sl[k]) + q * 8192);
#pragma unroll
        for (int m = 0; m < 8; ++m) v[k][m] = src[th + 256 * m];
      }
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (sl[k] >= 0) {
#pragma unroll
        for (int m = 0; m < 8; ++m) acc[m] += v[k][m];
      }
    if (sl[1] < 0) break;
  }
  double tacc = 0.0;
#pragma unroll
  for (int k = 0; k < kReduceBlocks / 256; ++k) tacc += tp[k];
  const double tau = block_sum256(tacc, red);
  __shared__ double tau_sh;
  if (th == 0) {
    tau_sh = tau;
    if (blockIdx.x == 0 && a.tau_out) *a.tau_out = tau;
  }
  __syncthreads();
  const double scale = 1.0 / tau_sh;
  // vector th + 256 m of the quadrant holds values 4 vq + c of block
  // ij = m / 2, part m % 2, lane th % 64, vq = th / 64
  const int lane = th & 63, vq = th >> 6;
  float rs[2][4], cs[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4)
      rs[i][c4] = a.sa[int64_t(tr) * XT + qr * 64 + i * 32 + 8 * vq + 4 * (lane >> 5) + c4];
    cs[i] = float(scale * double(a.sb[int64_t(tc) * XT + qc * 64 + i * 32 + (lane & 31)]));
  }
  if constexpr (X0G == 0) {
    Cx<float>* C = static_cast<Cx<float>*>(a.C);
    float* Cf = reinterpret_cast<float*>(C);
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int c4 = 0; c4 < 4; ++c4) {
        const int part = m & 1, vv = 4 * vq + c4, ij = m >> 1;
        const int i = ij >> 1, j = ij & 1;
        const int64_t r = int64_t(tr) * XT + qr * 64 + i * 32 + 8 * (vv >> 2) + 4 * (lane >> 5) + (vv & 3);
        const int64_t c = int64_t(tc) * XT + qc * 64 + j * 32 + (lane & 31);
        float x = acc[m][c4] * cs[j] * rs[i][c4];
        if (i == j && r == c) x = part ? 0.f : x6_diag<64>(diag, int(r & 63), scale);
        Cf[2 * (r * a.ldc + c) + part] = x;
        // the mirror: every off-diagonal tile, and the lower-left quadrant
        // of a diagonal tile (whose upper-right quadrant is not computed here)
        if (tr != tc || qr != qc) Cf[2 * (c * a.ldc + r) + part] = part ? -x : x;
      }
  } else {
    constexpr int G = X0G;
    constexpr int S = 64 >> G;
    constexpr int TG = 1 << (2 * G);
    constexpr int M = (1 << G) - 1;
    float* Lf = reinterpret_cast<float*>(L);
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int c4 = 0; c4 < 4; ++c4) {
        const int part = m & 1, vv = 4 * vq + c4, ij = m >> 1;
        const int i = ij >> 1, j = ij & 1;
        const int r = i * 32 + 8 * (vv >> 2) + 4 * (lane >> 5) + (vv & 3), c = j * 32 + (lane & 31);
        float x = acc[m][c4] * cs[j] * rs[i][c4];
        if (i == j && tr == tc && qr == qc && r == c) x = part ? 0.f : x6_diag<64>(diag, r, scale);
        Lf[2 * (((r >> G) * S + (c >> G)) * TG + swz<G>(r & M, c & M)) + part] = x;
      }
    __syncthreads();
    gemm::GemmArgs g{};
    g.x0 = a.x0;
    g.x0g = a.x0g;
    g.x0up = a.x0up;
    gemm::x0_rounds<float, G>(g, int64_t(2) * tr + qr, int64_t(2) * tc + qc, L);
  }
}

// ---------------------------------------------------------------------------
// 64 x 64 tiles (d <= 1024): at d = 1024 G' T has 64 tiles of 128 x 128 for
// 256 compute units, and T T^dagger 36, which only a split of K could spread
// (54.7 us, and 25.6 us with 15.9 us to add the partials); 256 and 136 tiles
// of 64 x 64 need no split.  Per MFMA they read twice the LDS bytes and
// stream twice the operand bytes, still below what the LDS and the L2 give.
// Four waves of one 32 x 32 block each; the slabs are 16 KB, and the copies
// run seven of them ahead.  Fragments alternate between two buffers.
// ---------------------------------------------------------------------------
constexpr int YT = kX6SmallTile;
constexpr int YSLOT = 16 * 1024;      // 16 units: 2 row blocks of A and of B
constexpr int YNSLOT = 8;
constexpr int YDIST = YNSLOT - 1;
constexpr int YCOPY = 4;              // units copied per wave and slab
constexpr int YCHAIN = 4;             // panels per accumulation chain (of 8 at d = 128; as XCHAIN)
static_assert(YSLOT * YNSLOT == XLDS, "one dynamic LDS size");
static_assert((YDIST - 1) * YCOPY < 64, "vmcnt immediate");

// All panels of output tile (tr, tc): (re, im) of the wave's block.
template <bool HERK>
__device__ __forceinline__ void x6_tile64(const XArgs& a, char* lds, int tr, int tc, float (&re)[16], float (&im)[16]) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w >> 1, wc = w & 1;
  const int npan = a.d / 16;
  const uint32_t lbase = __builtin_amdgcn_readfirstlane(lds_address(lds));
  uint32_t voff[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) voff[u] = uint32_t(lane) * 16 + u * 1024;
  const u16x8* cbase =
      uniform_ptr((w >= 2 ? a.B : a.A) + (int64_t(w >= 2 ? tc : tr) * (YT / 32) + (w & 1)) * npan * kX6BlockVecs);
  auto copy = [&](int kp, int i) {
    dma16(cbase + int64_t(min(kp, npan - 1)) * kX6BlockVecs, voff[i],
          lbase + uint32_t((kp % YNSLOT) * YSLOT) + uint32_t(w * 4096 + i * 1024));
  };
  const h16x8* ring = reinterpret_cast<const h16x8*>(lds);
  auto read = [&](int kp, int rb, int pl) { return ring[(kp % YNSLOT) * (YSLOT / 16) + (rb * 4 + pl) * XUNIT + lane]; };
  enum { RH, RL, IH, IL };
  h16x8 fa[2][4], fb[2][4];  // [buffer][plane]
  f16v R, I, K;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    re[v] = im[v] = 0.f;
    R[v] = I[v] = K[v] = 0.f;
  }
#pragma unroll
  for (int s = 0; s < YDIST; ++s)
#pragma unroll
    for (int i = 0; i < YCOPY; ++i) copy(s, i);
  QST_VMCNT((YDIST - 1) * YCOPY);
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int pl = 0; pl < 4; ++pl) {
    fa[0][pl] = read(0, wr, pl);
    fb[0][pl] = read(0, 2 + wc, pl);
  }
  auto panel = [&](auto buf_c, int kp) {
    constexpr int BUF = decltype(buf_c)::value;
    QST_VMCNT((YDIST - 2) * YCOPY);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const h16x8(&A)[4] = fa[BUF];
    const h16x8(&B)[4] = fb[BUF];
    h16x8 sh, sl, dh, dl, nh, nl, nb, mr;
#pragma unroll
    for (int m = 0; m < 10; ++m) {
      if constexpr (HERK) {
        if (m == 0) R = mfma32(A[RH], B[RH], R);
        if (m == 1) I = mfma32(A[IH], B[RH], I);
        if (m == 2) R = mfma32(A[IH], B[IH], R);
        if (m == 3) I = mfma32(A[RH], nb, I);
        if (m == 5) R = mfma32(A[IH], dl, R);
        if (m == 6) I = mfma32(A[RH], nl, I);
        if (m == 8) R = mfma32(A[IL], dh, R);
        if (m == 9) I = mfma32(A[RL], nh, I);
      } else {
        if (m == 0) I = mfma32(A[RH], B[IH], I);
        if (m == 1) R = mfma32(A[RH], B[RH], R);
        if (m == 2) I = mfma32(A[IH], B[RH], I);
        if (m == 3) R = mfma32(A[IH], nb, R);
        if (m == 5) I = mfma32(A[RH], dl, I);
        if (m == 6) R = mfma32(A[IH], nl, R);
        if (m == 8) I = mfma32(A[RL], dh, I);
        if (m == 9) R = mfma32(A[IL], nh, R);
      }
      if (m == 4) K = mfma32(sh, B[RL], K);
      if (m == 7) K = mfma32(sl, B[RH], K);
      if (m == 0) nb = negated(B[IH]);
      if (m == 1) mr = negated(B[RL]);
      if (m == 2) dl = B[IL] + mr;
      if (m == 2) sh = A[RH] + A[IH];
      if (m == 3) nl = negated(B[IL]);
      if (m == 4) nl = nl + mr;
      if (m == 5) mr = negated(B[RH]);
      if (m == 5) sl = A[RL] + A[IL];
      if (m == 6) dh = B[IH] + mr;
      if (m == 7) nh = nb + mr;
      // the next slab's fragments first: they are needed right after this panel
      if (m < 4) {
        fa[1 - BUF][m] = read(kp + 1, wr, m);
        fb[1 - BUF][m] = read(kp + 1, 2 + wc, m);
      } else if (m < 4 + YCOPY) {
        copy(kp + YDIST, m - 4);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr std::integral_constant<int, 0> b0{};
  constexpr std::integral_constant<int, 1> b1{};
  for (int c0 = 0; c0 < npan; c0 += YCHAIN) {  // npan is a multiple of 2
    const int end = min(npan, c0 + YCHAIN);
    for (int kp = c0; kp < end; kp += 2) {
      panel(b0, kp);
      panel(b1, kp + 1);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      re[v] += R[v];
      im[v] += I[v];
      R[v] = I[v] = 0.f;
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    re[v] += K[v];
    im[v] += K[v];
  }
  QST_VMCNT(0);
  __syncthreads();
}

__global__ __launch_bounds__(256, 1) void x6_hemm64_kernel(XArgs a) {
  extern __shared__ __align__(16) char lds[];
  if (x6_off(a)) return;
  int tr, tc;
  x6_hemm_tile(a.d / YT, tr, tc);
  double scale = 2.0 / *a.tau;
  if (a.up) scale *= *a.up;
  float re[16], im[16];
  x6_tile64<false>(a, lds, tr, tc, re, im);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t r0 = int64_t(tr) * YT + (w >> 1) * 32 + 4 * (lane >> 5), c = int64_t(tc) * YT + (w & 1) * 32 + (lane & 31);
  const float cs = float(scale * double(a.sb[c]));
  Cx<float>* C = static_cast<Cx<float>*>(a.C);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t r = r0 + 8 * (v >> 2) + (v & 3);
    const float rs = a.sa[r];
    C[r * a.ldc + c] = Cx<float>{re[v] * cs * rs, im[v] * cs * rs};
  }
}

// One lower tile per workgroup: rho (X0G 0), or the first POVM pass.
template <int X0G>
__global__ __launch_bounds__(256, 1) void x6_herk64_kernel(XArgs a) {
  extern __shared__ __align__(16) char lds[];
  if (x6_off(a)) return;
  int tr, tc;
  tri_decode(xcd_order(blockIdx.x, gridDim.x), tr, tc);
  float re[16], im[16];
  x6_tile64<true>(a, lds, tr, tc, re, im);
  const double tau = x6_tau(a, lds);
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.tau_out) *a.tau_out = tau;
  const double scale = 1.0 / tau;
  const int64_t R0 = int64_t(tr) * YT, C0 = int64_t(tc) * YT;
  double* diag = reinterpret_cast<double*>(lds + 64 * 64 * sizeof(Cx<float>));
  if (tr == tc) {
    x6_diag_sums<64>(a, R0, diag);
    __syncthreads();
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int rl = (w >> 1) * 32 + 4 * (lane >> 5), c = (w & 1) * 32 + (lane & 31);
  const float cs = float(scale * double(a.sb[C0 + c]));
  Cx<float>* L = reinterpret_cast<Cx<float>*>(lds);
  Cx<float>* C = static_cast<Cx<float>*>(a.C);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = rl + 8 * (v >> 2) + (v & 3);
    const float rs = a.sa[R0 + r];
    Cx<float> x{re[v] * cs * rs, im[v] * cs * rs};
    if (tr == tc && r == c) x = Cx<float>{x6_diag<64>(diag, r, scale), 0.f};
    if constexpr (X0G == 0) {
      C[(R0 + r) * a.ldc + C0 + c] = x;
      if (tr != tc) C[(C0 + c) * a.ldc + R0 + r] = Cx<float>{x.re, -x.im};
    } else {
      constexpr int G = X0G, S = 64 >> G, TG = 1 << (2 * G), M = (1 << G) - 1;
      L[((r >> G) * S + (c >> G)) * TG + swz<G>(r & M, c & M)] = x;
    }
  }
  if constexpr (X0G != 0) {
    __syncthreads();
    gemm::GemmArgs g{};
    g.x0 = a.x0;
    g.x0g = a.x0g;
    g.x0up = a.x0up;
    gemm::x0_rounds<float, X0G>(g, tr, tc, L);
  }
}

unsigned x6_split_grid(int d) { return unsigned(int64_t(d / 32) * (d / 128)); }

template <int X0G>
hipError_t x6_run_herk(const XArgs& a, bool small, hipStream_t s) {
  if (small) {
    hipError_t e = x6_allow_lds<x6_herk64_kernel<X0G>, XLDS>();
    if (e != hipSuccess) return e;
    const int ts = a.d / YT;
    x6_herk64_kernel<X0G><<<unsigned(ts * (ts + 1) / 2), 256, XLDS, s>>>(a);
    return hipGetLastError();
  }
  hipError_t e = x6_allow_lds<x6_herk_kernel<X0G>, XLDS>();
  if (e != hipSuccess) return e;
  const int64_t grid = a.sc.rounds > 0 ? a.sc.P : a.sc.Q;
  x6_herk_kernel<X0G><<<unsigned(grid), 256, XLDS, s>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t x6_launch_fixup(const XArgs& a, int x0g, hipStream_t s) {
  const unsigned grid = unsigned(a.ntiles) * 4;
  if (x0g == 6) x6_fixup_kernel<6><<<grid, 256, 0, s>>>(a);
  else if (x0g == 5) x6_fixup_kernel<5><<<grid, 256, 0, s>>>(a);
  else if (x0g == 4) x6_fixup_kernel<4><<<grid, 256, 0, s>>>(a);
  else x6_fixup_kernel<0><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_x6_herk(qst_prec prec, const void* T, int64_t ldt, void* rho, int64_t ldr, int n,
                          double* tau_partials, const void* f, double* tau_dev, void* planes, void* partials,
                          hipStream_t s, const Pass0Out* x0, void* tt_planes, X6Gate* sparse) {
  const int d = 1 << n;
  if (d < kX6Tile || !tau_partials) return hipErrorInvalidValue;
  if (x0 && (x0->g < 4 || x0->g > 6 || !x0->tetra)) return hipErrorInvalidValue;
  u16x8* P = static_cast<u16x8*>(x6_herk_planes(planes, n));
  const X6Scales sc = x6_herk_scales(planes, n);
  hipError_t e;
  {
    ProfScope prof("x6_split_t", s);
    const Cx<float>* Tf = static_cast<const Cx<float>*>(T);
    const float* ff = static_cast<const float*>(f);
    u16x8* PT = static_cast<u16x8*>(tt_planes);
    const float low = x6_dense_low(n);
    if (f) x6_absmax_t_kernel<true><<<kReduceBlocks, 256, 0, s>>>(Tf, ldt, d, sc, tau_partials, ff);
    else x6_absmax_t_kernel<false><<<kReduceBlocks, 256, 0, s>>>(Tf, ldt, d, sc, tau_partials, ff);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (PT) x6_split_t_kernel<true><<<x6_split_grid(d), 256, 0, s>>>(Tf, ldt, d, sc, P, PT, low);
    else x6_split_t_kernel<false><<<x6_split_grid(d), 256, 0, s>>>(Tf, ldt, d, sc, P, PT, low);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  ProfScope prof("herk_x6", s);
  const bool small = x6_small_tiles(n);
  XArgs a{};
  a.A = P;
  a.B = P;
  a.gate = X6Gate{{sc.bad, sc.bad}, {sc.near + 1, sc.near + 1}, d / 8};  // T's rows on both sides
  if (sparse) *sparse = a.gate;
  a.when = kX6Dense;
  a.sa = sc.rinv;
  a.sb = sc.rinv;
  a.rsum = sc.rsum;
  a.C = rho;
  a.ldc = ldr;
  a.d = d;
  a.tau = tau_dev;
  a.tau_part = tau_partials;
  a.tau_out = tau_dev;
  a.part = static_cast<float*>(partials);
  a.ntiles = (d / XT) * (d / XT + 1) / 2;
  a.kIters = d / 16;
  a.sc = x6_herk_sched(n, x6_cus());
  const int g = x0 ? x0->g : 0;
  if (x0) {
    a.x0 = x0->X;
    a.x0g = x0->g;
    a.x0up = n - x0->g;
  }
  e = g == 6   ? x6_run_herk<6>(a, small, s)
      : g == 5 ? x6_run_herk<5>(a, small, s)
      : g == 4 ? x6_run_herk<4>(a, small, s)
               : x6_run_herk<0>(a, small, s);
  if (e != hipSuccess) return e;
  if (prec == QST_F32) return small ? hipSuccess : x6_launch_fixup(a, g, s);
  // QST_F32X6, T not dense: its partial tiles take the same fix-up
  if ((e = x3_launch_herk(a, T, ldt, g, P, sc.rinv, s)) != hipSuccess) return e;
  a.when = small ? kX6Sparse : kX6Always;
  return x6_launch_fixup(a, g, s);
}

hipError_t launch_x6_hemm(qst_prec prec, const void* G, int64_t ldg, const void* T, int64_t ldt, void* out,
                          int64_t ldo, int n, const double* tau_dev, const double* upstream_dev, void* planes,
                          hipStream_t s, const X6Scales* t_ready, X6Gate* sparse) {
  const int d = 1 << n;
  if (d < kX6Tile || !planes) return hipErrorInvalidValue;
  u16x8* PG = static_cast<u16x8*>(x6_hemm_planes(planes, n));
  u16x8* PT = PG + x6_plane_bytes(n) / sizeof(u16x8);
  hipError_t e;
  const X6Pair p{{static_cast<const Cx<float>*>(G), static_cast<const Cx<float>*>(T)},
                 {ldg, ldt},
                 {x6_hemm_scales(planes, n, 0), t_ready ? *t_ready : x6_hemm_scales(planes, n, 1)},
                 {PG, PT},
                 x6_dense_low(n)};
  {
    ProfScope prof("x6_split_gt", s);
    const unsigned mg = unsigned(std::min<int64_t>(kReduceBlocks, int64_t(d / 64) * (d / 64))), ny = t_ready ? 1 : 2;
    x6_absmax_gt_kernel<<<dim3(mg, ny), 256, 0, s>>>(p, d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    x6_split_gt_kernel<<<dim3(x6_split_grid(d), ny), 256, 0, s>>>(p, d, int(mg));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const bool small = x6_small_tiles(n);
  if ((e = small ? x6_allow_lds<x6_hemm64_kernel, XLDS>() : x6_allow_lds<x6_hemm_kernel, XLDS>()) != hipSuccess)
    return e;
  XArgs a{};
  a.A = PG;
  a.B = PT;
  a.gate = X6Gate{{p.sc[0].bad, p.sc[1].bad + 1}, {p.sc[0].near + 1, p.sc[1].near}, d / 8};
  if (sparse) *sparse = a.gate;
  a.when = kX6Dense;
  a.sa = p.sc[0].rinv;
  a.sb = p.sc[1].cinv;
  a.C = out;
  a.ldc = ldo;
  a.d = d;
  a.tau = tau_dev;
  a.up = upstream_dev;
  a.kIters = d / 16;
  const int ts = d / (small ? YT : XT);
  {
    ProfScope prof("hemm_x6", s, true);
    hipExtLaunchKernelGGL(small ? x6_hemm64_kernel : x6_hemm_kernel, dim3(unsigned(ts * ts)), dim3(256), XLDS, s,
                          prof.start(), prof.stop(), 0, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (prec == QST_F32) return hipSuccess;
  return x3_launch_hemm(a, G, ldg, T, ldt, PG, p.sc[0].rinv, p.sc[1].cinv, s);
}

}  // namespace qst
