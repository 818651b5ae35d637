// Pieces shared by the split product kernels (k_xgemm.hip) and the batched
// kernel's split products (k_batch.hip): the asynchronous global -> LDS copy,
// its waits, the MFMA and the operand sums of the correction products.
#pragma once

#include "qst_device.h"
#include "qst_split.h"

namespace qst {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

// A wave-uniform pointer moved into scalar registers.  The builtin takes
// and returns a signed 32-bit value per half; each half is taken back as
// unsigned, so that the high half is not sign-extended over.
__device__ __forceinline__ const u16x8* uniform_ptr(const u16x8* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(u)));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(u >> 32)));
  return reinterpret_cast<const u16x8*>((uint64_t(hi) << 32) | uint64_t(lo));
}

// global -> LDS copy of one 16-byte vector per lane into the 1 KB at LDS
// byte address lds (wave-uniform).  Written as an asm statement so that the
// compiler's wait-count pass, which cannot tell ring slots apart, does not
// order every LDS read after every such copy; the kernel waits for them
// itself (vmcnt) before the barrier that publishes a slab.  Nothing is
// written to registers.
// sbase: wave-uniform base address (SGPR pair); voff: the lane's byte offset.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds) {
  uint32_t m0v;  // M0 is an output of the statement, so the compiler keeps no value of its own there
  asm volatile("s_mov_b32 %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               : "={m0}"(m0v)
               : "v"(voff), "s"(sbase), "s"(lds)
               : "memory");
  (void)m0v;
}
// LDS byte address of a pointer into the workgroup's shared memory
__device__ __forceinline__ uint32_t lds_address(const char* p) {
  return (uint32_t)(uintptr_t)(lds_void_t*)p;
}
// s_waitcnt vmcnt(n), other counters unconstrained (gfx9 encoding)
#define QST_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0f70 | ((n) & 15) | (((n) >> 4) << 14))

__device__ __forceinline__ f16v mfma32(h16x8 a, h16x8 b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f16v mfma32b(u16x8 a, u16x8 b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// -x.  The empty statement hides the sign flip from the compiler, which
// would otherwise fold it into the sum it is used in and take that apart
// into scalar subtractions (three instructions for one packed addition).
__device__ __forceinline__ h16x8 negated(h16x8 x) {
  u32x4 v = __builtin_bit_cast(u32x4, x) ^ 0x80008000u;
  asm("" : "+v"(v));
  return __builtin_bit_cast(h16x8, v);
}

}  // namespace qst
