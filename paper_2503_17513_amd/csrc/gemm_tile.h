// What the tiled int4 GEMM kernels share: vector types, LDS swizzle, DMA and waits.
#pragma once
#include "pme_internal.h"

namespace pme {
namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

#define PME_AS1 __attribute__((address_space(1)))
#define PME_AS3 __attribute__((address_space(3)))

enum { MODE_BF16 = 0, MODE_ASYM = 1, MODE_I32 = 2 };

// LDS swizzle: the 16-byte chunk kc of tile row r sits at chunk position kc ^ swz(r), so that the rows
// read together by one ds_read_b128 spread over the banks.  RB = bytes per tile row per K step.  The two
// functions are the fastest of the XOR patterns tried on MI355X (timed in the whole kernel, where the
// pattern also decides which global chunk each DMA lane fetches).
template <int RB> __device__ __forceinline__ int swz(int r) {
    return RB == 64 ? (((r >> 2) ^ r) & 3) : (r & 7);
}

// LDS-only barrier: DMA (counted by vmcnt) stays in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// 16 bytes per lane from global memory straight into LDS at lds_base + 16 * lane (lds_base wave-uniform).
// The statement overwrites M0, which the compiler reserves and does not keep values in; no other code in
// these kernels makes the compiler emit an M0 use.
// The source is a wave-uniform 64-bit base (SGPR pair) plus a 32-bit byte offset per lane: no vector
// arithmetic is needed to move the window along K.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_base) : "memory");
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const bf16x2 p = __builtin_convertvector(f32x2{a, b}, bf16x2);     // v_cvt_pk_bf16_f32: round half to even
    return __builtin_bit_cast(uint32_t, p);
}

}  // namespace
}  // namespace pme
