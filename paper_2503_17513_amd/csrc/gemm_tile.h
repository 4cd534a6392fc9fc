// What the tiled GEMM kernels share: vector types, LDS swizzle, rounding.
#pragma once
#include "dma.h"

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

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const bf16x2 p = __builtin_convertvector(f32x2{a, b}, bf16x2);     // v_cvt_pk_bf16_f32: round half to even
    return __builtin_bit_cast(uint32_t, p);
}

}  // namespace
}  // namespace pme
