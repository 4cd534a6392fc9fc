// DMA from global memory into LDS and the waits on it, as inline assembly so that the compiler does not order other LDS
// accesses after them.
#pragma once
#include "pme_internal.h"

namespace pme {
namespace {

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

}  // namespace
}  // namespace pme
