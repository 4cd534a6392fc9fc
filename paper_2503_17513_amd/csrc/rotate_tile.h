// What the kernels that rotate a token share: the in-register butterflies, the reduction of a token's range, the layout of a bf16
// token in LDS, and the codes.
#pragma once
#include "dma.h"

namespace pme {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

template <int KLOG2> struct Layout {
    static constexpr int NC = 1 << KLOG2;      // FWHT length
    static constexpr int MT = NC / 16;         // 16-row MFMA tiles along c
    static constexpr int NREG = MT * 4;        // values per lane per a'-tile
    static constexpr int NBITS = KLOG2 - 2;    // register index bits
    static constexpr int RUN = NC / 4;         // contiguous outputs per lane after the FWHT
    // Position (within the lane's contiguous run) of register index idx after the FWHT.
    // Before: idx bit 0,1 = c0,c1; idx bits 2.. = c4..c(k-1); lane bit 4 = c2, lane bit 5 = c3.
    // After (k >= 6): the two top idx bits hold c2, c3; lane bits 4, 5 hold c(k-2), c(k-1).
    // After (k == 5): idx bits = c0, c1, c2; lane bit 4 = c4, lane bit 5 = c3.
    static constexpr int run_pos(int idx) {
        if (KLOG2 == 5) return idx;
        int lo = idx & 3;
        int mid = (idx >> 2) & ((1 << (NBITS - 4)) - 1);     // c4 .. c(k-3)
        int c2 = (idx >> (NBITS - 2)) & 1, c3 = (idx >> (NBITS - 1)) & 1;
        return lo | (c2 << 2) | (c3 << 3) | (mid << 4);
    }
    // inverse of run_pos as a constant table, so that an unrolled loop indexes registers with constants
    struct Table { int v[NC / 4]; };
    static constexpr Table make_table() {
        Table t{};
        for (int idx = 0; idx < NREG; ++idx) t.v[run_pos(idx)] = idx;
        return t;
    }
    static constexpr Table kRegOfRun = make_table();
    static constexpr int reg_of_run_pos(int j) { return kRegOfRun.v[j]; }
};

// lane bit 4 (5) <-> the register bit that distinguishes r0 / r1
__device__ __forceinline__ void swap16(uint32_t& r0, uint32_t& r1) {
    const u32x2 v = __builtin_amdgcn_permlane16_swap(r0, r1, false, false);
    r0 = v.x;
    r1 = v.y;
}
__device__ __forceinline__ void swap32(uint32_t& r0, uint32_t& r1) {
    const u32x2 v = __builtin_amdgcn_permlane32_swap(r0, r1, false, false);
    r0 = v.x;
    r1 = v.y;
}
__device__ __forceinline__ void swap16(float& r0, float& r1) {
    uint32_t a = __float_as_uint(r0), b = __float_as_uint(r1);
    swap16(a, b);
    r0 = __uint_as_float(a);
    r1 = __uint_as_float(b);
}
__device__ __forceinline__ void swap32(float& r0, float& r1) {
    uint32_t a = __float_as_uint(r0), b = __float_as_uint(r1);
    swap32(a, b);
    r0 = __uint_as_float(a);
    r1 = __uint_as_float(b);
}

template <int NREG, int BIT> __device__ __forceinline__ void butterfly(float (&v)[NREG]) {
#pragma unroll
    for (int i = 0; i < NREG; ++i)
        if (!(i & (1 << BIT))) {
            const float u = v[i], w = v[i | (1 << BIT)];
            v[i] = u + w;
            v[i | (1 << BIT)] = u - w;
        }
}
template <int NREG, int BIT> __device__ __forceinline__ void lane_swap16(float (&v)[NREG]) {
#pragma unroll
    for (int i = 0; i < NREG; ++i)
        if (!(i & (1 << BIT))) swap16(v[i], v[i | (1 << BIT)]);
}
template <int NREG, int BIT> __device__ __forceinline__ void lane_swap32(float (&v)[NREG]) {
#pragma unroll
    for (int i = 0; i < NREG; ++i)
        if (!(i & (1 << BIT))) swap32(v[i], v[i | (1 << BIT)]);
}

template <int NREG, int BIT> struct RegStages {
    static __device__ __forceinline__ void run(float (&v)[NREG]) {
        butterfly<NREG, BIT>(v);
        RegStages<NREG, BIT - 1>::run(v);
    }
};
template <int NREG> struct RegStages<NREG, -1> {
    static __device__ __forceinline__ void run(float (&)[NREG]) {}
};

template <int KLOG2> __device__ __forceinline__ void fwht_lane(float (&v)[Layout<KLOG2>::NREG]) {
    using L = Layout<KLOG2>;
    RegStages<L::NREG, L::NBITS - 1>::run(v);          // every c bit that starts in a register
    if constexpr (KLOG2 == 5) {
        lane_swap16<L::NREG, 2>(v);                    // idx bit 2: c4 -> c2
        butterfly<L::NREG, 2>(v);
        lane_swap32<L::NREG, 2>(v);                    // idx bit 2: c2 -> c3 (lane bit 5 now c2)
        butterfly<L::NREG, 2>(v);
        lane_swap32<L::NREG, 2>(v);                    // back: idx bit 2 = c2, lane bit 5 = c3
    } else {
        lane_swap16<L::NREG, L::NBITS - 2>(v);
        lane_swap32<L::NREG, L::NBITS - 1>(v);
        butterfly<L::NREG, L::NBITS - 2>(v);
        butterfly<L::NREG, L::NBITS - 1>(v);
    }
}

// First output column of this lane's run, for lane bits (l4, l5).
template <int KLOG2> __device__ __forceinline__ int run_start(int l4, int l5) {
    using L = Layout<KLOG2>;
    if (KLOG2 == 5) return 8 * l5 + 16 * l4;
    return L::RUN * (l4 + 2 * l5);
}

// Maxima over the 16 lanes of a row and over the wavefront, result in every lane, of values that are not negative: their bit
// patterns compare like unsigned integers, whose maximum takes the data-parallel move (xor 1, xor 2, mirrored halves, mirrored
// row) as an operand and needs no canonical form -- one instruction a step where the float maximum takes three.  The same steps
// through ds_bpermute cost an LDS round trip each, which no other work of the wave covers.
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
    auto step = [&](auto ctrl) { v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, decltype(ctrl)::value, 0xF, 0xF, true)); };
    step(std::integral_constant<int, 0xB1>{});     // quad_perm [1, 0, 3, 2]
    step(std::integral_constant<int, 0x4E>{});     // quad_perm [2, 3, 0, 1]
    step(std::integral_constant<int, 0x141>{});    // row_half_mirror
    step(std::integral_constant<int, 0x140>{});    // row_mirror
    return v;
}
// The maximum over both rows of each half of the wavefront.
__device__ __forceinline__ uint32_t half_max(uint32_t v) {
    v = row_max(v);
    uint32_t w = v;
    swap16(v, w);
    return max(v, w);
}
// Lower half of the wavefront: the maximum of a over the half's own lanes and their partners in the other; upper half: of b.
__device__ __forceinline__ uint32_t pair_max(uint32_t a, uint32_t b) {
    swap32(a, b);
    return max(a, b);
}
__device__ __forceinline__ uint32_t magnitude(float f) { return __float_as_uint(f) & 0x7FFFFFFFu; }

#define PME_AS1 __attribute__((address_space(1)))
#define PME_AS3 __attribute__((address_space(3)))
typedef __attribute__((ext_vector_type(4))) short s16x4;

// Physical LDS position (in 16-byte chunks) of the 8 inputs (a, c .. c+7), c a multiple of 8, in the
// bf16 layout: blocks of 4 rows x 16 columns stored contiguously (128 bytes), so that the 16 lanes of
// a transposing LDS read touch one contiguous 128-byte block.
template <int MT> __device__ __forceinline__ int chunk_of(int a, int c) {
    return ((a >> 2) * MT + (c >> 4)) * 8 + (a & 3) * 2 + ((c >> 3) & 1);
}

// Scale, reciprocal and zero point of a token from its unnormalised range: hi the largest magnitude (symmetric) or both ends.
struct TokenScale { float s, rinv; int z; };
__device__ __forceinline__ TokenScale symmetric_scale(float hi, float g7) {
    TokenScale q{1.f, 0.f, 0};
    if (hi > 0.f) {
        q.s = hi * g7;                      // absmax * gamma / 7
        q.rinv = 7.f * __builtin_amdgcn_rcpf(hi);
    }
    return q;
}
__device__ __forceinline__ TokenScale asymmetric_scale(float hi, float lo, float g15) {
    TokenScale q{1.f, 0.f, 0};
    if (hi > lo) {
        // fp32 like the symmetric case: scale = range * fp32(gamma / 15), codes from u * (15 / range)
        const float range = hi - lo;
        q.s = range * g15;
        q.rinv = 15.f * __builtin_amdgcn_rcpf(range);
        q.z = (int)__builtin_rintf(-lo * q.rinv);
        q.z = min(15, max(0, q.z));
    }
    return q;
}

// Eight codes, value(0) in the lowest nibble.
// fma(u, rinv, 1.5 * 2^23 + 8) has the bit pattern C + e with C = 0x4B400000 and e = rne(u * rinv) + 8
// in [1, 15].  Eight of them are combined by Horner steps acc = (acc << 4) + bits; the digits are
// non-negative, so no carries cross nibbles, and the accumulated constant C * 0x11111111 is
// subtracted once.  e ^ 8 is the 4-bit two's-complement code.
constexpr uint32_t kCodeSum = 0x4B400000u * 0x11111111u;
template <class F> __device__ __forceinline__ uint32_t symmetric_codes(float rinv, F value) {
    uint32_t accw = 0;
#pragma unroll
    for (int nb = 7; nb >= 0; --nb) {
        const float f = __builtin_fmaf(value(nb), rinv, 12582920.f);
        accw = (accw << 4) + __float_as_uint(f);
    }
    return (accw - kCodeSum) ^ 0x88888888u;
}
// The zero point rides in the rounding constant cz = 1.5 * 2^23 + z (rne(u rinv + z) = rne(u rinv) + z), the clamp
// to [0, 15] is one median-of-three on the float, then the same Horner packing.
template <class F> __device__ __forceinline__ uint32_t asymmetric_codes(float rinv, float cz, F value) {
    uint32_t accw = 0;
#pragma unroll
    for (int nb = 7; nb >= 0; --nb) {
        float f = __builtin_fmaf(value(nb), rinv, cz);
        f = __builtin_amdgcn_fmed3f(f, 12582912.f, 12582927.f);
        accw = (accw << 4) + __float_as_uint(f);
    }
    return accw - kCodeSum;
}

}  // namespace
}  // namespace pme
