// The int4 layer of one token in one kernel: rotate, quantize, multiply (paper Sections 3 and 4).
//
// One token through two kernels is bound by the host, which takes 3.4 us to enqueue a kernel with arguments (and 10 us for the
// call), and on the GPU by two chains of latencies with a launch between them (4.6 + 5.3 us).  Here every workgroup rotates the token
// itself and multiplies it with 16 channels, whose weights it has asked for before the rotation and finds in registers
// after it; no codes pass through memory.  Us a call in a Python loop / in a graph, three sets of operands in turn: 1 x 2048 x 8448 9.8 / 8.3 ->
// 7.2 / 6.9, 1 x 2048 x 8704 9.8 / 9.2 -> 8.0 / 7.9, 1 x 4096 x 8448 10.0 / 9.3 -> 8.1 / 8.4, 1 x 2048 x 10240 10.5 / 10.1 -> 8.5 / 8.5.  A second token costs every workgroup another 1.6 us and gains nothing any more (2 x 2048 x 8448 9.4 and
// 9.2), nor do the blocks of 256 columns, whose token is three to five waves' work (1 x 2048 x 12288 11.2 either way).
//   1. the token is fetched into LDS by DMA, the wave's block fragments and weights into registers;
//   2. base block on the matrix cores, butterflies in registers, range across the waves, codes into the token's place in LDS, as
//      k_rotate_mfma does them (a wave owns one 16-wide tile of the block): the codes are the same bits;
//   3. the waves split K: 64-byte chunks of weights and codes on v_mfma_i32_16x16x64_i8, unpacked as in k_gemm_decode;
//      partial sums are added through LDS.
#include "rotate_tile.h"

#include <cmath>

namespace pme {
namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int kMostWaves = 10;       // waves, each a 16-wide tile of the block

struct TokenArgs {
    const uint16_t* x;
    int d, d_e, b;
    const u32x4* ptable;             // the block's fragment (tile, ks) at (tile stride + ks) 64 + lane
    int stride;
    float g;                         // gamma / 7, asymmetric gamma / 15
    const uint8_t* qw;
    const float* sw;
    const int32_t* wsum;             // asymmetric, else null
    int N;
    uint16_t* y;
};

// KS: K steps of the base block.  KB: 64-byte chunks of a wave's share of K, at most.
template <int KLOG2, int KS, bool ASYM, int KB>
__global__ void __launch_bounds__(64 * (KLOG2 == 6 ? kMostWaves : 5)) k_layer_token(TokenArgs a) {
    using L = Layout<KLOG2>;
    constexpr int NC = L::NC, MT = L::MT, NREG = L::NREG;
    __shared__ __align__(1024) unsigned char tsm[KS * MT * 1024];  // the token, then its codes
    __shared__ uint32_t red[32];                                   // the waves' upper ends, then their lower ends
    __shared__ int part[kMostWaves][4][4];
    const int tid = threadIdx.x, nthreads = blockDim.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthreads >> 6;
    const int l15 = lane & 15, g = lane >> 4;
    const int kb = a.d_e >> 1;

    // ---- the token into LDS: chunk p holds the 8 inputs (row, column .. column + 7) of chunk_of's layout
    const uint32_t lds0 = (uint32_t)(uintptr_t)(PME_AS3 unsigned char*)tsm;
    for (int base = wave * 64; base < 64 * KS * MT; base += nthreads) {
        const int p = base + lane, blk = p >> 3, r = p & 7;
        const int at = (4 * (blk / MT) + (r >> 1)) * NC + 16 * (blk % MT) + 8 * (r & 1);
        if (at < a.d) dma16(a.x, 2u * (uint32_t)at, __builtin_amdgcn_readfirstlane(lds0 + base * 16));
        else *reinterpret_cast<u32x4*>(tsm + p * 16) = u32x4{0u, 0u, 0u, 0u};
    }
    // ---- this wave's block fragments and what the epilogue needs, then its weights, which stay in flight during the rotation
    bf16x8 bfrag[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) bfrag[ks] = __builtin_bit_cast(bf16x8, a.ptable[(wave * a.stride + ks) * 64 + lane]);
    const int n0 = blockIdx.x * 16, nchunks = kb >> 6;
    float esw = 0.f;
    int ews = 0;
    if (tid < 16) {
        esw = a.sw[min(n0 + tid, a.N - 1)];
        if (ASYM) ews = a.wsum[min(n0 + tid, a.N - 1)];
    }
    const int c0 = wave * nchunks / nwaves, c1 = (wave + 1) * nchunks / nwaves;        // at most KB
    const uint8_t* wrow = a.qw + (int64_t)min(n0 + l15, a.N - 1) * kb + g * 16;
    u32x4 w[KB];
#pragma unroll
    for (int i = 0; i < KB; ++i)       // beyond the share: chunks that other waves use, so that every wave has KB loads on the way
        w[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wrow + (int64_t)min(c0 + i, nchunks - 1) * 64));
    if (tid < 32) red[tid] = 0;        // the places of waves that do not exist stay so
    wait_vm<KB>();                     // everything but the newest KB loads: the token has landed
    lds_barrier();

    // ---- rotate
    float v[NREG];
    {
        f32x4 acc[MT];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const unsigned char* p0 = tsm + ((8 * ks + 2 * g) * MT + mt) * 128 + 8 * l15;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 PME_AS3*)p0);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 PME_AS3*)(p0 + MT * 128));
                typedef __attribute__((ext_vector_type(8))) short s16x8;
                const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, both), bfrag[ks],
                                                                  ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[mt], 0, 0, 0);
            }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[mt * 4 + r] = acc[mt][r];
    }
    fwht_lane<KLOG2>(v);
    float hi = 0.f, lo = 0.f;
    if constexpr (ASYM) {
#pragma unroll
        for (int i = 0; i < NREG; i += 2) {
            hi = __builtin_fmaxf(__builtin_fmaxf(hi, v[i]), v[i + 1]);
            lo = __builtin_fminf(__builtin_fminf(lo, v[i]), v[i + 1]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NREG; i += 2) hi = __builtin_fmaxf(__builtin_fmaxf(hi, __builtin_fabsf(v[i])), __builtin_fabsf(v[i + 1]));
    }
    uint32_t ends = half_max(pair_max(magnitude(hi), magnitude(ASYM ? lo : hi)));
    if ((lane & 31) == 0) red[(lane >> 5) * 16 + wave] = ends;
    lds_barrier();                     // every wave has read the token and written its range
    ends = row_max(red[(lane >> 5) * 16 + l15]);
    if constexpr (ASYM) {
        uint32_t lower = ends;
        swap32(ends, lower);
        lo = -__uint_as_float(lower);
    }
    hi = __uint_as_float(ends);
    const TokenScale q = ASYM ? asymmetric_scale(hi, lo, a.g) : symmetric_scale(hi, a.g);
    const int ap = wave * 16 + l15;
    if (ap < a.b) {
        // the codes take the place of the inputs; a lane's run starts at column RUN g
        uint32_t* o = reinterpret_cast<uint32_t*>(tsm + ((ap * NC + L::RUN * g) >> 1));
#pragma unroll
        for (int wd = 0; wd < L::RUN / 8; ++wd) {
            auto value = [&](int nb) { return v[L::reg_of_run_pos(wd * 8 + nb)]; };
            o[wd] = ASYM ? asymmetric_codes(q.rinv, 12582912.f + (float)q.z, value) : symmetric_codes(q.rinv, value);
        }
    }
    lds_barrier();

    // ---- the waves' shares of K: 16 channels x the token (in every one of the operand's 16 rows)
    i32x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < KB; ++i) {
        if (c0 + i < c1) {             // scalar operands, hence a branch: matrix instructions ignore the execution mask
            u32x4 xv = *reinterpret_cast<const u32x4*>(tsm + (c0 + i) * 64 + g * 16);
            if (ASYM) xv ^= 0x88888888u;           // unsigned code u: u ^ 8 as a signed nibble is u - 8
            i32x4 wlo, whi, xlo, xhi;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                wlo[e] = (int)((w[i][e] & 0x0F0F0F0Fu) << 4);
                whi[e] = (int)(w[i][e] & 0xF0F0F0F0u);
                xlo[e] = (int)((xv[e] & 0x0F0F0F0Fu) << 4);
                xhi[e] = (int)(xv[e] & 0xF0F0F0F0u);
            }
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(wlo, xlo, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(whi, xhi, acc, 0, 0, 0);
        }
    }
    // element i of lane 16 g: channel 4 g + i
    if (l15 == 0) *reinterpret_cast<i32x4*>(part[wave][g]) = acc;
    lds_barrier();
    if (tid < 16 && n0 + tid < a.N) {
        int s = 0;
#pragma unroll
        for (int w2 = 0; w2 < kMostWaves; ++w2)
            if (w2 < nwaves) s += part[w2][tid >> 2][tid & 3];
        s >>= 8;                       // exact: the low 8 bits are zero
        if (ASYM) s -= (q.z - 8) * ews;
        a.y[n0 + tid] = f32_to_bf16_bits((float)s * q.s * esw);
    }
}

template <int KLOG2, int KS, int KB> pme_status launch_token(const TokenArgs& a, int nwaves, hipStream_t stream) {
    const dim3 grid((unsigned)((a.N + 15) / 16)), block(64 * nwaves);
    if (a.wsum) hipLaunchKernelGGL((k_layer_token<KLOG2, KS, true, KB>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((k_layer_token<KLOG2, KS, false, KB>), grid, block, 0, stream, a);
    return hip_status(hipGetLastError());
}

}  // namespace

pme_status launch_layer_token(const RotateArgs& ra, const GemmArgs& ga) {
    // up to 4096 channels: one workgroup per compute unit, each of which rotates the token again
    if (ra.T != 1 || ga.N > 4096 || ra.xt != PME_BF16) return PME_ERR_UNSUPPORTED_PATH;
    // the rotation's and the GEMM's own conditions on alignment and K
    if ((ra.d & 7) || (reinterpret_cast<uintptr_t>(ra.x) & 15) || (reinterpret_cast<uintptr_t>(ga.qw) & 15)) return PME_ERR_UNSUPPORTED_PATH;
    if (ra.d_e % 128 || ra.d_e >= (1 << 17)) return PME_ERR_UNSUPPORTED_PATH;
    RotateArgs f = ra;
    fold_stages(f);
    if (f.k != 6 && f.k != 7) return PME_ERR_UNSUPPORTED_PATH;
    const int nc = 1 << f.k, rows = (int)((f.d + nc - 1) >> f.k), ks = (rows + 31) / 32, nt = (f.b + 15) / 16;
    const int share = (int)((ra.d_e / 128 + nt - 1) / nt);
    if (nt > (f.k == 6 ? kMostWaves : 5) || share > (f.k == 6 ? 8 : 16)) return PME_ERR_UNSUPPORTED_PATH;
    // the blocks of 132 .. 152 by 64 columns and of 65 .. 80 by 128, of 8192 inputs or nearly so: 16 KB, which also hold the codes
    if (ks != (f.k == 6 ? 4 : 2) || f.b <= 64) return PME_ERR_UNSUPPORTED_PATH;
    pme_status st = PME_OK;
    int stride = 0;
    const void* table = rotate_table(f, rows, &stride, &st);
    // without a table (a shape that is captured cold, a full pool) the two kernels answer: some rows, such as those of a pitch that
    // the matrix-core rotation does not take, go through the plain one, which needs no table
    if (!table) return PME_ERR_UNSUPPORTED_PATH;
    const double gamma = 1.0 / sqrt((double)ra.d_e);
    const TokenArgs a{static_cast<const uint16_t*>(ra.x), (int)ra.d, (int)ra.d_e, f.b, static_cast<const u32x4*>(table), stride,
                      (float)(gamma / (ga.zx ? 15.0 : 7.0)), ga.qw, ga.sw, ga.wsum, (int)ga.N, static_cast<uint16_t*>(ga.y)};
    return f.k == 6 ? launch_token<6, 4, 8>(a, nt, ra.stream) : launch_token<7, 2, 16>(a, nt, ra.stream);
}

}  // namespace pme
