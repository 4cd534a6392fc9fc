// MXFP4 GEMM for outputs that give a compute unit one small tile: the waves of a workgroup split K, as in gemm_kslice.hip.
//
//   y[t][n] = bf16( sum over blocks of 32 of 2^(ex - 127) 2^(ew - 127) sum_i P_x,i P_w,i )   (paper Section 4, OCP MXFP4).
//
// A workgroup owns an output tile of 32 FM x 32 FN (or of 8 or 16 tokens).  Each of its NW waves takes a contiguous NW-th of K
// and computes the whole tile over it, from an LDS ring of its own that it fills by DMA itself: no barrier in the K loop.  The
// fp32 partial tiles are added through LDS in the order of K, four 32 x 32 blocks at a time.
// What bounds it is the way from L2 into LDS: a compute unit takes at most one line of 128 bytes every two cycles, and a
// request for a part of a line costs as much as one for all of it.  Hence K steps of whole lines (128 bytes a row, 256 codes;
// layer 333 x 2048 x 9728 21.1 us with 64-byte rows, 18.8 with 128), and the scale bytes of 512 codes at a time, sixteen a row
// (25.5 us with the four of every 128 codes).  Contiguous K: what a wave fetches next is in the line after, or in the same one.
// The layer on 64 x 64 tiles whose waves share the K loop, and on this kernel (us, three sets of operands in turn): 46 x 3904 x
// 22016 45.7 and 26.4, 78 x 704 x 15360 35.1 and 14.1, 265 x 604 x 8960 26.1 and 15.5, 333 x 2048 x 9728 24.6 and 18.7; and on the
// weight-streaming kernel: 10 x 4864 x 10240 22.5 and 11.5, 16 x 2048 x 8704 12.7 and 10.4.
#include "gemm_tile.h"

#include <algorithm>
#include <cstdio>
#include <string>

namespace pme {
namespace {

typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// As dma16, from an address of each lane's own.
__device__ __forceinline__ void dma16_lane(const void* src, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_base) : "memory");
}

constexpr int mx_kslice_scale_blocks(int ar, int bn) { return (ar + bn + 63) / 64; }      // DMA of 64 rows' scale bytes
constexpr int mx_kslice_ring(int ar, int bn, int rb, int nstage) { return nstage * (ar + bn) * rb + 2 * mx_kslice_scale_blocks(ar, bn) * 1024; }
constexpr int mx_kslice_lds(int ar, int bn, int nw, int rb, int nstage) {
    const int blocks = ((ar + 31) / 32) * (bn / 32);
    const int rings = nw * mx_kslice_ring(ar, bn, rb, nstage), parts = (blocks < 4 ? blocks : 4) * nw * 4096 + 8192;
    return rings > parts ? rings : parts;
}

struct MxSliceArgs {
    const uint8_t *qx, *ex, *qw, *ew;
    int T, N, kb, eb;
    uint16_t* y;
    int64_t ldo;
    int tiles_m, tiles_n, xcd_gm, vec_store;
};

template <int AR, int BN, int NW, int RB, int NSTAGE> __device__ __forceinline__ void mx_kslice_tile(const MxSliceArgs& args) {
    const uint8_t *__restrict__ qx = args.qx, *__restrict__ ex = args.ex, *__restrict__ qw = args.qw, *__restrict__ ew = args.ew;
    uint16_t* __restrict__ y = args.y;
    const int T = args.T, N = args.N, kb = args.kb, eb = args.eb, tiles_m = args.tiles_m, tiles_n = args.tiles_n, xcd_gm = args.xcd_gm, vec_store = args.vec_store;
    const int64_t ldo = args.ldo;
    constexpr int BM = (AR + 31) / 32 * 32, FM = BM / 32, FN = BN / 32, ROWS = AR + BN;
    static_assert((AR == 8 || AR == 16 || AR % 32 == 0) && BN % 32 == 0, "whole 32-row fragments, or one that repeats 8 or 16 rows");
    constexpr int CPR = RB / 16, RPB = 64 / CPR;  // 16-byte chunks per row and K step; rows per DMA instruction
    constexpr int CH = ROWS / RPB;                // code DMA instructions per stage
    constexpr int H = RB / 64;                    // units of 128 codes (two sub-steps of the matrix instruction) per K step
    static_assert(H == 1 || H == 2, "64- or 128-byte rows");
    constexpr int SCH = mx_kslice_scale_blocks(AR, BN);          // scale DMA instructions per group of four units
    constexpr int STAGE = ROWS * RB, SCALES = NSTAGE * STAGE, GROUP = SCH * 1024, RING = mx_kslice_ring(AR, BN, RB, NSTAGE);
    static_assert(NSTAGE <= (H == 1 ? 4 : 3), "a group of scales issued with unit 4 g must have landed before unit 4 g + 3");
    constexpr int NBLK = FM * FN, ROUNDS = (NBLK + 3) / 4;
    constexpr int BLOCK = 32 * 32 * 4;            // bytes of a partial block
    constexpr int SHARE = NW / 4, QN = 4 / SHARE; // waves that finish a block together; groups of 8 channels each takes
    constexpr int SLAB = 32 * 16 * QN;            // bytes of a wave's finished bf16 part
    static_assert(NW == 4 || NW == 8, "one or two waves per SIMD");
    constexpr int PART = (NBLK < 4 ? NBLK : 4) * NW * BLOCK;
    static_assert(PART + NW * SLAB <= mx_kslice_lds(AR, BN, NW, RB, NSTAGE), "the partial blocks go through the rings");
    static_assert((NSTAGE - 1) * CH + 2 * SCH <= 63, "the wait counts must fit vmcnt");

    extern __shared__ __align__(1024) unsigned char smem[];      // a ring per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    xcd_tile((int)blockIdx.x, tiles_m, tiles_n, xcd_gm, tm, tn);
    const int m0 = tm * AR, n0 = tn * BN;
    unsigned char* ring = smem + wave * RING;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(PME_AS3 unsigned char*)ring;
    const int KT = kb / RB;                                      // K steps in all
    const int first = __builtin_amdgcn_readfirstlane(wave * KT / NW);
    const int steps = __builtin_amdgcn_readfirstlane((wave + 1) * KT / NW) - first;       // this wave's, at least one

    // DMA of codes: block blk covers tile rows RPB blk .. RPB blk + RPB - 1; lane L fills chunk position L % CPR of row L / CPR,
    // which holds chunk (L % CPR) ^ swz(row) (the swizzle looks at row bits below RPB only)
    static_assert(RPB % (RB == 64 ? 16 : 8) == 0 && AR % RPB == 0, "whole blocks of either operand");
    uint32_t voff[CH];
    {
        const int lr = lane / CPR, kc = (lane % CPR) ^ swz<RB>(lr);
#pragma unroll
        for (int blk = 0; blk < CH; ++blk) {
            const int r = RPB * blk + lr;
            const int row = (r < AR) ? min(m0 + r, T - 1) : min(n0 + r - AR, N - 1);
            voff[blk] = (uint32_t)row * (uint32_t)kb + (uint32_t)(kc * 16);
        }
    }
    // of scale bytes: a lane moves the sixteen of one row and four units (lanes beyond the tile's rows repeat its last one)
    const uint8_t* srow[SCH];
#pragma unroll
    for (int q = 0; q < SCH; ++q) {
        const int r = min(64 * q + lane, ROWS - 1);
        srow[q] = (r < AR) ? ex + (int64_t)min(m0 + r, T - 1) * eb : ew + (int64_t)min(n0 + r - AR, N - 1) * eb;
    }
    // the i-th of this wave's steps (beyond the last one a later K step or the last of all, into a stage that nobody reads, so
    // that every step issues the same number of DMA instructions and the wait counts are constants)
    auto step_of = [&](int i) { return __builtin_amdgcn_readfirstlane(min(first + i, KT - 1)); };
    auto issue_codes = [&](int stage, int kt, int q) {
        dma16((q < AR / RPB ? qx : qw) + (int64_t)kt * RB, voff[q], __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + q * 1024));
    };
    // group g: this wave's units 4 g .. 4 g + 3; the last group of a row ends with the row (it has at least NW units)
    auto group_base = [&](int g) { return __builtin_amdgcn_readfirstlane(min(H * first + 4 * g, H * KT - 4)); };
    auto issue_scales = [&](int g, int q) {
        dma16_lane(srow[q] + 4 * group_base(g), __builtin_amdgcn_readfirstlane(lds0 + SCALES + (g & 1) * GROUP + q * 1024));
    };

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int frow = lane & 31, fk = lane >> 5;
    // sub-step s of a step reads chunk 2 s + fk, at position (fk ^ swz(r)) ^ 2 s; rows 32 i + frow share frow's swizzle
    // (a tile of 8 or 16 tokens repeats them over the fragment's rows: the surplus results are never stored)
    const int arow = AR < 32 ? frow & (AR - 1) : frow;
    const int offa = arow * RB + ((fk ^ swz<RB>(arow)) << 4), offb = (AR + frow) * RB + ((fk ^ swz<RB>(frow)) << 4);
    struct Frags { u32x4 a[2][FM], b[2][FN]; uint32_t sa[FM], sb[FN]; };      // a unit: 32 codes per lane and sub-step
    auto load_frags = [&](Frags& f, int stage, int u) {          // unit u, which lives in stage `stage`
        const int h = u % H;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const unsigned char *pa = ring + stage * STAGE + (offa ^ ((2 * h + s) << 5)), *pb = ring + stage * STAGE + (offb ^ ((2 * h + s) << 5));
#pragma unroll
            for (int i = 0; i < FM; ++i) f.a[s][i] = *reinterpret_cast<const u32x4*>(pa + 32 * i * RB);
#pragma unroll
            for (int j = 0; j < FN; ++j) f.b[s][j] = *reinterpret_cast<const u32x4*>(pb + 32 * j * RB);
        }
        const int g = u >> 2, at = min(H * first + u, H * KT - 1) - group_base(g);      // place of the unit in its group
        const unsigned char* ps = ring + SCALES + (g & 1) * GROUP + 4 * at;
#pragma unroll
        for (int i = 0; i < FM; ++i) f.sa[i] = *reinterpret_cast<const uint32_t*>(ps + 16 * arow + 512 * i);
#pragma unroll
        for (int j = 0; j < FN; ++j) f.sb[j] = *reinterpret_cast<const uint32_t*>(ps + 16 * (AR + frow) + 512 * j);
    };
    // the scale of block 2 s + fk is byte 2 s of the row's dword shifted by fk bytes; the matrix instruction selects it
    auto shift_scales = [&](Frags& f) {
#pragma unroll
        for (int i = 0; i < FM; ++i) f.sa[i] >>= 8 * fk;
#pragma unroll
        for (int j = 0; j < FN; ++j) f.sb[j] >>= 8 * fk;
    };
    constexpr int NMFMA = 2 * FM * FN;
    auto mfma_one = [&](const Frags& f, auto mc) {
        constexpr int M = decltype(mc)::value, S = M / (FM * FN), I = M % (FM * FN) / FN, J = M % FN;
        const i32x8 xa = {(int)f.a[S][I][0], (int)f.a[S][I][1], (int)f.a[S][I][2], (int)f.a[S][I][3], 0, 0, 0, 0};
        const i32x8 wb = {(int)f.b[S][J][0], (int)f.b[S][J][1], (int)f.b[S][J][2], (int)f.b[S][J][3], 0, 0, 0, 0};
        // formats 4 = FP4 E2M1 for both operands
        acc[I][J] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wb, xa, acc[I][J], 4, 4, 2 * S, (int)f.sb[J], 2 * S, (int)f.sa[I]);
    };

    // The refill of a stage is issued in H parts: the first with the last unit of the step it held, the second with the first
    // unit of the next step.
    constexpr int PARTA = H == 1 ? CH : (CH + 1) / 2;
#pragma unroll
    for (int q = 0; q < SCH; ++q) issue_scales(0, q);
#pragma unroll
    for (int st = 0; st < NSTAGE; ++st) {
        const int kt = step_of(st);
#pragma unroll
        for (int q = 0; q < (st == NSTAGE - 1 ? PARTA : CH); ++q) issue_codes(st, kt, q);
    }
    wait_vm<(NSTAGE - 2) * CH + PARTA>();
    Frags f[2];
    load_frags(f[0], 0, 0);
    int cur = 0;                        // stage of the step that the unit belongs to
    // Unit u, whose fragments are in registers: the next unit's are read while the matrix cores work on this one's, and the
    // DMA instructions of a refill go between the matrix instructions.  Every fourth unit also fetches the scales of the
    // group after its own: behind them come the codes of at least NSTAGE - 2 steps before their first reader waits, which
    // leaves no more than those in flight.
    auto region = [&](int u, auto hc, Frags& now, Frags& next) {
        constexpr int HU = decltype(hc)::value;             // u % H
        constexpr bool LAST = HU == H - 1;
        const int i = u / H, nxt = (cur == NSTAGE - 1) ? 0 : cur + 1, prv = (cur == 0) ? NSTAGE - 1 : cur - 1;
        if constexpr (LAST) {
            // the next step has landed, and every read of this one has left the stage that is refilled now
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NSTAGE - 2) * CH) : "memory");
            load_frags(next, nxt, u + 1);
        } else {
            load_frags(next, cur, u + 1);
        }
        shift_scales(now);
        if ((u & 3) == 0) {
#pragma unroll
            for (int q = 0; q < SCH; ++q) issue_scales((u >> 2) + 1, q);
        }
        const int kt = step_of(LAST ? i + NSTAGE : i + NSTAGE - 1), dst = LAST ? cur : prv;
        constexpr int Q0 = LAST ? 0 : PARTA, NQ = LAST ? PARTA : CH - PARTA;
        constexpr int NP = NMFMA < NQ ? NMFMA : NQ;
        static_for<NP>([&](auto pc) {
            constexpr int P = decltype(pc)::value;
            static_for<NMFMA>([&](auto mc) {
                if constexpr (decltype(mc)::value * NP / NMFMA == P) mfma_one(now, mc);
            });
            __builtin_amdgcn_sched_barrier(0);
            static_for<NQ>([&](auto qc) {
                if constexpr (decltype(qc)::value * NP / NQ == P) issue_codes(dst, kt, Q0 + decltype(qc)::value);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (LAST) cur = nxt;
    };
    const int units = steps * H;
    int u = 0;
    for (; u + 2 < units; u += 2) {
        region(u, std::integral_constant<int, 0>{}, f[0], f[1]);
        region(u + 1, std::integral_constant<int, 1 % H>{}, f[1], f[0]);
    }
    if (H == 2 || u + 1 < units) {      // two units left (wave-uniform)
        region(u, std::integral_constant<int, 0>{}, f[0], f[1]);
        shift_scales(f[1]);
        static_for<NMFMA>([&](auto mc) { mfma_one(f[1], mc); });
    } else {
        shift_scales(f[0]);
        static_for<NMFMA>([&](auto mc) { mfma_one(f[0], mc); });
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");

    // ---- partial tiles: in rounds of four blocks every wave writes its partial blocks to LDS, then adds and finishes
    // block 4 round + wave / SHARE (with two waves per block, half of its channels each)
    unsigned char* slab = smem + PART + wave * SLAB;
    static_for<ROUNDS>([&](auto rc) {
        constexpr int R = decltype(rc)::value;
        lds_barrier();                  // the rings, or the previous round's blocks, have been read
        static_for<4>([&](auto bc) {
            constexpr int B = 4 * R + decltype(bc)::value;
            if constexpr (B < NBLK) {
                unsigned char* p = smem + (decltype(bc)::value * NW + wave) * BLOCK + lane * 16;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(p + q * 1024) = f32x4{acc[B / FN][B % FN][4 * q], acc[B / FN][B % FN][4 * q + 1],
                                                                    acc[B / FN][B % FN][4 * q + 2], acc[B / FN][B % FN][4 * q + 3]};
            }
        });
        lds_barrier();
        const int blk = 4 * R + wave / SHARE, q0 = (wave % SHARE) * QN;
        if (blk < NBLK) {               // wave-uniform
            const int tbase = m0 + 32 * (blk / FN), cbase = 32 * (blk % FN) + 8 * q0, nbase = n0 + cbase;
            constexpr int PITCH = 16 * QN;        // bytes of a slab row: 8 QN channels
            // element 4 q + e of the part: channel 8 q + 4 fk + e, token frow
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    sum += *reinterpret_cast<const f32x4*>(smem + ((wave / SHARE) * NW + w) * BLOCK + (q0 + q) * 1024 + lane * 16);
                *reinterpret_cast<u32x2*>(slab + frow * PITCH + (8 * q + 4 * fk) * 2) = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slab is this wave's own
            if (vec_store) {
#pragma unroll
                for (int c = lane; c < 32 * QN; c += 64) {
                    const int row = c / QN, col = (c % QN) * 8;
                    if ((AR >= 32 || row < AR) && tbase + row < T && nbase + col < N)
                        *reinterpret_cast<u32x4*>(y + (int64_t)(tbase + row) * ldo + nbase + col) =
                            *reinterpret_cast<const u32x4*>(slab + row * PITCH + col * 2);
                }
            } else {
                for (int c = lane; c < 32 * 8 * QN; c += 64) {
                    const int row = c / (8 * QN), col = c % (8 * QN);
                    if ((AR >= 32 || row < AR) && tbase + row < T && nbase + col < N)
                        y[(int64_t)(tbase + row) * ldo + nbase + col] = *reinterpret_cast<const uint16_t*>(slab + row * PITCH + col * 2);
                }
            }
        }
    });
}

template <int AR, int BN, int NW, int RB, int NSTAGE> __global__ void __launch_bounds__(64 * NW) k_mxgemm_kslice(MxSliceArgs a) {
    mx_kslice_tile<AR, BN, NW, RB, NSTAGE>(a);
}

template <int AR, int BN, int NW, int RB, int NSTAGE> pme_status launch_mx_kslice(const MxGemmArgs& a) {
    const int kb = (int)(a.d_e / 2), eb = (int)(a.d_e / 32);
    if (kb % RB || kb < RB * NW) return PME_ERR_UNSUPPORTED_PATH;      // whole K steps, at least one for each wave
    if ((int64_t)std::max(a.T, a.N) * kb >= (int64_t(1) << 32)) return PME_ERR_UNSUPPORTED_PATH;   // 32-bit DMA offsets
    if (a.dry) {
        if (a.plan) {
            static const std::string name = [] {
                char buf[64];
                snprintf(buf, sizeof buf, "k_mxgemm_kslice<%d, %d, %d, %d, %d>", AR, BN, NW, RB, NSTAGE);
                return std::string(buf);
            }();
            *a.plan = name.c_str();
        }
        return PME_OK;
    }
    const int tiles_m = (int)((a.T + AR - 1) / AR), tiles_n = (int)((a.N + BN - 1) / BN);
    constexpr int lds = mx_kslice_lds(AR, BN, NW, RB, NSTAGE);
    static_assert(lds <= 160 * 1024, "the rings fit in LDS");
    constexpr auto kern = k_mxgemm_kslice<AR, BN, NW, RB, NSTAGE>;
    static std::atomic<uint32_t> done;
    if (lds > 64 * 1024 && allow_dynamic_lds(kern, lds, done) != PME_OK) return PME_ERR_HIP;
    const int vec = (a.N % 8 == 0 && a.ldy % 8 == 0 && (reinterpret_cast<uintptr_t>(a.y) & 15) == 0) ? 1 : 0;
    const MxSliceArgs args{a.qx, a.ex, a.qw, a.ew, (int)a.T, (int)a.N, kb, eb, static_cast<uint16_t*>(a.y), a.ldy,
                           tiles_m, tiles_n, xcd_grid_m(tiles_m, tiles_n, AR, BN), vec};
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * NW), lds, a.stream, args);
    return hip_status(hipGetLastError());
}

}  // namespace

// The caller has checked that d_e % 128 == 0 and that code rows are 16-byte and scale rows 4-byte aligned.  Four waves: nothing
// is unpacked, so one wave per SIMD keeps up with its matrix instructions, and the rings reach three steps of whole lines; eight
// for up to eight tokens, whose rings are short enough (8 x 640 x 8448, layer: 10.6 us with four waves, 9.1 with eight).
pme_status launch_mxgemm_kslice(const MxGemmArgs& a, int tile) {
    switch (tile) {
        case 0: return launch_mx_kslice<8, 32, 8, 128, 3>(a);
        case 1: return launch_mx_kslice<16, 32, 4, 128, 3>(a);
        case 2: return launch_mx_kslice<32, 32, 4, 128, 3>(a);
        case 3: return launch_mx_kslice<64, 32, 4, 128, 2>(a);
        case 4: return launch_mx_kslice<64, 64, 4, 128, 2>(a);
        case 5: return launch_mx_kslice<32, 32, 4, 64, 4>(a);
    }
    return PME_ERR_UNSUPPORTED_PATH;
}

}  // namespace pme
