// W4A4 GEMM for outputs that give a compute unit one small tile: the NW = 4 or 8 waves of a workgroup split K.
//
//   acc[t][n] = sum_j qx[t][j] qw[n][j],  y[t][n] = bf16(acc * sx[t] * sw[n])   (paper Sections 3 and 4).
//
// A workgroup owns a 32 FM x 32 FN output tile (or one of 8 or 16 tokens).  Wave w takes the K steps w, w + NW, w + 2 NW, ... and
// computes the whole tile over them, from an LDS ring of its own that it fills by DMA itself: there is no barrier in
// the K loop, and against waves that share the tile's quarters each fragment read and unpacked feeds twice the matrix
// instructions.  What bounds the tiled kernel at these sizes is that one wave per SIMD meets a workgroup barrier every
// 256 codes with little matrix work in between; here a wave only ever waits for its own DMA.  The partial tiles
// (exact integers) are added through LDS at the end, four 32 x 32 blocks at a time, one per wave (of eight waves, half of
// one), and each wave finishes what it added.
// What bounds this kernel is the way from L2 into LDS, which takes a line of 128 bytes at a time: a step of 128 codes asks for half
// lines and gets half the rate.  Where d_e is a multiple of 256 and LDS has room a step is 256 codes, whole lines.  Layers, half
// and whole lines, us (three sets of operands in turn): 32 x 4096 x 15360 16.7 and 14.1, 517 x 2048 x 8704 24.1 and 22.1, 1673 x 896 x
// 22016 71.4 and 67.0, 48 x 6144 x 8704 14.2 and 13.1, 463 x 640 x 18432 24.5 and 21.5, 333 x 2048 x 9728 18.1 and 17.3.  Few tokens,
// weight-streaming kernel and 8 or 16 x 32 of whole lines, GEMM alone, us from the caches / from memory: 8 x 1088 x 22016 12.6 / 12.7 and
// 8.9 / 11.7, 16 x 2048 x 10240 9.0 / 9.1 and 6.2 / 8.8; but 12 x 2048 x 8704 6.9 / 6.9 and 5.2 / 7.4, which streams (see kslice_cost).
// Consecutive steps of one wave instead of every NW-th: 2-5 % slower.
// Operands, unpacking (a nibble in the top of a byte is 16 x its value), fragment layout and epilogue as in gemm_mfma.hip.
#include "gemm_tile.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <string>

namespace pme {
namespace {

// MODE: what is written, and HALF_LINES for K steps of 128 codes (64 bytes a row) where d_e is no multiple of 256.
constexpr int HALF_LINES = 4;
// Whole lines: K steps of 256 codes, 128 bytes a row.  Not for 128 x 64 with three stages and 128 x 128, whose rings of whole
// lines do not fit in LDS.
constexpr bool kslice_lines(int ar, int bn, int nstage, int mode) {
    return !(mode & HALF_LINES) && !(ar == 128 && bn == 64 && nstage == 3) && !(ar == 128 && bn == 128);
}
// Stages in LDS.  Whole lines: of the NSTAGE steps one is in registers, of 64 x 32 two, the others in LDS.
constexpr int kslice_lds_stages(int ar, int bn, int nstage, int mode) {
    return !kslice_lines(ar, bn, nstage, mode) ? nstage : ar == 64 && bn == 32 ? nstage - 2 : nstage - 1;
}
// Bytes of a wave's ring.
constexpr int kslice_ring(int ar, int bn, int nstage, int mode) {
    return kslice_lds_stages(ar, bn, nstage, mode) * (ar + bn) * (kslice_lines(ar, bn, nstage, mode) ? 128 : 64);
}
// LDS: the rings, which also hold a round of partial blocks (four blocks of 4 KB of every wave), the finished parts (8 KB in
// all) and the tile's scales.
constexpr int kslice_lds(int ar, int bn, int nw, int nstage, int mode) {
    const int blocks = ((ar + 31) / 32) * (bn / 32);
    const int rings = nw * kslice_ring(ar, bn, nstage, mode), parts = (blocks < 4 ? blocks : 4) * nw * 4096 + 8192 + (ar + bn) * 8;
    return rings > parts ? rings : parts;
}

struct KSliceArgs {
    const uint8_t *qx, *qw;
    const float *sx, *sw;
    const int32_t *zx, *wsum;
    int T, N, kb;
    void* out;
    int64_t ldo;
    int tiles_m, tiles_n, xcd_gm, vec_store;
};

// NW: waves (slices of K), 4 or 8: one or two per SIMD.  AR: tokens of the tile, 8, 16 or a multiple of 32.
template <int AR, int BN, int NW, int NSTAGE, int MODE_> __device__ __forceinline__ void kslice_tile(const KSliceArgs& args) {
    constexpr int MODE = MODE_ & ~HALF_LINES;
    const uint8_t *__restrict__ qx = args.qx, *__restrict__ qw = args.qw;
    const float *__restrict__ sx = args.sx, *__restrict__ sw = args.sw;
    const int32_t *__restrict__ zx = args.zx, *__restrict__ wsum = args.wsum;
    void* __restrict__ out = args.out;
    const int T = args.T, N = args.N, kb = args.kb;
    const int64_t ldo = args.ldo;
    constexpr int BM = (AR + 31) / 32 * 32, FM = BM / 32, FN = BN / 32, ROWS = AR + BN;
    static_assert((AR == 8 || AR == 16 || AR % 32 == 0) && BN % 32 == 0, "whole 32-row fragments, or one that repeats 8 or 16 rows");
    constexpr bool LINES = kslice_lines(AR, BN, NSTAGE, MODE_);
    constexpr int RB = LINES ? 128 : 64;          // bytes per row and K step
    constexpr int LS = kslice_lds_stages(AR, BN, NSTAGE, MODE_);  // stages in LDS
    constexpr int CPR = RB / 16, RPB = 64 / CPR;  // 16-byte chunks per row and K step; rows per DMA instruction
    constexpr int CH = ROWS / RPB;                // DMA instructions per stage
    constexpr int STAGE = ROWS * RB, RING = LS * STAGE;
    constexpr int NBLK = FM * FN;                 // 32 x 32 blocks of the tile
    constexpr int ROUNDS = (NBLK + 3) / 4;
    constexpr int BLOCK = 32 * 32 * 4;            // bytes of a partial block
    constexpr int SHARE = NW / 4, QN = 4 / SHARE; // waves that finish a block together; groups of 8 channels each takes
    constexpr int SLAB = 32 * 16 * QN;            // bytes of a wave's finished bf16 part
    static_assert(NW == 4 || NW == 8, "one or two waves per SIMD");
    constexpr int PART = (NBLK < 4 ? NBLK : 4) * NW * BLOCK;      // a round's four blocks of every wave
    static_assert(RING == kslice_ring(AR, BN, NSTAGE, MODE_) && PART + NW * SLAB + ROWS * 8 <= kslice_lds(AR, BN, NW, NSTAGE, MODE_), "the partial blocks go through the rings");
    static_assert((LS - 1) * CH <= 63, "the wait counts must fit vmcnt");

    extern __shared__ __align__(1024) unsigned char smem[];      // a ring per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    xcd_tile((int)blockIdx.x, args.tiles_m, args.tiles_n, args.xcd_gm, tm, tn);
    const int m0 = tm * AR, n0 = tn * BN;
    unsigned char* ring = smem + wave * RING;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(PME_AS3 unsigned char*)ring;
    const int KT = kb / RB;                                      // K steps in all
    const int steps = __builtin_amdgcn_readfirstlane((KT - wave + NW - 1) / NW);       // this wave's, at least one: wave, wave + NW, ...

    // DMA: block blk covers tile rows RPB blk .. RPB blk + RPB - 1; lane L fills chunk position L % CPR of row L / CPR, which
    // holds chunk (L % CPR) ^ swz(row) (the swizzle looks at row bits below RPB only)
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
    // the i-th of this wave's steps (beyond the last one: the last K step again, into a stage that nobody reads, so that
    // every step issues the same number of DMA instructions and the wait counts are constants)
    auto step_offset = [&](int i) { return __builtin_amdgcn_readfirstlane(min(wave + NW * i, KT - 1) * RB); };
    auto issue_slot = [&](int stage, int koff, int blk) {
        dma16((blk < AR / RPB ? qx : qw) + koff, voff[blk], __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + blk * 1024));
    };
    // scales (with 1/256, which removes the 16 x 16 of the nibble trick) and the asymmetric terms: fetched now, parked in
    // LDS for the epilogue once the rings are free
    constexpr int NT = 64 * NW, PRE = (ROWS + NT - 1) / NT;
    float pre[PRE];
    int prez[PRE];
#pragma unroll
    for (int q = 0; q < PRE; ++q) {
        const int idx = tid + NT * q;
        pre[q] = 0.f;
        prez[q] = 0;
        if constexpr (MODE != MODE_I32) {
            if (idx < AR) pre[q] = sx[min(m0 + idx, T - 1)] * (MODE == MODE_ASYM ? 1.f : 1.f / 256.f);
            else if (idx < ROWS) pre[q] = sw[min(n0 + idx - AR, N - 1)];
        }
        if constexpr (MODE == MODE_ASYM) {
            if (idx < AR) prez[q] = zx[min(m0 + idx, T - 1)];
            else if (idx < ROWS) prez[q] = wsum[min(n0 + idx - AR, N - 1)];
        }
    }

    i32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

    const int frow = lane & 31, fk = lane >> 5;
    // sub-step s of a step reads chunk 2 s + fk, at position (fk ^ swz(r)) ^ 2 s; rows 32 i + frow share frow's swizzle
    // (a tile of 8 or 16 tokens repeats them over the fragment's rows: the surplus results are never stored)
    const int arow = AR < 32 ? frow & (AR - 1) : frow;
    const int offa = arow * RB + ((fk ^ swz<RB>(arow)) << 4), offb = (AR + frow) * RB + ((fk ^ swz<RB>(frow)) << 4);
    struct Frags { u32x4 a[FM], b[FN]; };
    struct Unpacked { i32x4 alo[FM], ahi[FM], blo[FN], bhi[FN]; };
    auto load_frags = [&](Frags& f, const unsigned char* stage, int s) {
        const unsigned char *pa = stage + (offa ^ (s << 5)), *pb = stage + (offb ^ (s << 5));
#pragma unroll
        for (int i = 0; i < FM; ++i) f.a[i] = *reinterpret_cast<const u32x4*>(pa + 32 * i * RB);
#pragma unroll
        for (int j = 0; j < FN; ++j) f.b[j] = *reinterpret_cast<const u32x4*>(pb + 32 * j * RB);
    };
    // part c of NPART of the fragments' dwords / of the matrix instructions
    constexpr int NITEM = 4 * (FM + FN), NMFMA = 2 * FM * FN;
    auto unpack_part = [&](const Frags& f, Unpacked& u, int c, int nparts) {
#pragma unroll
        for (int q = 0; q < NITEM; ++q) {
            if (q * nparts / NITEM != c) continue;
            const int fr = q >> 2, e = q & 3;
            if (fr < FM) {
                uint32_t w = f.a[fr][e];
                if (MODE == MODE_ASYM) w ^= 0x88888888u;
                u.alo[fr][e] = (int)((w & 0x0F0F0F0Fu) << 4);
                u.ahi[fr][e] = (int)(w & 0xF0F0F0F0u);
            } else {
                const uint32_t w = f.b[fr - FM][e];
                u.blo[fr - FM][e] = (int)((w & 0x0F0F0F0Fu) << 4);
                u.bhi[fr - FM][e] = (int)(w & 0xF0F0F0F0u);
            }
        }
    };
    auto mfma_part = [&](const Unpacked& u, int c, int nparts) {
#pragma unroll
        for (int m = 0; m < NMFMA; ++m) {
            if (m * nparts / NMFMA != c) continue;
            const int i = m / (2 * FN), j = (m >> 1) % FN;
            if ((m & 1) == 0) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(u.blo[j], u.alo[i], acc[i][j], 0, 0, 0);
            else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(u.bhi[j], u.ahi[i], acc[i][j], 0, 0, 0);
        }
    };
    constexpr int NVALU = (FM + FN) * 12 + (MODE == MODE_ASYM ? FM * 4 : 0);
    constexpr int VPM = (NVALU + NMFMA - 1) / NMFMA;
    if constexpr (LINES) {
        // A step of 256 codes goes from LDS into registers as a whole, so that its stage can be refilled before the first of its
        // matrix instructions: with one stage of whole lines in LDS as many bytes are on their way as with two of half lines.
        constexpr int NSUB = RB / 32;
        auto issue_step = [&](int stage, int koff, int q0, int q1) {
#pragma unroll
            for (int blk = 0; blk < CH; ++blk)
                if (blk >= q0 && blk < q1) issue_slot(stage, koff, blk);
        };
        struct Step { Frags sub[NSUB]; };
        auto load_step = [&](Step& f, int stage) {
#pragma unroll
            for (int s = 0; s < NSUB; ++s) load_frags(f.sub[s], ring + stage * STAGE, s);
        };
        Unpacked unp[2];
        // the matrix instructions of sub-step S, the unpacking of S + 1 and DMA slots [Q0, Q1) of a refill, in parts
        auto sub_step = [&](const Step& f, auto sc, int stage, int koff, auto q0, auto q1) {
            constexpr int S = decltype(sc)::value, Q0 = decltype(q0)::value, NQ = decltype(q1)::value - Q0;
            constexpr int NP = NQ > 0 ? (NQ < NMFMA ? NQ : NMFMA) : 1;
            static_for<NP>([&](auto pc) {
                constexpr int P = decltype(pc)::value;
                if constexpr (S + 1 < NSUB) unpack_part(f.sub[S + 1], unp[(S + 1) & 1], P, NP);
                mfma_part(unp[S & 1], P, NP);
                constexpr int MPP = (NMFMA + NP - 1) / NP;
#pragma unroll
                for (int m = 0; m < MPP; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                constexpr int A = Q0 + (NQ * P + NP - 1) / NP, B = Q0 + (NQ * (P + 1) + NP - 1) / NP;
                issue_step(stage, koff, A, B);
                __builtin_amdgcn_sched_barrier(0);
            });
        };
#pragma unroll
        for (int st = 0; st < LS; ++st) issue_step(st, step_offset(st), 0, CH);
        if constexpr (LS == NSTAGE - 1) {
            int cur = 0;
            for (int i = 0; i < steps; ++i) {
                wait_vm<(LS - 1) * CH>();               // this step has landed
                Step f;
                load_step(f, cur);
                const int koff = step_offset(i + LS);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // every read has left the stage
                unpack_part(f.sub[0], unp[0], 0, 1);
                static_for<NSUB>([&](auto sc) {
                    constexpr int S = decltype(sc)::value;
                    sub_step(f, sc, cur, koff, std::integral_constant<int, CH * S / NSUB>{}, std::integral_constant<int, CH * (S + 1) / NSUB>{});
                });
                cur = (cur == LS - 1) ? 0 : cur + 1;
            }
        } else {
            // two steps in registers: the next one is read under this one's first sub-step, and the stage refilled under the others
            static_assert(LS == 1 && NSTAGE == 3, "one stage in LDS, two in registers");
            Step f[2];
            wait_vm<0>();
            load_step(f[0], 0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_step(0, step_offset(1), 0, CH);
            auto step = [&](int i, const Step& now, Step& next) {
                const int koff = step_offset(i + 2);
                wait_vm<0>();                           // the next step has landed
                load_step(next, 0);
                unpack_part(now.sub[0], unp[0], 0, 1);
                using zero = std::integral_constant<int, 0>;
                sub_step(now, zero{}, 0, koff, zero{}, zero{});
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // every read has left the stage
                static_for<NSUB - 1>([&](auto sc) {
                    constexpr int S = decltype(sc)::value;
                    sub_step(now, std::integral_constant<int, S + 1>{}, 0, koff, std::integral_constant<int, CH * S / (NSUB - 1)>{},
                             std::integral_constant<int, CH * (S + 1) / (NSUB - 1)>{});
                });
            };
            int i = 0;
            for (; i + 1 < steps; i += 2) {
                step(i, f[0], f[1]);
                step(i + 1, f[1], f[0]);
            }
            if (i < steps) step(i, f[0], f[1]);         // wave-uniform
        }
        wait_vm<0>();
    } else {
        // A region: fragments of sub-step g + 2 are read, those of g + 1 unpacked, the matrix cores work on g; ND DMA
        // instructions (slots D0 ..) go between the matrix instructions, which keep the pipe busy meanwhile.
        auto region = [&](Frags& fill, const unsigned char* stage, int s, const Frags& next, Unpacked& unext, const Unpacked& now,
                          int dst, int koff, auto d0, auto nd) {
            constexpr int D0 = decltype(d0)::value, ND = decltype(nd)::value, NP = ND > 0 ? ND : 1;
            load_frags(fill, stage, s);
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                unpack_part(next, unext, c, NP);
                mfma_part(now, c, NP);
                if (c == 0) __builtin_amdgcn_sched_group_barrier(0x100, FM + FN, 0);
                constexpr int MPP = (NMFMA + NP - 1) / NP;
#pragma unroll
                for (int m = 0; m < MPP; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
                }
                if constexpr (ND > 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    issue_slot(dst, koff, D0 + c);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };

#pragma unroll
        for (int st = 0; st < LS; ++st) {
            const int koff = step_offset(st);
#pragma unroll
            for (int blk = 0; blk < CH; ++blk) issue_slot(st, koff, blk);
        }
        wait_vm<(LS - 1) * CH>();
        Frags raw[2];
        Unpacked unp[2];
        load_frags(raw[0], ring, 0);
        load_frags(raw[1], ring, 1);
        unpack_part(raw[0], unp[0], 0, 1);
        // With two stages the refill must be under way early in the step; with more it is spread over the whole step.
        constexpr int DMA0 = LS == 2 ? CH : CH / 2;
        auto k_step = [&](int i, int cs) {
            const int nxt = (cs == LS - 1) ? 0 : cs + 1;
            const unsigned char* snxt = ring + nxt * STAGE;
            const int koff = step_offset(i + LS);
            // the next step has landed, and every read of this one has left the stage that is refilled now
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((LS - 2) * CH) : "memory");
            region(raw[0], snxt, 0, raw[1], unp[1], unp[0], cs, koff, std::integral_constant<int, 0>{}, std::integral_constant<int, DMA0>{});
            region(raw[1], snxt, 1, raw[0], unp[0], unp[1], cs, koff, std::integral_constant<int, DMA0>{}, std::integral_constant<int, CH - DMA0>{});
        };
        int cur = 0;
        for (int i = 0; i + 1 < steps; ++i) {
            k_step(i, cur);
            cur = (cur == LS - 1) ? 0 : cur + 1;
        }
        // the last step: its first sub-step is unpacked, its second read
        unpack_part(raw[1], unp[1], 0, 1);
        mfma_part(unp[0], 0, 1);
        mfma_part(unp[1], 0, 1);
        wait_vm<0>();
    }

    // ---- partial tiles: in rounds of four blocks every wave writes its partial blocks to LDS, then adds and finishes
    // block 4 round + wave / SHARE (with two waves per block, half of its channels each)
    unsigned char* slab = smem + PART + wave * SLAB;
    float* sc = reinterpret_cast<float*>(smem + PART + NW * SLAB);       // [AR] token scales, [BN] channel scales
    int* zc = reinterpret_cast<int*>(sc + ROWS);
    static_for<ROUNDS>([&](auto rc) {
        constexpr int R = decltype(rc)::value;
        lds_barrier();                  // the rings, or the previous round's blocks, have been read
        static_for<4>([&](auto bc) {
            constexpr int B = 4 * R + decltype(bc)::value;
            if constexpr (B < NBLK) {
                unsigned char* p = smem + (decltype(bc)::value * NW + wave) * BLOCK + lane * 16;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<i32x4*>(p + q * 1024) = i32x4{acc[B / FN][B % FN][4 * q], acc[B / FN][B % FN][4 * q + 1],
                                                                    acc[B / FN][B % FN][4 * q + 2], acc[B / FN][B % FN][4 * q + 3]};
            }
        });
        if constexpr (R == 0 && MODE != MODE_I32) {
#pragma unroll
            for (int q = 0; q < PRE; ++q) {
                const int idx = tid + NT * q;
                if (idx < ROWS) {
                    sc[idx] = pre[q];
                    if constexpr (MODE == MODE_ASYM) zc[idx] = prez[q];
                }
            }
        }
        lds_barrier();
        const int blk = 4 * R + wave / SHARE, q0 = (wave % SHARE) * QN;
        if (blk < NBLK) {               // wave-uniform
            i32x4 sum[QN];
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                sum[q] = i32x4{0, 0, 0, 0};
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    sum[q] += *reinterpret_cast<const i32x4*>(smem + ((wave / SHARE) * NW + w) * BLOCK + (q0 + q) * 1024 + lane * 16);
            }
            const int bi = blk / FN, bj = blk % FN;
            const int tbase = m0 + 32 * bi, cbase = 32 * bj + 8 * q0, nbase = n0 + cbase;
            // element 4 q + e of the part: channel 8 q + 4 fk + e, token frow
            if constexpr (MODE == MODE_I32) {
#pragma unroll
                for (int q = 0; q < QN; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int n = nbase + 8 * q + 4 * fk + e;
                        if ((AR >= 32 || frow < AR) && tbase + frow < T && n < N) static_cast<int32_t*>(out)[(int64_t)(tbase + frow) * ldo + n] = sum[q][e] >> 8;
                    }
            } else {
                constexpr int PITCH = 16 * QN;        // bytes of a slab row: 8 QN channels
                const float sxs = sc[32 * bi + arow];
                const int zoff = MODE == MODE_ASYM ? zc[32 * bi + arow] - 8 : 0;
#pragma unroll
                for (int q = 0; q < QN; ++q) {
                    const int cn = AR + cbase + 8 * q + 4 * fk;
                    float f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        int a = sum[q][e];
                        if (MODE == MODE_ASYM) a = (a >> 8) - zoff * zc[cn + e];
                        f[e] = (float)a * sxs * sc[cn + e];
                    }
                    *reinterpret_cast<u32x2*>(slab + frow * PITCH + (8 * q + 4 * fk) * 2) = u32x2{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3])};
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slab is this wave's own
                uint16_t* y = static_cast<uint16_t*>(out);
                if (args.vec_store) {
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
        }
    });
}

template <int AR, int BN, int NW, int NSTAGE, int MODE> __global__ void __launch_bounds__(64 * NW) k_gemm_kslice(KSliceArgs a) {
    kslice_tile<AR, BN, NW, NSTAGE, MODE>(a);
}

template <int AR, int BN, int NW, int NSTAGE> const char* kslice_name(int mode) {
    auto make = [](int m) {
        char buf[64];
        snprintf(buf, sizeof buf, "k_gemm_kslice<%d, %d, %d, %d, %d>", AR, BN, NW, NSTAGE, m);
        return std::string(buf);
    };
    static const std::string names[7] = {make(MODE_BF16), make(MODE_ASYM), make(MODE_I32), "", make(HALF_LINES + MODE_BF16), make(HALF_LINES + MODE_ASYM),
                                         make(HALF_LINES + MODE_I32)};
    return names[mode].c_str();
}

template <int AR, int BN, int NW, int NSTAGE, int MODE> pme_status launch_kslice_mode(const GemmArgs& a) {
    const int kb = (int)(a.d_e / 2);
    constexpr int RB = kslice_lines(AR, BN, NSTAGE, MODE) ? 128 : 64;
    if (kb % RB || kb < RB * NW) return PME_ERR_UNSUPPORTED_PATH;      // whole K steps, at least one for each wave
    if ((int64_t)std::max(a.T, a.N) * kb >= (int64_t(1) << 32)) return PME_ERR_UNSUPPORTED_PATH;   // 32-bit DMA offsets
    if (a.dry) {
        if (a.plan) *a.plan = kslice_name<AR, BN, NW, NSTAGE>(MODE);
        return PME_OK;
    }
    const int tiles_m = (int)((a.T + AR - 1) / AR), tiles_n = (int)((a.N + BN - 1) / BN);
    constexpr int lds = kslice_lds(AR, BN, NW, NSTAGE, MODE);
    static_assert(lds <= 160 * 1024, "the rings fit in LDS");
    constexpr auto kern = k_gemm_kslice<AR, BN, NW, NSTAGE, MODE>;
    static std::atomic<uint32_t> done;
    if (lds > 64 * 1024 && allow_dynamic_lds(kern, lds, done) != PME_OK) return PME_ERR_HIP;
    const int vec = (a.N % 8 == 0 && a.ldy % 8 == 0 && (reinterpret_cast<uintptr_t>(a.y) & 15) == 0) ? 1 : 0;
    const KSliceArgs args{a.qx, a.qw, a.sx, a.sw, a.zx, a.wsum, (int)a.T, (int)a.N, kb, a.y, a.ldy,
                          tiles_m, tiles_n, xcd_grid_m(tiles_m, tiles_n, AR, BN), vec};
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * NW), lds, a.stream, args);
    return hip_status(hipGetLastError());
}
// ODD: the tile also takes d_e that is no multiple of 256 (nor of 256 NW at least), on half lines.
template <int AR, int BN, int NW, int NSTAGE, bool ODD> pme_status launch_kslice(const GemmArgs& a) {
    constexpr bool LINES = kslice_lines(AR, BN, NSTAGE, 0);
    if constexpr (LINES && ODD) {
        if (a.d_e % 256 || a.d_e < 256 * NW) {
            if (a.out_i32) return launch_kslice_mode<AR, BN, NW, NSTAGE, HALF_LINES + MODE_I32>(a);
            if (a.zx) return launch_kslice_mode<AR, BN, NW, NSTAGE, HALF_LINES + MODE_ASYM>(a);
            return launch_kslice_mode<AR, BN, NW, NSTAGE, HALF_LINES + MODE_BF16>(a);
        }
    }
    if (a.out_i32) return launch_kslice_mode<AR, BN, NW, NSTAGE, MODE_I32>(a);
    if (a.zx) return launch_kslice_mode<AR, BN, NW, NSTAGE, MODE_ASYM>(a);
    return launch_kslice_mode<AR, BN, NW, NSTAGE, MODE_BF16>(a);
}

}  // namespace

// The caller has checked that d_e % 128 == 0, that d_e is in the accumulator's range and that code rows are 16-byte aligned.
// Two waves per SIMD where their registers and rings allow (up to 64 x 64): one alone issues a vector instruction only
// every five cycles and could not unpack as fast as the matrix cores consume (64 x 64, layer 333 x 2048 x 9728: four
// waves 6 % slower than eight).  32 x 32 with two steps (one in LDS, one in registers) leaves room for two workgroups per
// compute unit; 64 x 32 keeps two steps in registers, since a second one does not fit in LDS (112 x 2560 x 15360: 16.7 us, 18.8 on
// half lines).  Measured and not kept: four waves at 32 x 32 and 64 x 32 (up to 7 % slower), four stages at 8 and 16 x 32.
pme_status launch_gemm_kslice(const GemmArgs& a, int tile) {
    switch (tile) {
        case 0: return launch_kslice<32, 32, 8, 2, true>(a);
        case 1: return launch_kslice<64, 32, 8, 3, true>(a);
        case 2: return launch_kslice<64, 64, 8, 2, true>(a);
        case 3: return launch_kslice<96, 64, 4, 3, true>(a);
        case 4: return launch_kslice<128, 64, 4, 3, true>(a);
        case 5: return launch_kslice<128, 128, 4, 2, true>(a);
        case 6: return launch_kslice<8, 32, 8, 3, false>(a);
        case 7: return launch_kslice<16, 32, 8, 3, false>(a);
    }
    return PME_ERR_UNSUPPORTED_PATH;
}

// ---- the choice among the K-split tiles, the weight-streaming kernel and the 64 x 64 tile with a loader wave, by estimated time.
// From d_e = 8192 on in whole steps of 256 codes: coefficients of tile_cost, fitted (least squares of the relative error) to 12 000
// outputs of 1 .. 8192 tokens, 64 .. 28672 channels and d_e up to 32768, each timed on every tile as the layer runs it: after the
// rotation that writes its codes, three sets of operands in turn.  Layer over the same with half lines and the earlier choice: 0.91 in the
// mean up to 64 tokens, 0.92 up to 256, 0.95 up to 1024; of 8273 outputs of the paper's expansions one is more than 3 % slower.
inline bool lines_range(int64_t d_e) { return d_e % 256 == 0 && d_e >= 8192 && d_e <= 32768; }
struct LinesCost { int bm, bn; double c[8]; };
const LinesCost kLinesCosts[kKsliceTiles] = {
    {32, 32, {2.804, 0.6993, 0.04158, 0.0208, 0.004255, 0.04177, 0.006524, 2.216}},
    {64, 32, {3.805, 1.542, 0.05949, 0.02261, 0.01627, 0.06261, 0, 2.778}},
    {64, 64, {3.995, 2.084, 0.08929, 0.04617, 0.05776, 0.08723, 0, 1.336}},
    {96, 64, {5.487, 3.129, 0.1273, 0.03226, 0.03437, 0.135, 0, 1.252}},
    {128, 64, {5.856, 2.992, 0.1608, 0.04045, 0.05443, 0.1536, 0, 1.006}},
    {128, 128, {8.979, 5.881, 0.2418, 0.07264, 0.1111, 0.2538, 0, 0.6033}},
    {8, 32, {2.925, 0.08114, 0.03037, 0.03603, 0.03821, 0.05732, 0, 6.128}},
    {16, 32, {3.02, 1.07, 0.03139, 0.03477, 0.04609, 0.05784, 0, 4.008}}};
const double kLinesLoader64[8] = {2.993, 0.03986, 0.1686, 0.005481, 0.07819, 0.06149, 0.005724, 1.068};

// Other d_e: estimated times in us of the three kernels for outputs of less than a chip of large tiles, K in steps of 128 codes.  Fitted
// to 4500 outputs of 1 .. 2048 tokens, 320 .. 28672 channels and d_e 1024 .. 32768, each timed with three weight matrices in
// turn (in the caches) and with 600 MB of them in turn (from memory); the estimate is of the geometric mean of the two, good
// to 4-10 % for the K-split tiles and 5 % for the others.  Weights that come from memory slow the K-split kernel most (64-byte
// rows, a ring of two or three steps: 16 x 2048 x 8704 takes 6.6 us warm and 9.5 cold, the streaming kernel 8.0 and 7.8).
// The fit is of half lines.  Where d_e is a multiple of 256 the tiles up to 96 x 64 run on whole lines here too, on the same choice: 0.97
// of the half lines' time from the caches and 0.89 from memory in the mean of 840 outputs of d_e 1024 .. 7936, three of them more than 3 %
// slower in the geometric mean (largest 5 %), and within 1-2 % of the fastest tile.

// K-split tile: one round of workgroups; the 32 x 32 one, of which two share a compute unit, also several.  A second round of
// the others pays prologue and sum again and loses to the tiled kernel (647 x 2834 x 9728: 33.5 us on two rounds of 64 x 64, 26.9
// there; 1616 x 1152 x 15360: 42.8 and 37.3).
double kslice_cost(int64_t T, int64_t N, int64_t d_e, int tile) {
    if (lines_range(d_e)) {
        const auto& k = kLinesCosts[tile];
        const int64_t tiles = ((T + k.bm - 1) / k.bm) * ((N + k.bn - 1) / k.bn);
        // 8 or 16 tokens fill one row of their tiles, and only up to 4096 channels: beyond, 32 x 32 is within 3 %.  Weights that come
        // from memory, as a decode step reads them, and not from the caches as in the fit, slow these tiles more than the streaming kernel,
        // which has all of them on the way at once.  Their time over its, from the caches / from memory (largest), GEMM alone, three sets
        // and 700 MB of weights in turn, geometric means of 1500 outputs of 400 .. 4096 channels; what streams, all that lost more than 5 %:
        //   1 token below d_e = 15000 0.90 / 1.09 (1.12), 2 .. 4 0.86 / 1.06 (1.11); 9 .. 12 below 10000 0.84 / 1.08 (1.16);
        // and what does not: up to 4 tokens from 15000 on 0.80 / 0.98 (1.06); 5 .. 8 below 15000 0.82 / 1.04 (1.07), from there on 0.74 / 0.95;
        // 9 .. 12 from 10000 on 0.72 / 0.97 (1.06); 13 .. 16 below 10000 0.78 / 1.04 (1.10), from there on 0.66 / 0.93.
        const int64_t least = T <= 4 ? 15000 : T <= 8 ? 11000 : T <= 12 ? 10000 : 0;
        if (tile >= 6 && (T > k.bm || N > 4096 || d_e < least)) return 1e30;
        // Two rounds of 32 x 32 up to 32 tokens; above, larger tiles are as fast and vary less (267 x 1731 x 15360: 11 % slower on two).
        if (tile < 6 && tiles > (tile == 0 && T <= 32 ? 512 : 256)) return 1e30;
        if (tile == 0 && T <= 16 && N <= 4096) return 1e30;
        return tile_cost(k.c, tiles, T, N, d_e);
    }
    if (tile > 5) return 1e30;
    static const struct { int bm, bn; double fixed, step, by_fill, by_rows; } t[6] = {
        {32, 32, 3.15, 0.0576, 0.0344, 0.0378}, {64, 32, 3.84, 0.0713, 0.0201, 0.0534}, {64, 64, 4.16, 0.1062, 0.0250, 0.0865},
        {96, 64, 5.16, 0.1512, 0.0330, 0.1135}, {128, 64, 5.72, 0.1720, 0.0441, 0.0957}, {128, 128, 9.13, 0.2447, 0.0759, 0.1588}};
    const auto& k = t[tile];
    const double steps = (double)(d_e / 128), rows = (double)((N + k.bn - 1) / k.bn) / 256.0;
    const double fill = (double)((T + k.bm - 1) / k.bm) * rows;
    // 4.3: the largest that was timed; below d_e = 2048 only the 32 x 32 tile gains, and only on a single round (768 x 1024 x 1024:
    // 6.5 us on three of them to a unit, 5.2 tiled)
    if (fill > (tile == 0 && d_e >= 2048 ? 4.3 : 1.0) || (tile > 0 && d_e < 2048)) return 1e30;
    if (tile == 0) {
        const double more = std::max(0.0, fill - 1.0), rounds = std::ceil(fill) - 1.0, tokens = (double)std::min<int64_t>(T, 32) / 32.0;
        return k.fixed + 0.64 * more + steps * (k.step + 0.0306 * rounds + k.by_fill * more + (k.by_rows + 0.0355 * tokens) * rows);
    }
    return k.fixed + steps * (k.step + k.by_fill * fill + k.by_rows * rows);
}

// The weight-streaming kernel: rounds of 4096 channels, one workgroup per compute unit.
double decode_cost(int64_t T, int64_t N, int64_t d_e) {
    if (lines_range(d_e)) {
        const double steps = (double)(d_e / 128), fill = (double)((N + 15) / 16) / 256.0, more = fill > 1.0 ? std::ceil(fill) - 1.0 : 0.0;
        return 2.095 + 0.0897 * more + steps * (0.04276 + 0.02245 * std::min(fill, 1.0) + 0.0309 * std::max(fill - 1.0, 0.0) + 0.02677 * more + 0.02455 * (double)T / 16.0);
    }
    const double steps = (double)(d_e / 128), rounds = (double)((N + 4095) / 4096);
    return 2.59 + steps * (rounds * (0.0386 + 0.0022 * (double)T) + 0.0179 * (double)N / 4096.0);
}

// 64 x 64 tiles with a loader wave, of which two and more share a compute unit.
double loader64_cost(int64_t T, int64_t N, int64_t d_e) {
    if (lines_range(d_e)) return tile_cost(kLinesLoader64, ((T + 63) / 64) * ((N + 63) / 64), T, N, d_e);
    const double steps = (double)(d_e / 128), fill = (double)(((T + 63) / 64) * ((N + 63) / 64)) / 256.0;
    const double rounds = std::ceil(fill) - 1.0;
    return 3.76 + 0.74 * rounds + steps * (0.1616 + 0.0250 * std::min(fill, 1.0) + 0.0882 * std::max(fill - 1.0, 0.0) + 0.0381 * rounds);
}

// The K-split tile that is estimated to beat `other` us by more than 4 %, or -1.  With half lines its time over that of the kernel
// it replaces, on 3900 fitted outputs of up to 6144 channels: from the caches 0.92 in the mean up to 16 tokens, 0.61 up to 64 and 0.72
// above, beyond 1.03 on 30 outputs; from memory 0.98, 0.82 and 0.79, beyond 1.03 on one output in ten (mostly 12 .. 32 tokens
// by less than 2048 channels, up to 1.28, where it gains 30 % from the caches).
int kslice_choice(int64_t T, int64_t N, int64_t d_e, double other, double* us_out) {
    if (!kslice_range(d_e)) return -1;
    double best = 0.96 * other;
    int tile = -1;
    for (int k = 0; k < kKsliceTiles; ++k) {
        const double us = kslice_cost(T, N, d_e, k);
        if (us < best) { best = us; tile = k; }
    }
    if (us_out) *us_out = best;
    return tile;
}

}  // namespace pme
