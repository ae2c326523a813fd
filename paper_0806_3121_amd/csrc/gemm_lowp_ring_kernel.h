// Low-precision product for any k: BM x BN block of WM x WN waves.
// K advances in halves of a 128-byte slab, 64 bytes of k per row, that go
// global -> LDS directly (global_load_lds_dwordx4: lane L of a wave writes 16
// bytes at base + 16 L; measured on gfx950) through a ring of RING buffers, with
// no register staging and no LDS write instructions.  bfloat16 takes one
// 16 x 16 x 32 instruction per half and tile pair (chunk lane / 16 of its row per
// lane), FP8 one 32 x 32 x 64 (chunks 2 (lane / 32) and the next).
//
// LDS layout per half and operand: row r occupies 64 bytes = 4 chunks of 16
// bytes; chunk kc of row r is stored at slot kc ^ ((r >> 2) & 3).  The 16 lanes
// of a quarter-wave read chunk kc of 16 consecutive rows: (r & 3, slot) then
// covers all 16 four-bank groups, so fragment reads are conflict-free.  The
// swizzle is applied on the global side: lane L of a load instruction fetches
// the chunk that belongs in slot L % 4 of row L / 4.
//
// Rows beyond M (columns beyond N) load a clamped valid row; they only feed
// results that are not stored.  K that is not a multiple of the half: the last
// half's chunks past K are loaded from a valid address and the fragments made
// of them are zeroed on both sides (TAIL).  Every tile shape multiplies in the
// same order over k, so C does not depend on the tile.
#pragma once

#include <type_traits>

#include "gemm_lowp_kernel.h"
#include "gemm_mfma2_kernel.h"

namespace abft {

template <class Ops_, int BM_, int BN_, int WM_, int WN_, int MINB_, int RING_ = 4>
struct LowpRing {
    typedef Ops_ Ops;
    typedef typename Ops::E E;
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, RING = RING_, MINB = MINB_, GROUP_M = 8;
    static constexpr int NW = WM * WN, THREADS = 64 * NW;
    static constexpr int HALF = 64;                        // bytes of k per row and half slab
    static constexpr int BK = HALF / (int)sizeof(E);       // k per half
    static constexpr int VEC = 16 / (int)sizeof(E);        // elements per 16-byte chunk
    static constexpr int STAGE = (BM + BN) * HALF;
    static constexpr int HDR = 256;                        // keeps every LDS base address non-zero
    static constexpr int LPA = BM / 16 / NW, LPB = BN / 16 / NW;   // load instructions (16 rows each) per wave
    static constexpr int MT = Ops::MT;                     // tile of one instruction
    static constexpr int TA = BM / WM / MT, TB = BN / WN / MT;     // instruction tiles per wave
    static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;     // 16 x 16 tiles per wave (epilogue layout)
    static constexpr int CPF = MT == 32 ? 2 : 1;           // chunks per fragment
    static_assert(LPA * 16 * NW == BM && LPB * 16 * NW == BN, "load split");
    static_assert(TA * MT * WM == BM && TB * MT * WN == BN, "wave tile");
};

template <class T, bool FUSED, bool TAIL>
__global__ __launch_bounds__(T::THREADS, T::MINB) void k_gemm_lowp(const typename T::E *__restrict__ A, int64_t lda,
                                                             const typename T::E *__restrict__ Bt, int64_t ldb,
                                                             float *__restrict__ C, int64_t ldc, int64_t M, int64_t N,
                                                             int64_t K, const int *__restrict__ scale_exp, EpiArgs epi) {
    typedef typename T::E E;
    typedef typename T::Ops Ops;
    constexpr int BM = T::BM, BN = T::BN, HALF = T::HALF, STAGE = T::STAGE, HDR = T::HDR, RING = T::RING;
    constexpr int LPA = T::LPA, LPB = T::LPB, LP = LPA + LPB, TA = T::TA, TB = T::TB, MT = T::MT, CPF = T::CPF;
    constexpr int TM = T::TM, TN = T::TN, VEC = T::VEC;
    __shared__ __attribute__((aligned(16))) uint8_t lds[HDR + RING * STAGE];

    const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int64_t tm, tn;
    tile_of<T::GROUP_M>(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    const int64_t row0 = tm * BM, col0 = tn * BN;

    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wm = wave / T::WN, wn = wave % T::WN;

    // global sources of this lane's A and B chunks per half
    const E *srcA[LPA], *srcB[LPB];
#pragma unroll
    for (int q = 0; q < LPA; ++q) {
        const int r = (wave * LPA + q) * 16 + lane / 4;
        const int64_t ga = row0 + r < M ? row0 + r : M - 1;
        srcA[q] = A + ga * lda + ((lane % 4) ^ ((r >> 2) & 3)) * VEC;
    }
#pragma unroll
    for (int q = 0; q < LPB; ++q) {
        const int r = (wave * LPB + q) * 16 + lane / 4;
        const int64_t gb = col0 + r < N ? col0 + r : N - 1;
        srcB[q] = Bt + gb * ldb + ((lane % 4) ^ ((r >> 2) & 3)) * VEC;
    }
    const int64_t nh = (K + T::BK - 1) / T::BK;
    auto load = [&](int64_t half, int64_t k0) {
        uint8_t *a = lds + HDR + (int)(half % RING) * STAGE + wave * LPA * 1024;
        uint8_t *b = lds + HDR + (int)(half % RING) * STAGE + BM * HALF + wave * LPB * 1024;
#pragma unroll
        for (int q = 0; q < LPA; ++q)
            __builtin_amdgcn_global_load_lds((const void *)(srcA[q] + k0), (void *)(a + q * 1024), 16, 0, 0);
#pragma unroll
        for (int q = 0; q < LPB; ++q)
            __builtin_amdgcn_global_load_lds((const void *)(srcB[q] + k0), (void *)(b + q * 1024), 16, 0, 0);
    };
    auto issue = [&](int64_t half) { load(half, half * T::BK); };
    // the rows of one instruction share r >> 2 modulo 4 lane by lane, so a lane's chunk is the same in all
    auto issue_any = [&](int64_t half) {
        if (TAIL && half == nh - 1) load(half, min(half * T::BK, K - VEC - ((lane % 4) ^ ((lane >> 4) & 3)) * VEC));
        else issue(half);
    };

    // fragments: row of the wave tile and chunk(s) of the half
    typedef typename std::conditional<MT == 32, v16f, v4f>::type vacc;
    struct frag { v4u c[CPF]; };
    vacc acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = vacc{};
    const int lr = lane % MT, lq = lane / MT * CPF;        // first chunk
    const int arow = wm * (BM / T::WM) + lr, brow = wn * (BN / T::WN) + lr;
    auto frag_at = [&](const uint8_t *S, int r) {
        frag f;
#pragma unroll
        for (int q = 0; q < CPF; ++q) f.c[q] = *(const v4u *)(S + r * HALF + (((lq + q) ^ ((r >> 2) & 3)) << 4));
        return f;
    };
    auto read = [&](int64_t half, frag (&fa)[TA], frag (&fb)[TB]) {
        const uint8_t *As = lds + HDR + (int)(half % RING) * STAGE, *Bs = As + BM * HALF;
#pragma unroll
        for (int a = 0; a < TA; ++a) fa[a] = frag_at(As, arow + MT * a);
#pragma unroll
        for (int b = 0; b < TB; ++b) fb[b] = frag_at(Bs, brow + MT * b);
    };
    auto mma = [&](const frag (&fa)[TA], const frag (&fb)[TB]) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                if constexpr (MT == 32) {
                    typename Ops::v8i x, y;
                    __builtin_memcpy(&x, &fa[a], 32);
                    __builtin_memcpy(&y, &fb[b], 32);
                    Ops::mfma(x, y, acc[a][b]);
                } else {
                    Ops::mfma(fa[a].c[0], fb[b].c[0], acc[a][b]);
                }
            }
    };
    // K is a multiple of VEC: a chunk is wholly inside or wholly past it
    auto mask = [&](frag (&fa)[TA], frag (&fb)[TB]) {
#pragma unroll
        for (int q = 0; q < CPF; ++q)
            if ((nh - 1) * T::BK + (lq + q) * VEC >= K) {
#pragma unroll
                for (int a = 0; a < TA; ++a) fa[a].c[q] = v4u{};
#pragma unroll
                for (int b = 0; b < TB; ++b) fb[b].c[q] = v4u{};
            }
    };
    // scheduling groups (masks: 0x008 MFMA, 0x020 global load, 0x100 LDS read):
    // the half's loads, then its fragment reads, spread over the MFMAs
    auto spread = [&](auto loads) {
        constexpr int NMF = TA * TB, NRD = (TA + TB) * CPF;
        constexpr int PV = LP * 4 > NMF ? 2 : 1, PD = NRD * 2 > NMF ? 2 : 1;
        if constexpr (decltype(loads)::value) {
#pragma unroll
            for (int i = 0; i < (LP + PV - 1) / PV; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, PV, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < (NRD + PD - 1) / PD; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, PD, 0);
        }
    };

    // Software pipeline over the halves: while half h is multiplied its
    // successor's fragments are read and the loads of half h + RING are issued
    // into h's buffer, which every wave left before the last barrier; the wait
    // before the next barrier covers half h + 2 only.  Each half so has RING - 1
    // halves' multiplications to land.
    frag fa0[TA], fb0[TB], fa1[TA], fb1[TB];
#pragma unroll
    for (int s = 0; s < RING; ++s)
        if (s < nh) issue_any(s);
    if (nh >= RING) wait_vm<(RING - 2) * LP>();
    else wait_vm<0>();
    bare_barrier();
    read(0, fa0, fb0);
    wait_vm_lds<(RING - 2) * LP>();
    bare_barrier();
    auto steady = [&](int64_t h, frag (&fa)[TA], frag (&fb)[TB], frag (&ga)[TA], frag (&gb)[TB]) {
        issue(h + RING);
        read(h + 1, ga, gb);
        mma(fa, fb);
        spread(std::true_type{});
        __builtin_amdgcn_sched_barrier(0);
        wait_vm_lds<(RING - 2) * LP>();
        bare_barrier();
    };
    auto rest = [&](int64_t h, frag (&fa)[TA], frag (&fb)[TB], frag (&ga)[TA], frag (&gb)[TB]) {
        if (h + RING < nh) issue_any(h + RING);
        if (h + 1 < nh) read(h + 1, ga, gb);
        if (TAIL && h + 1 == nh) mask(fa, fb);
        mma(fa, fb);
        wait_vm_lds<0>();
        bare_barrier();
    };
    const int64_t plain = TAIL ? nh - 1 : nh;              // halves loaded without clamping
    int64_t h = 0;
    for (; h + 1 + RING < plain; h += 2) {
        steady(h, fa0, fb0, fa1, fb1);
        steady(h + 1, fa1, fb1, fa0, fb0);
    }
    for (; h < nh; h += 2) {
        rest(h, fa0, fb0, fa1, fb1);
        if (h + 1 < nh) rest(h + 1, fa1, fb1, fa0, fb0);
    }

    // accumulators in the 16 x 16 layout of the epilogue
    v4f c16[TM][TN];
    if constexpr (MT == 32) {
        // 32 x 32 -> 16 x 16 layout, one 32 x 32 tile at a time through a
        // wave-private column-major 32 x 36 float block placed after the
        // epilogue's partial-sum area: lane l writes its column l % 32, rows
        // 8 j + 4 (l / 32) + 0..3, then reads column 16 sb + l % 16, rows
        // 16 sa + 4 (l / 16) + 0..3 of quarter (sa, sb).
        constexpr int TLD = 36, SUMS = (T::WM * BN + T::WN * BM) * 8;
        static_assert(SUMS + T::NW * 32 * TLD * 4 <= RING * STAGE, "conversion block inside LDS");
        float *X = (float *)(lds + HDR + SUMS) + wave * (32 * TLD);
        const int lh = lane / 32;
        auto lds_order = [] {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);    // lgkmcnt(0)
            asm volatile("" ::: "memory");
        };
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *(v4f *)(X + lr * TLD + 8 * j + 4 * lh) =
                        v4f{acc[a][b][4 * j], acc[a][b][4 * j + 1], acc[a][b][4 * j + 2], acc[a][b][4 * j + 3]};
                lds_order();
#pragma unroll
                for (int sa = 0; sa < 2; ++sa)
#pragma unroll
                    for (int sb = 0; sb < 2; ++sb)
                        c16[2 * a + sa][2 * b + sb] =
                            *(const v4f *)(X + (16 * sb + lane % 16) * TLD + 16 * sa + 4 * (lane / 16));
                lds_order();
            }
    } else {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) c16[a][b] = acc[a][b];
    }

    // FP8: the result is scaled back by 2^-(eA + eB) with ldexp (exact unless it leaves binary32's range;
    // the factor itself may not be a binary32 number)
    const int sh = scale_exp ? -(scale_exp[0] + scale_exp[1]) : 0;
    // epilogue extras (uniform branches): the accumulator flip hook, then the
    // store with the fused partial sums
    auto rowof = [](int l, int v) { return 4 * (l / 16) + v; };
    const int64_t gr0 = row0 + wm * (BM / T::WM), gc0 = col0 + wn * (BN / T::WN);
    if (epi.fbit >= 0 && epi.fi >= row0 && epi.fi < row0 + BM && epi.fj >= col0 && epi.fj < col0 + BN)
        epi_flip(c16, epi, gr0, gc0, lane, rowof);
    if constexpr (FUSED) {
        epi_store_fused<TM, TN, T::WM, T::WN, BM, BN>(c16, epi, (double *)(lds + HDR), row0, col0, tm, tn, M, N, wm, wn,
                                                      lane, sh, C, ldc, false, rowof);
        return;
    }
    auto store = [&](auto inside) {
        const int64_t gc = gc0 + lane % 16;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t gr = gr0 + a * 16 + 4 * (lane / 16) + v;
                if (!inside.value && gr >= M) continue;
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    if (inside.value || gc + b * 16 < N) C[gr * ldc + gc + b * 16] = __builtin_ldexpf(c16[a][b][v], sh);
            }
    };
    if (row0 + BM <= M && col0 + BN <= N) store(std::true_type{});
    else store(std::false_type{});
}

template <class T>
inline int launch_gemm_lowp(const typename T::E *A, int64_t lda, const typename T::E *Bt, int64_t ldb, float *C,
                             int64_t ldc, int64_t M, int64_t N, int64_t K, const int *scale_exp, hipStream_t s,
                             EpiArgs *epi = nullptr) {
    const int64_t tiles = ((M + T::BM - 1) / T::BM) * ((N + T::BN - 1) / T::BN);
    if (tiles > INT32_MAX) return ABFT_E_ARG;
    EpiArgs e = epi ? *epi : epi_none();
    if (epi) {
        epi->tiles_m = (M + T::BM - 1) / T::BM;
        epi->tiles_n = (N + T::BN - 1) / T::BN;
    }
    auto run = [&](auto fused, auto tail) {
        // the fused partial sums' layout has no room for smaller tiles: such picks are not made
        if constexpr (!fused.value || (T::BM >= kMinTileEdge && T::BN >= kMinTileEdge)) {
            k_gemm_lowp<T, fused.value, tail.value><<<(unsigned)tiles, T::THREADS, 0, s>>>(A, lda, Bt, ldb, C, ldc, M, N,
                                                                                           K, scale_exp, e);
            return (int)ABFT_OK;
        } else {
            return (int)ABFT_E_UNSUPPORTED;
        }
    };
    const bool tail = K % T::BK != 0;
    if (e.pc) return tail ? run(std::true_type{}, std::true_type{}) : run(std::true_type{}, std::false_type{});
    return tail ? run(std::false_type{}, std::true_type{}) : run(std::false_type{}, std::false_type{});
}

}  // namespace abft
