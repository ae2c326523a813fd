// Low-precision product for any k: BM x BN block of WM x WN waves.
// K advances in slabs of 128 bytes per row that go global -> LDS directly
// (global_load_lds_dwordx4: lane L of a wave writes 16 bytes at base + 16 L;
// measured on gfx950) through a ring of STAGES buffers, with no register staging
// and no LDS write instructions.  A slab is two steps of 64 bytes of k: bfloat16
// takes one 16 x 16 x 32 instruction per step and tile pair (chunk 4 step +
// lane / 16 of its row per lane), FP8 one 32 x 32 x 64 (chunks 4 step +
// 2 (lane / 32) and the next).
//
// Whole slabs, because rows of a ragged k start anywhere: 128 bytes of a row
// then lie on two lines, and loading them in halves asks for most lines twice
// (bfloat16 8431 x 8116 x 8824: 1600 us in halves, 1272 here; 1024 x 58368 x 4720
// 710 and 565, 68015 x 1008 x 752 224 and 181; k of whole lines 8832 1178 and 1019).
//
// LDS layout per slab and operand: row r occupies 128 bytes = 8 chunks of 16
// bytes; chunk kc of row r is stored at slot kc ^ ((r >> 1) & 7), so fragment
// reads are conflict-free.  The swizzle is applied on the global side: lane L of
// a load instruction fetches the chunk that belongs in slot L % 8 of row L / 8.
//
// Rows beyond M (columns beyond N) load a clamped valid row; they only feed
// results that are not stored.  K that is not a multiple of the slab: the last
// slab's chunks past K are loaded from a valid address and cleared in LDS by the
// lanes that loaded them, before the slab is handed to the other waves (TAIL;
// masking the fragments instead takes registers that a 256 x 256 tile does not
// have).  Every tile shape multiplies in the same order over k, so C does not
// depend on the tile.
#pragma once

#include <type_traits>

#include "gemm_lowp_kernel.h"
#include "gemm_mfma2_kernel.h"

namespace abft {

template <class Ops_, int BM_, int BN_, int WM_, int WN_, int MINB_, int STAGES_>
struct LowpRing {
    typedef Ops_ Ops;
    typedef typename Ops::E E;
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, STAGES = STAGES_, MINB = MINB_, GROUP_M = 8;
    static constexpr int NW = WM * WN, THREADS = 64 * NW;
    static constexpr int SLAB = 128;                       // bytes of k per row and slab
    static constexpr int BK = SLAB / (int)sizeof(E);       // k per slab
    static constexpr int VEC = 16 / (int)sizeof(E);        // elements per 16-byte chunk
    static constexpr int STAGE = (BM + BN) * SLAB;
    static constexpr int HDR = 256;                        // keeps every LDS base address non-zero
    static constexpr int LPA = BM / 8 / NW, LPB = BN / 8 / NW;     // load instructions (8 rows each) per wave
    static constexpr int MT = Ops::MT;                     // tile of one instruction
    static constexpr int TA = BM / WM / MT, TB = BN / WN / MT;     // instruction tiles per wave
    static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;     // 16 x 16 tiles per wave (epilogue layout)
    static constexpr int CPF = MT == 32 ? 2 : 1;           // chunks per fragment
    static_assert(LPA * 8 * NW == BM && LPB * 8 * NW == BN, "load split");
    static_assert(TA * MT * WM == BM && TB * MT * WN == BN, "wave tile");
};

template <class T, bool FUSED, bool TAIL>
__global__ __launch_bounds__(T::THREADS, T::MINB) void k_gemm_lowp(const typename T::E *__restrict__ A, int64_t lda,
                                                             const typename T::E *__restrict__ Bt, int64_t ldb,
                                                             float *__restrict__ C, int64_t ldc, int64_t M, int64_t N,
                                                             int64_t K, const int *__restrict__ scale_exp, EpiArgs epi) {
    typedef typename T::E E;
    typedef typename T::Ops Ops;
    constexpr int BM = T::BM, BN = T::BN, SLAB = T::SLAB, STAGE = T::STAGE, HDR = T::HDR, STAGES = T::STAGES;
    constexpr int LPA = T::LPA, LPB = T::LPB, LP = LPA + LPB, TA = T::TA, TB = T::TB, MT = T::MT, CPF = T::CPF;
    constexpr int TM = T::TM, TN = T::TN, VEC = T::VEC;
    __shared__ __attribute__((aligned(16))) uint8_t lds[HDR + STAGES * STAGE];

    const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int64_t tm, tn;
    tile_of<T::GROUP_M>(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    const int64_t row0 = tm * BM, col0 = tn * BN;

    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wm = wave / T::WN, wn = wave % T::WN;

    // chunk of the row that this lane loads with instruction inst of an operand (rows 8 inst + lane / 8)
    auto chunk_of = [&](int inst) { return (lane % 8) ^ (((inst * 8 + lane / 8) >> 1) & 7); };
    // global sources of this lane's A and B chunks per slab
    const E *srcA[LPA], *srcB[LPB];
#pragma unroll
    for (int q = 0; q < LPA; ++q) {
        const int64_t r = row0 + (wave * LPA + q) * 8 + lane / 8;
        srcA[q] = A + (r < M ? r : M - 1) * lda + chunk_of(wave * LPA + q) * VEC;
    }
#pragma unroll
    for (int q = 0; q < LPB; ++q) {
        const int64_t r = col0 + (wave * LPB + q) * 8 + lane / 8;
        srcB[q] = Bt + (r < N ? r : N - 1) * ldb + chunk_of(wave * LPB + q) * VEC;
    }
    const int64_t nk = (K + T::BK - 1) / T::BK;
    auto bufA = [&](int64_t slab) { return lds + HDR + (int)(slab % STAGES) * STAGE + wave * LPA * 1024; };
    auto bufB = [&](int64_t slab) { return lds + HDR + (int)(slab % STAGES) * STAGE + BM * SLAB + wave * LPB * 1024; };
    // A chunk at or past K, in the last slab of a K that is not a multiple of it, is fetched from the row's last
    // chunk: the lane's offset stops at kmax, which by the swizzle takes two values, for even and odd instructions
    // (a wave's first is even).
    static_assert(LPA % 2 == 0 && LPB % 2 == 0, "a wave's first load instruction is even");
    const int64_t kmax[2] = {K - VEC - chunk_of(0) * VEC, K - VEC - chunk_of(1) * VEC};
    auto issue = [&](int64_t slab) {
        uint8_t *a = bufA(slab), *b = bufB(slab);
        const int64_t k0 = slab * T::BK, k[2] = {TAIL ? min(k0, kmax[0]) : k0, TAIL ? min(k0, kmax[1]) : k0};
#pragma unroll
        for (int q = 0; q < LPA; ++q)
            __builtin_amdgcn_global_load_lds((const void *)(srcA[q] + k[q % 2]), (void *)(a + q * 1024), 16, 0, 0);
#pragma unroll
        for (int q = 0; q < LPB; ++q)
            __builtin_amdgcn_global_load_lds((const void *)(srcB[q] + k[q % 2]), (void *)(b + q * 1024), 16, 0, 0);
    };
    // Such chunks are cleared after this wave's loads of the slab have landed (K is a multiple of VEC: a chunk is
    // wholly inside or wholly past it).
    auto clear_tail = [&] {
        asm volatile("" ::: "memory");
        const int64_t left = K - (nk - 1) * T::BK;
        uint8_t *a = bufA(nk - 1) + lane * 16, *b = bufB(nk - 1) + lane * 16;
#pragma unroll
        for (int q = 0; q < LPA; ++q)
            if (chunk_of(wave * LPA + q) * VEC >= left) *(v4u *)(a + q * 1024) = v4u{};
#pragma unroll
        for (int q = 0; q < LPB; ++q)
            if (chunk_of(wave * LPB + q) * VEC >= left) *(v4u *)(b + q * 1024) = v4u{};
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0)
    };

    // fragments: row of the wave tile and chunk(s) of the step
    typedef typename std::conditional<MT == 32, v16f, v4f>::type vacc;
    struct frag { v4u c[CPF]; };
    vacc acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = vacc{};
    const int lr = lane % MT, lq = lane / MT * CPF;        // first chunk within the step
    const int arow = wm * (BM / T::WM) + lr, brow = wn * (BN / T::WN) + lr;
    auto frag_at = [&](const uint8_t *S, int r, int step) {
        frag f;
#pragma unroll
        for (int q = 0; q < CPF; ++q) f.c[q] = *(const v4u *)(S + r * SLAB + (((4 * step + lq + q) ^ ((r >> 1) & 7)) << 4));
        return f;
    };
    auto read = [&](int64_t slab, int step, frag (&fa)[TA], frag (&fb)[TB]) {
        const uint8_t *As = lds + HDR + (int)(slab % STAGES) * STAGE, *Bs = As + BM * SLAB;
#pragma unroll
        for (int a = 0; a < TA; ++a) fa[a] = frag_at(As, arow + MT * a, step);
#pragma unroll
        for (int b = 0; b < TB; ++b) fb[b] = frag_at(Bs, brow + MT * b, step);
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
    // scheduling groups (masks: 0x008 MFMA, 0x020 global load, 0x100 LDS read): n loads or reads spread over m MFMAs
    constexpr int NMF = TA * TB, NRD = (TA + TB) * CPF;
    auto spread = [](auto mask, auto over) {
        constexpr int MASK = decltype(mask)::value, n = MASK == 0x020 ? LP : NRD, m = decltype(over)::value;
        constexpr int per = n > m ? (n + m - 1) / m : 1, mf = n > m ? 1 : m / n;
#pragma unroll
        for (int i = 0; i < (n + per - 1) / per; ++i) {
            __builtin_amdgcn_sched_group_barrier(MASK, per, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, mf, 0);
        }
    };
    const std::integral_constant<int, 0x100> reads;
    const std::integral_constant<int, 0x020> loads;
    const std::integral_constant<int, (NMF > 1 ? NMF / 2 : 1)> half;
    const std::integral_constant<int, (NMF > 3 ? NMF / 4 : 1)> quarter;

    // Software pipeline: the fragments of a step are read while the step
    // before it is multiplied, and the slab's one barrier stands between its
    // two steps, when every wave holds the rest of the slab in registers (its
    // buffer then takes slab kt + STAGES) and slab kt + 1 has landed.
    frag fa0[TA], fb0[TB], fa1[TA], fb1[TB];
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < nk) issue(s);
    if (nk >= STAGES) wait_vm<(STAGES - 1) * LP>();
    else wait_vm<0>();
    if (TAIL && nk == 1) clear_tail();
    bare_barrier();
    read(0, 0, fa0, fb0);
    int64_t kt = 0;
    for (; kt + STAGES < nk; ++kt) {
        read(kt, 1, fa1, fb1);
        mma(fa0, fb0);
        spread(reads, half);                               // ahead of the next step's first MFMA, which needs them
        __builtin_amdgcn_sched_barrier(0);
        wait_vm_lds<(STAGES - 2) * LP>();
        bare_barrier();
        issue(kt + STAGES);
        read(kt + 1, 0, fa0, fb0);
        mma(fa1, fb1);
        spread(loads, half);
        spread(reads, quarter);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (; kt + 1 < nk; ++kt) {                            // no more loads
        read(kt, 1, fa1, fb1);
        mma(fa0, fb0);
        wait_vm_lds<0>();
        if (TAIL && kt + 2 == nk) clear_tail();
        bare_barrier();
        read(kt + 1, 0, fa0, fb0);
        mma(fa1, fb1);
    }
    read(kt, 1, fa1, fb1);                                 // the last slab
    mma(fa0, fb0);
    mma(fa1, fb1);
    __syncthreads();                                       // LDS is reused below and by the epilogue

    // accumulators in the 16 x 16 layout of the epilogue
    v4f c16[TM][TN];
    if constexpr (MT == 32) {
        // 32 x 32 -> 16 x 16 layout, one 32 x 32 tile at a time through a
        // wave-private column-major 32 x 36 float block placed after the
        // epilogue's partial-sum area: lane l writes its column l % 32, rows
        // 8 j + 4 (l / 32) + 0..3, then reads column 16 sb + l % 16, rows
        // 16 sa + 4 (l / 16) + 0..3 of quarter (sa, sb).
        constexpr int TLD = 36, SUMS = (T::WM * BN + T::WN * BM) * 8;
        static_assert(SUMS + T::NW * 32 * TLD * 4 <= STAGES * STAGE, "conversion block inside LDS");
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
