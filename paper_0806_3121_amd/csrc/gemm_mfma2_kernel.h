// binary64 / binary32 product kernel, direct-to-LDS variant (gfx950):
// BM x BN block of WM x WN waves, v_mfma_f64_16x16x4_f64 or
// v_mfma_f32_16x16x4_f32.  K advances in slabs of 128 bytes per row (16
// binary64 or 32 binary32 values) that go global -> LDS directly
// (global_load_lds_dwordx4: lane L of a wave writes the 16 bytes at
// base + 16 L), through a ring of STAGES buffers, with no register staging
// and no LDS write instructions.  MFMA-bound: the fragments of each half slab
// are read under the MFMAs of the half before, with the slab's one barrier
// between its halves (see the k loop).
//
// LDS layout per slab and operand: row r is 128 bytes = 8 chunks of 16
// bytes; chunk kc of row r is stored at slot kc ^ ((r >> 1) & 7), so the 16
// rows a quarter-wave reads at one chunk index fall on 16 distinct four-bank
// groups.  The swizzle is applied on the global side: the lane that writes
// slot s of row r fetches chunk s ^ ((r >> 1) & 7).
//
// Inside a 16-deep k group each lane holds four consecutive k of its row and
// feeds them to four MFMAs, as in gemm_mfma_kernel.h; A and B use the same k
// order, and every tile shape the same order over k, so C does not depend on
// the tile.  Rows beyond M (columns beyond N) load a clamped valid row and
// their results are not stored.  K that is not a multiple of the slab: the
// last slab's chunks past K are loaded from a valid address and the fragments
// made of them are zeroed on both sides (TAIL).
#pragma once

#include <type_traits>

#include "gemm_mfma_kernel.h"

namespace abft {

// s_waitcnt with vmcnt = N (N < 64) and no wait on the other counters.
template <int N> __device__ inline void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0F70);
}

// A barrier without the memory fence of __syncthreads, which would also wait
// for every load still in flight.
__device__ inline void bare_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// s_waitcnt with vmcnt = N and lgkmcnt = 0.
template <int N> __device__ inline void wait_vm_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0070);
}

template <typename E_, int STAGES_, int BM_ = 256, int BN_ = 128, int WM_ = 4, int WN_ = 2, int MINB_ = 1>
struct Mfma2Tile {
    typedef E_ E;
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, GROUP_M = 8, STAGES = STAGES_, MINB = MINB_;
    static constexpr int THREADS = 64 * WM * WN;
    static constexpr int SLAB = 128;                                  // bytes of k per row and slab
    static constexpr int BK = SLAB / (int)sizeof(E);                 // k per slab
    static constexpr int STAGE = (BM + BN) * SLAB;                   // bytes per slab of both operands
    static constexpr int HDR = 256;                                   // keeps every LDS base address non-zero
    static constexpr int LPA = BM * SLAB / 1024 / (WM * WN);         // 1 KB load instructions per wave, A
    static constexpr int LPB = BN * SLAB / 1024 / (WM * WN);         // and B
    static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
    static_assert(LPA * 1024 * WM * WN == BM * SLAB && LPB * 1024 * WM * WN == BN * SLAB, "load split");
};

template <class T, bool FUSED, bool TAIL>
__global__ __launch_bounds__(T::THREADS, T::MINB) void k_gemm_mfma2(const typename T::E *__restrict__ A, int64_t lda,
                                                             const typename T::E *__restrict__ Bt, int64_t ldb,
                                                             typename T::E *__restrict__ C, int64_t ldc, int64_t M,
                                                             int64_t N, int64_t K, int accumulate, EpiArgs epi) {
    typedef typename T::E E;
    typedef MfmaOps<E> Ops;
    typedef typename Ops::vec16 v16;
    constexpr int BM = T::BM, BN = T::BN, SLAB = T::SLAB, STAGE = T::STAGE, HDR = T::HDR, STAGES = T::STAGES;
    constexpr int LPA = T::LPA, LPB = T::LPB, LP = LPA + LPB, TM = T::TM, TN = T::TN;
    constexpr int VEC = 16 / (int)sizeof(E);
    __shared__ __attribute__((aligned(16))) uint8_t lds[HDR + STAGES * STAGE];

    const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int64_t tm, tn;
    tile_of<T::GROUP_M>(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    const int64_t row0 = tm * BM, col0 = tn * BN;

    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wm = wave / T::WN, wn = wave % T::WN;

    // global sources of this lane's chunks per slab (swizzled on the global side)
    const E *srcA[LPA];
    const E *srcB[LPB];
#pragma unroll
    for (int q = 0; q < LPA; ++q) {
        const int c = (wave * LPA + q) * 64 + lane, r = c / 8, slot = c % 8;
        const int64_t ga = row0 + r < M ? row0 + r : M - 1;
        srcA[q] = A + ga * lda + (slot ^ ((r >> 1) & 7)) * VEC;
    }
#pragma unroll
    for (int q = 0; q < LPB; ++q) {
        const int c = (wave * LPB + q) * 64 + lane, r = c / 8, slot = c % 8;
        const int64_t gb = col0 + r < N ? col0 + r : N - 1;
        srcB[q] = Bt + gb * ldb + (slot ^ ((r >> 1) & 7)) * VEC;
    }
    const int64_t nk = (K + T::BK - 1) / T::BK;
    auto load = [&](int buf, auto at) {
        uint8_t *a = lds + HDR + buf * STAGE + wave * LPA * 1024;
        uint8_t *b = lds + HDR + buf * STAGE + BM * SLAB + wave * LPB * 1024;
#pragma unroll
        for (int q = 0; q < LPA; ++q)
            __builtin_amdgcn_global_load_lds((const void *)(srcA[q] + at(wave * LPA + q)), (void *)(a + q * 1024), 16, 0,
                                             0);
#pragma unroll
        for (int q = 0; q < LPB; ++q)
            __builtin_amdgcn_global_load_lds((const void *)(srcB[q] + at(wave * LPB + q)), (void *)(b + q * 1024), 16, 0,
                                             0);
    };
    auto issue = [&](int64_t slab) {
        load((int)(slab % STAGES), [&](int) { return slab * T::BK; });
    };
    // the last slab of a K that is not a multiple of it: a chunk at or past K is
    // fetched from the row's last chunk instead (its fragments are zeroed below)
    auto issue_any = [&](int64_t slab) {
        if (TAIL && slab == nk - 1)
            load((int)(slab % STAGES), [&](int inst) {
                const int c = inst * 64 + lane, kc = ((c % 8) ^ ((c / 8 >> 1) & 7)) * VEC;
                return min(slab * T::BK, K - VEC - kc);
            });
        else issue(slab);
    };

    typename Ops::acc acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = typename Ops::acc{};

    // Two steps per slab, one 16-byte chunk of each fragment row per step:
    // binary64 chunk 2 (lane / 16) + step (two k, so the four k of a lane's
    // group take both steps), binary32 chunk 4 step + lane / 16 (four k).
    const int lr = lane % 16, lq = lane / 16;
    const int arow = wm * (BM / T::WM) + lr, brow = wn * (BN / T::WN) + lr;
    auto chunk = [&](int step) { return sizeof(E) == 8 ? 2 * lq + step : 4 * step + lq; };
    auto read = [&](int64_t slab, int step, v16 (&fa)[TM], v16 (&fb)[TN]) {
        const uint8_t *As = lds + HDR + (int)(slab % STAGES) * STAGE, *Bs = As + BM * SLAB;
        const int kc = chunk(step);
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            const int r = arow + 16 * a;
            fa[a] = *(const v16 *)(As + r * SLAB + ((kc ^ ((r >> 1) & 7)) << 4));
        }
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int r = brow + 16 * b;
            fb[b] = *(const v16 *)(Bs + r * SLAB + ((kc ^ ((r >> 1) & 7)) << 4));
        }
    };
    auto mma = [&](const v16 (&fa)[TM], const v16 (&fb)[TN]) {
#pragma unroll
        for (int q = 0; q < VEC; ++q)
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) acc[a][b] = Ops::mfma(fa[a][q], fb[b][q], acc[a][b]);
    };
    // K is a multiple of VEC: a chunk is wholly inside or wholly past it
    auto mask = [&](int64_t slab, int step, v16 (&fa)[TM], v16 (&fb)[TN]) {
        if (slab * T::BK + chunk(step) * VEC >= K) {
#pragma unroll
            for (int a = 0; a < TM; ++a) fa[a] = v16{};
#pragma unroll
            for (int b = 0; b < TN; ++b) fb[b] = v16{};
        }
    };
    // scheduling groups (masks: 0x008 MFMA, 0x020 global load, 0x100 LDS read):
    // one read, or one slab load, beside each MFMA
    auto spread = [&](bool loads) {
        if (loads) {
#pragma unroll
            for (int i = 0; i < LP; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < TM + TN; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    // Software pipeline: the fragments of a step are read while the step
    // before it is multiplied, and the slab's one barrier stands between its
    // two steps, when every wave holds the rest of the slab in registers (its
    // buffer then takes slab kt + STAGES) and slab kt + 1 has landed.
    v16 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < nk) issue_any(s);
    if (nk >= STAGES) wait_vm<(STAGES - 1) * LP>();
    else wait_vm<0>();
    bare_barrier();
    read(0, 0, fa0, fb0);
    const int64_t steady = TAIL ? nk - 1 : nk;         // slabs loaded without clamping
    int64_t kt = 0;
    for (; kt + STAGES < steady; ++kt) {
        read(kt, 1, fa1, fb1);
        mma(fa0, fb0);
        spread(false);
        __builtin_amdgcn_sched_barrier(0);
        wait_vm_lds<(STAGES - 2) * LP>();
        bare_barrier();
        issue(kt + STAGES);
        read(kt + 1, 0, fa0, fb0);
        mma(fa1, fb1);
        spread(true);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (; kt < nk; ++kt) {
        const bool last = kt + 1 == nk;
        read(kt, 1, fa1, fb1);
        if (TAIL && last) mask(kt, 0, fa0, fb0);
        mma(fa0, fb0);
        wait_vm_lds<0>();
        bare_barrier();
        if (kt + STAGES < nk) issue_any(kt + STAGES);
        if (!last) read(kt + 1, 0, fa0, fb0);
        if (TAIL && last) mask(kt, 1, fa1, fb1);
        mma(fa1, fb1);
    }

    // epilogue extras (uniform branches): the accumulator flip hook, then the
    // store with the fused partial sums; LDS is free once every wave is past the loop
    auto rowof = [](int l, int v) { return Ops::crow(l, v); };
    if (epi.fbit >= 0 && epi.fi >= row0 && epi.fi < row0 + BM && epi.fj >= col0 && epi.fj < col0 + BN)
        epi_flip(acc, epi, row0 + wm * (BM / T::WM), col0 + wn * (BN / T::WN), lane, rowof);
    if constexpr (FUSED) {
        __syncthreads();
        epi_store_fused<TM, TN, T::WM, T::WN, BM, BN>(acc, epi, (double *)(lds + HDR), row0, col0, tm, tn, M, N, wm,
                                                     wn, lane, 0, C, ldc, accumulate != 0, rowof);
        return;
    }
    // Rows of accumulator tiles at a time; with accumulate all of a row's old
    // values are requested before the first is used (one at a time cost a
    // memory latency each).  Only tiles on C's edge test their elements.
    const bool whole = row0 + BM <= M && col0 + BN <= N;
    const int64_t gr0 = row0 + wm * (BM / T::WM), gc0 = col0 + wn * (BN / T::WN) + lane % 16;
    auto store = [&](auto inside) {
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            E *row[4];
            bool rin[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t gr = gr0 + a * 16 + Ops::crow(lane, v);
                rin[v] = inside.value || gr < M;
                row[v] = C + (rin[v] ? gr : M - 1) * ldc + gc0;
            }
            if (accumulate) {
                E old[TN][4];
#pragma unroll
                for (int b = 0; b < TN; ++b)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        old[b][v] = (inside.value || (rin[v] && gc0 + b * 16 < N)) ? row[v][b * 16] : E(0);
#pragma unroll
                for (int b = 0; b < TN; ++b)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[a][b][v] = old[b][v] + acc[a][b][v];
            }
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (inside.value || (rin[v] && gc0 + b * 16 < N)) row[v][b * 16] = acc[a][b][v];
        }
    };
    if (whole) store(std::true_type{});
    else store(std::false_type{});
}

template <class T>
inline int launch_gemm_mfma2(const typename T::E *A, int64_t lda, const typename T::E *Bt, int64_t ldb,
                             typename T::E *C, int64_t ldc, int64_t M, int64_t N, int64_t K, hipStream_t s,
                             bool accumulate = false, EpiArgs *epi = nullptr) {
    const int64_t tiles = ((M + T::BM - 1) / T::BM) * ((N + T::BN - 1) / T::BN);
    if (tiles > INT32_MAX) return ABFT_E_ARG;
    EpiArgs e = epi ? *epi : epi_none();
    if (epi) {
        epi->tiles_m = (M + T::BM - 1) / T::BM;
        epi->tiles_n = (N + T::BN - 1) / T::BN;
    }
    auto run = [&](auto fused, auto tail) {
        // the fused partial sums' layout has no room for smaller tiles, and a binary64 128 x 128 tile none
        // for a ragged k's registers: such picks are not made
        constexpr bool room = !fused.value || (T::BM >= kMinTileEdge && T::BN >= kMinTileEdge);
        constexpr bool regs = !tail.value || sizeof(typename T::E) == 4 || T::BM * T::BN < 128 * 128;
        if constexpr (room && regs) {
            k_gemm_mfma2<T, fused.value, tail.value><<<(unsigned)tiles, T::THREADS, 0, s>>>(A, lda, Bt, ldb, C, ldc, M, N,
                                                                                           K, accumulate, e);
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
