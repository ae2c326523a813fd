// Carried checksum blocks of C_f computed as skinny products with binary64
// accumulation (the "sliver" path, used when a checksum block is thinner than
// a matrix-core tile):
//   carried row block    C_f[m + r, j] = sum_l (C_C^T A)[r, l] B_f[l, j]   (r < br, j < N)
//   carried column block C_f[i, n + c] = sum_l A_f[i, l] (B C_R)[l, c]     (i < rows, c < bc)
// Both have the form out[u, s] = sum_l X[u, l] Y[s, l] with many rows u (a
// whole operand, streamed once from HBM) and few rows s (the checksum rows,
// L2-resident).  A wave owns one u, or several; lanes stride k with 16-byte
// loads; the few partial sums are folded with wavefront shuffles.
//
// HBM-bound.  The chunks of the next step are requested before the current
// ones are summed: with a step's loads, wait and sums in turn the rate stays
// at 5 TB/s however many rows share a wave, with the next step in flight it is
// 6.5 (2.1 GB binary64 operand against two rows, four rows per wave: 401 us
// and 330).  With a short k the sums over the lanes and the waves in flight
// count instead: the sums go by a reduce-scatter and widened values are held a
// part at a time (whole products, us, butterflies and whole chunks widened
// against this: FP8 215241 x 5 x 16 79 and 53, FP8 blocks of 512 362312 x 512 x
// 16 42034 and 27672, bfloat16 342573 x 62 x 16 106 and 79; 4096 x 4096 x 1024
// FP8 blocks of 16 83 and 74).
#pragma once

#include <type_traits>

#include "common.h"

namespace abft {

constexpr int kSliverThreads = 256;
constexpr int kSliverR = 8;   // few rows per pass

// out = v, or out += v (accumulate: the sum is taken in binary64 and rounded once)
template <typename T> __device__ inline void store_out(T *p, double v, bool accumulate);
template <> __device__ inline void store_out<double>(double *p, double v, bool accumulate) {
    *p = accumulate ? *p + v : v;
}
template <> __device__ inline void store_out<float>(float *p, double v, bool accumulate) {
    *p = (float)(accumulate ? (double)*p + v : v);
}

// X: U rows of type TX (ldx); Y: R rows of type TY (ldy), R <= kSliverR per launch.
// out[u*ou + s*os] = scale * sum_l X[u,l] Y[s,l].  K is a multiple of both vector widths.
template <typename TX, typename TY, typename TC> struct SliverJob {
    const TX *X;
    int64_t ldx, U;
    const TY *Y;
    int64_t ldy;
    int R;
    int64_t K;
    TC *out;
    int64_t ou, os;
    unsigned blocks;
};

// What else one launch may do: the corner of binary32 checksum rows,
// C_f[m + r, n + c] = scale * sum_l Yr[r, l] Yc[c, l], a block per entry, and the
// owner tag of the fused partial sums.
struct SliverExtra {
    const float *Yr, *Yc;     // null: no corner
    int64_t K, nc;            // columns of the corner
    float *out;
    int64_t ldo;
    unsigned blocks;
    uint64_t *tag;            // null: none
    uint64_t key;
    const int *scale_exp;     // FP8 scale exponents: scale = 2^-(e[0] + e[1]); null: 1
    int accumulate;
};
inline SliverExtra sliver_extra(const int *scale_exp, bool accumulate) {
    SliverExtra x{};
    x.scale_exp = scale_exp;
    x.accumulate = accumulate ? 1 : 0;
    return x;
}

// NR rows of X per wave, NY >= R rows of Y (rows at and past R repeat the last,
// and are not stored), UK chunks of k per lane in a step.  Every count of rows has
// an NY of its own: the checksum rows' reads from L2 and their widening are most
// of the work (five rows in eight places and in five, us, whole products: FP8
// 120 x 71585 x 1376 260 and 174, bfloat16 125 x 53450 x 792 84 and 65, binary64
// 25 x 36170 x 262 52 and 43).
template <typename TX, typename TY, typename TC, int NR, int NY, int UK, bool NT>
__device__ __attribute__((always_inline)) inline void sliver_rows(const SliverJob<TX, TY, TC> &j, double scale,
                                                                  bool accumulate, int64_t block) {
    constexpr int VX = vec16<TX>::N, VY = vec16<TY>::N;
    constexpr int V = VX > VY ? VX : VY;             // k per lane per chunk
    constexpr bool PFY = NY * (V / VY) <= 4;         // Y's chunks requested ahead too (as registers allow)
    const int lane = threadIdx.x % 64;
    const int64_t wave = block * (kSliverThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int64_t nwaves = (int64_t)j.blocks * (kSliverThreads / 64);
    for (int64_t u0 = wave * NR; u0 < j.U; u0 += nwaves * NR) {
        double acc[NR][NY];
        const TX *xr[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
#pragma unroll
            for (int y = 0; y < NY; ++y) acc[r][y] = 0.0;
            xr[r] = j.X + min(u0 + r, j.U - 1) * j.ldx;  // rows past U re-read the last (not stored)
        }
        // a chunk at or past K is clamped to the step's first and not summed
        auto at = [&](int64_t k0, int c) { return k0 + c * 64 * V < j.K ? k0 + c * 64 * V : k0; };
        auto get_x = [&](v4u32 (&x)[UK][NR][V / VX], int64_t k0) {
#pragma unroll
            for (int c = 0; c < UK; ++c)
#pragma unroll
                for (int r = 0; r < NR; ++r)
#pragma unroll
                    for (int q = 0; q < V / VX; ++q) x[c][r][q] = load_raw<NT, v4u32>(xr[r] + at(k0, c) + q * VX);
        };
        auto get_y = [&](v4u32 (&yw)[UK][NY][V / VY], int64_t k0) {
#pragma unroll
            for (int c = 0; c < UK; ++c)
#pragma unroll
                for (int y = 0; y < NY; ++y)
#pragma unroll
                    for (int q = 0; q < V / VY; ++q)
                        yw[c][y][q] = *(const v4u32 *)(j.Y + (int64_t)min(y, j.R - 1) * j.ldy + at(k0, c) + q * VY);
        };
        v4u32 nx[UK][NR][V / VX], ny[UK][NY][V / VY];
        int64_t k0 = (int64_t)lane * V;
        if (k0 < j.K) {
            get_x(nx, k0);
            if constexpr (PFY) get_y(ny, k0);
        }
        for (; k0 < j.K; k0 += UK * 64 * V) {
            v4u32 xw[UK][NR][V / VX], yw[UK][NY][V / VY];
#pragma unroll
            for (int c = 0; c < UK; ++c) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
#pragma unroll
                    for (int q = 0; q < V / VX; ++q) xw[c][r][q] = nx[c][r][q];
                if constexpr (PFY) {
#pragma unroll
                    for (int y = 0; y < NY; ++y)
#pragma unroll
                        for (int q = 0; q < V / VY; ++q) yw[c][y][q] = ny[c][y][q];
                }
            }
            if constexpr (!PFY) get_y(yw, k0);
            if (k0 + UK * 64 * V < j.K) {
                get_x(nx, k0 + UK * 64 * V);
                if constexpr (PFY) get_y(ny, k0 + UK * 64 * V);
            }
            // a part of four (binary64: two) k at a time, so that few widened values are held
            constexpr int P = vec16<TX>::P;
            static_assert(P == VY && VX % P == 0, "a part is a chunk of Y");
#pragma unroll
            for (int c = 0; c < UK; ++c) {
                if (k0 + c * 64 * V >= j.K) break;
#pragma unroll
                for (int p = 0; p < V / P; ++p) {
                    double xv[NR][P];
#pragma unroll
                    for (int r = 0; r < NR; ++r) vec16<TX>::widen_part(xw[c][r][p * P / VX], p * P % VX / P, xv[r]);
#pragma unroll
                    for (int y = 0; y < NY; ++y) {
                        double yv[P];
                        vec16<TY>::widen(yw[c][y][p], yv);
#pragma unroll
                        for (int r = 0; r < NR; ++r)
#pragma unroll
                            for (int q = 0; q < P; ++q) acc[r][y] = fma(xv[r][q], yv[q], acc[r][y]);
                    }
                }
            }
        }
        // the NR NY sums over the lanes by a reduce-scatter: each exchange halves the sums a lane holds until one
        // is left, then a butterfly within the lanes that share it -- per sum the same additions as a butterfly
        // over the wave, with about a fifth of the exchanges for eight sums (what a short k spends its time on)
        constexpr int NYP = NY <= 2 ? NY : (NY <= 4 ? 4 : 8), NS = NR * NYP;
        static_assert((NS & (NS - 1)) == 0 && NS <= 64, "a power of two");
        double v[NS];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int y = 0; y < NYP; ++y) v[r * NYP + y] = y < NY ? acc[r][y < NY ? y : 0] : 0.0;
#pragma unroll
        for (int off = 32, h = NS / 2; off > 0; off >>= 1, h >>= 1) {
            if (h > 0) {
                const bool up = lane & off;
#pragma unroll
                for (int e = 0; e < h; ++e) {
                    const double keep = up ? v[e + h] : v[e], send = up ? v[e] : v[e + h];
                    v[e] = keep + __shfl_xor(send, off, 64);
                }
            } else {
                v[0] += __shfl_xor(v[0], off, 64);
            }
        }
        const int e = lane / (64 / NS), r = e / NYP, y = e % NYP;
        if (lane % (64 / NS) == 0 && u0 + r < j.U && y < j.R)
            store_out<TC>(j.out + (u0 + r) * j.ou + y * j.os, scale * v[0], accumulate);
    }
}

__device__ inline void sliver_corner(const SliverExtra &x, double scale, int64_t e) {
    __shared__ double sh[kSliverThreads / 64];
    const int64_t r = e / x.nc, c = e - r * x.nc;
    const float *a = x.Yr + r * x.K, *b = x.Yc + c * x.K;
    double acc = 0.0;
    for (int64_t l = (int64_t)threadIdx.x * 4; l < x.K; l += kSliverThreads * 4) {
        double av[4], bv[4];
        vec16<float>::load(a + l, av);
        vec16<float>::load(b + l, bv);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = fma(av[q], bv[q], acc);
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kSliverThreads / 64; ++q) acc += sh[q];
        x.out[r * x.ldo + c] = (float)(scale * acc);
    }
}

// The corner of wide checksum blocks in a launch of its own: a wave takes four
// columns and four rows, so that the checksum rows are read from L2 half a row
// per entry instead of two.  From kCornerTiled entries on: fewer are spread over
// more of the device a block each, beside the carried rows and columns (us, the
// whole bfloat16 product 4096 x 4096 x 2048 with checksum blocks of 64, 128, 256
// and 1024, the corner by blocks 252 / 457 / 906 / 4478, by tiles 252 / 437 / 830
// / 3294).
constexpr int64_t kCornerTiled = 16384;
constexpr int kCornerRows = 4;
__global__ __launch_bounds__(kSliverThreads) void k_corner(SliverJob<float, float, float> j, int64_t rows,
                                                          const int *scale_exp) {
    const double scale = scale_exp ? ldexp(1.0, -(scale_exp[0] + scale_exp[1])) : 1.0;
    for (int64_t r0 = (int64_t)blockIdx.y * kCornerRows; r0 < rows; r0 += (int64_t)gridDim.y * kCornerRows) {
        SliverJob<float, float, float> p = j;
        p.Y += r0 * j.ldy;
        p.out += r0 * j.os;
        p.R = (int)min((int64_t)kCornerRows, rows - r0);
        sliver_rows<float, float, float, 4, kCornerRows, 1, false>(p, scale, false, blockIdx.x);
    }
}

// One or two jobs (blocks [0, a.blocks), then b's), then the extras.
template <typename TX, typename TY, typename TC, int NR, int NY, int UK, bool NT>
__device__ __attribute__((always_inline)) inline void sliver_launch(const SliverJob<TX, TY, TC> &a,
                                                                    const SliverJob<TX, TY, TC> &b,
                                                                    const SliverExtra &x) {
    const double scale = x.scale_exp ? ldexp(1.0, -(x.scale_exp[0] + x.scale_exp[1])) : 1.0;
    if (x.tag && blockIdx.x == 0 && threadIdx.x == 0) *x.tag = x.key;
    const unsigned blk = blockIdx.x;
    if (blk >= a.blocks + b.blocks) {
        sliver_corner(x, scale, blk - a.blocks - b.blocks);
        return;
    }
    const bool first = blk < a.blocks;
    sliver_rows<TX, TY, TC, NR, NY, UK, NT>(first ? a : b, scale, x.accumulate != 0, first ? blk : blk - a.blocks);
}
template <typename TX, typename TY, typename TC, int NY, bool NT>
__global__ __launch_bounds__(kSliverThreads, sizeof(TX) == 1 && NY >= 6 ? 2 : 4) void k_sliver(SliverJob<TX, TY, TC> a, SliverJob<TX, TY, TC> b,
                                                          SliverExtra x) {
    constexpr int V = vec16<TX>::N > vec16<TY>::N ? vec16<TX>::N : vec16<TY>::N;
    // chunks of k per lane in a step, fewer where more rows of Y hold registers
    constexpr int UK = V >= 16 ? 1 : (V >= 8 ? (NY > 2 ? 1 : 2) : (NY > 2 ? 1 : 4 / NY));
    sliver_launch<TX, TY, TC, 1, NY, UK, NT>(a, b, x);
}
// Few checksum rows over enough operand rows to fill the device: a wave takes
// several operand rows, so each chunk of Y is read once for them.  Per row the
// same sums in the same order as k_sliver.  HBM-bound: what counts is the bytes
// in flight and how often Y is read.  binary64, whose chunk is only two k, takes
// two rows and four chunks (17408 x 16384, two checksum rows: 368 us, 6.2 TB/s;
// four rows and one chunk 409, two and two 383, one and eight 444); the shorter
// types four rows and one chunk (two rows: binary32 16384 x 16384 169 us against
// 163, FP8 16384 x 16384 twice 138 against 120, bfloat16 16384 x 1024 twice 25
// against 22).
// A k of a chunk or two leaves nothing to keep in flight but rows: four rows
// then for binary64 too (whole product 111487 x 23 x k, two rows and four: k 72
// 56 and 38 us, 200 74 and 68, 256 81 and 79, 384 125 and 126, 512 167 and 178;
// 349475 x 29 x 8 123 and 74).
template <typename TX> constexpr int kSliverRows = sizeof(TX) == 8 ? 2 : 4;
template <typename TX> inline bool sliver_short(int64_t K) { return sizeof(TX) == 8 && K <= 256; }
template <typename TX, typename TY, typename TC, int NY, bool NT, int NR>
__global__ __launch_bounds__(kSliverThreads, sizeof(TX) == 8 ? 1 : (NY == 1 ? 4 : 3)) void k_sliver1(
    SliverJob<TX, TY, TC> a, SliverJob<TX, TY, TC> b, SliverExtra x) {
    sliver_launch<TX, TY, TC, NR, NY, NR == 2 ? 4 : 1, NT>(a, b, x);
}
inline bool sliver_multirow(int64_t R, int64_t U) { return R <= 2 && U >= 16384; }

// One or two skinny products (b null: one) and the extras, which go with the last launch.
template <typename TX, typename TY, typename TC>
inline int slivers(SliverJob<TX, TY, TC> a, const SliverJob<TX, TY, TC> *b, const SliverExtra &x, hipStream_t s) {
    typedef SliverJob<TX, TY, TC> Job;
    SliverExtra plain = sliver_extra(x.scale_exp, x.accumulate != 0);
    // at most kSliverR checksum rows of one job per launch
    auto run = [&](Job u, Job v, bool with_v, const SliverExtra &e) {
        if (!with_v) { v = u; v.blocks = 0; }
        const int64_t per_block = kSliverThreads / 64;
        const bool multi = sliver_multirow(u.R, u.U), brief = sliver_short<TX>(u.K);
        auto blocks = [&](const Job &j) {
            const int64_t rows = brief ? 4 : kSliverRows<TX>, waves = multi ? (j.U + rows - 1) / rows : j.U;
            return (unsigned)std::min<int64_t>((waves + per_block - 1) / per_block, 4096);
        };
        u.blocks = blocks(u);
        if (with_v) v.blocks = blocks(v);
        const int R = with_v ? std::max(u.R, v.R) : u.R;
        const bool nt = streams(std::max(u.U, with_v ? v.U : 0) * u.K * (int64_t)sizeof(TX));
        const unsigned grid = u.blocks + v.blocks + e.blocks;
        auto go = [&](auto ny, auto st) {
            constexpr int NY = decltype(ny)::value;
            constexpr bool NT = decltype(st)::value;
            if (multi) {
                if constexpr (NY <= 2) {
                    if (brief) k_sliver1<TX, TY, TC, NY, NT, 4><<<grid, kSliverThreads, 0, s>>>(u, v, e);
                    else k_sliver1<TX, TY, TC, NY, NT, kSliverRows<TX>><<<grid, kSliverThreads, 0, s>>>(u, v, e);
                }
            } else {
                k_sliver<TX, TY, TC, NY, NT><<<grid, kSliverThreads, 0, s>>>(u, v, e);
            }
        };
        auto by_ny = [&](auto st) {
            if (R == 1) go(std::integral_constant<int, 1>{}, st);
            else if (R == 2) go(std::integral_constant<int, 2>{}, st);
            else if (R == 3) go(std::integral_constant<int, 3>{}, st);
            else if (R == 4) go(std::integral_constant<int, 4>{}, st);
            else if (R == 5) go(std::integral_constant<int, 5>{}, st);
            else if (R == 6) go(std::integral_constant<int, 6>{}, st);
            else if (R == 7) go(std::integral_constant<int, 7>{}, st);
            else go(std::integral_constant<int, 8>{}, st);
        };
        nt ? by_ny(std::true_type{}) : by_ny(std::false_type{});
    };
    auto piece = [](Job j, int r0) {
        j.Y += r0 * j.ldy;
        j.out += r0 * j.os;
        j.R = std::min(j.R - r0, kSliverR);
        return j;
    };
    const bool one = b && a.R == b->R && a.R <= kSliverR && sliver_multirow(a.R, a.U) == sliver_multirow(b->R, b->U);
    if (one) {
        run(a, *b, true, x);
    } else {
        for (int r = 0; r < a.R; r += kSliverR) run(piece(a, r), a, false, !b && r + kSliverR >= a.R ? x : plain);
        for (int r = 0; b && r < b->R; r += kSliverR) run(piece(*b, r), a, false, r + kSliverR >= b->R ? x : plain);
    }
    ABFT_LAUNCHED();
    return ABFT_OK;
}

template <typename TX, typename TY, typename TC>
inline SliverJob<TX, TY, TC> sliver_job(const TX *X, int64_t ldx, int64_t U, const TY *Y, int64_t ldy, int64_t R, int64_t K,
                                        TC *out, int64_t ou, int64_t os) {
    return SliverJob<TX, TY, TC>{X, ldx, U, Y, ldy, (int)R, K, out, ou, os, 0};
}

// Carried row block: C_f[m + r, 0:N) = sum_l Acs[r, l] Bt[j, l] (checksum rows Acs, br x K; the
// operands may start at a k offset, K is the panel depth).
template <typename E>
inline SliverJob<E, E, E> sliver_carried_rows(const Geom &g, const E *Acs, int64_t ldacs, const E *Bt, int64_t ldb, E *C,
                                              int64_t ldc, int64_t K) {
    return sliver_job<E, E, E>(Bt, ldb, g.N, Acs, ldacs, g.br, K, C + g.m * ldc, 1, ldc);
}
// Carried column block: C_f[0:rows, n + c) = sum_l A[i, l] Bcs[c, l] (checksum columns Bcs, bc x K).
template <typename E>
inline SliverJob<E, E, E> sliver_carried_cols(const Geom &g, int64_t rows, const E *A, int64_t lda, const E *Bcs,
                                              int64_t ldbcs, E *C, int64_t ldc, int64_t K) {
    return sliver_job<E, E, E>(A, lda, rows, Bcs, ldbcs, g.bc, K, C + g.n, ldc, 1);
}

}  // namespace abft
