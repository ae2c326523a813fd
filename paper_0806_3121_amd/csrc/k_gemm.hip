// Protected product C_f = A_f B_f (Eq. ABFT-GEMM) dispatch.
//
// The data part and any thick checksum block (b > kSliverMaxB) run on the
// matrix cores (gemm_mfma2_kernel.h / gemm_mfma_kernel.h for binary64 and
// binary32, gemm_lowp2_kernel.h / gemm_lowp_ring_kernel.h for bfloat16 and FP8).
// A thin checksum block (b <= kSliverMaxB, e.g. the classic b = 1) would
// occupy a whole row or column of tiles for a few useful rows, so it is
// computed instead by the skinny-product kernel (sliver_kernel.h), which
// streams the other operand once with binary64 accumulation.  The tile pick
// lives in one function per element type, used by the launch and by
// abft_describe_gemm alike.
#include "gemm_lowp2_kernel.h"
#include "gemm_lowp_ring_kernel.h"
#include "gemm_mfma2_kernel.h"
#include "gemm_mfma_kernel.h"
#include "sliver_kernel.h"

#include <cstdio>

namespace abft {

constexpr int64_t kSliverMaxB = 8;

struct TileChoice { int id; int bm, bn; double eff; int per_cu = 0; };   // per_cu: tiles that share a CU, for choose_tile alone

// Estimated time ~ rounds x time per round (tile area / per-tile efficiency);
// the smallest wins.  A round is one tile on each of the 256 CUs: tiles that
// share a CU share its matrix cores, so only their number per CU counts.
// Returns the index of the pick in tab.
static int choose_rounds(const TileChoice *tab, int n, int64_t M, int64_t N) {
    double best = 0;
    int pick = 0;
    for (int q = 0; q < n; ++q) {
        const TileChoice &t = tab[q];
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        const double cost = (double)((tiles + 255) / 256) * t.bm * t.bn / t.eff;
        if (best == 0 || cost < best) { best = cost; pick = q; }
    }
    return pick;
}
// The same with rounds of per_cu resident tiles per CU.
static int choose_tile(const TileChoice *tab, int n, int64_t M, int64_t N) {
    double best = 0;
    int pick = 0;
    for (int q = 0; q < n; ++q) {
        const TileChoice &t = tab[q];
        int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        int64_t slots = 256 * t.per_cu;
        double rounds = (double)((tiles + slots - 1) / slots);
        double cost = rounds * (double)t.bm * t.bn * t.per_cu / t.eff;
        if (best == 0 || cost < best) { best = cost; pick = q; }
    }
    return pick;
}

// binary64 / binary32 direct-to-LDS candidates.  eff: share of the matrix
// cores' rate with many rounds (at 2048 .. 9216 squared, k 2048 .. 16384), which orders
// the tiles as measured, for instance (us, binary64 128x128 / 128x96 / 96x96 /
// 64x64 / 32x32): 2048^3 241 / 354 / 271 / 248 / 294, 2001 x 1503 x 1234
// 153 / 115 / 167 / 121 / 158, 5120 x 5120 x 4096 3260 / 3143 / 3171 / 3036 / 3626,
// 1024^3 121 / 93 / 71 / 38 / 40, 512^3 63 / 48 / 37 / 19 / 8.7, 256^3
// 34 / 26 / 21 / 11 / 7.7; binary32 256x128 / 128x128 / 64x64 / 32x32:
// 2001 x 1503 x 1236 150 / 81 / 66 / 81, 2048^3 238 / 126 / 131 / 149.
// A 256 x 128 binary64 tile measured the same as 128 x 128 and is not offered.
static const TileChoice kF64DirectTiles[] = {
    {1, 128, 128, 0.94}, {2, 128, 96, 0.935}, {3, 96, 96, 0.94}, {4, 64, 64, 0.90}, {5, 32, 32, 0.75},
};
static const TileChoice kF32DirectTiles[] = {
    {0, 256, 128, 0.93}, {1, 128, 128, 0.917}, {4, 64, 64, 0.868}, {5, 32, 32, 0.736},
};
// The fused partial sums in the workspace have room for tiles of this edge and more.
constexpr int kF64FusedTiles = 3, kF32FusedTiles = 2;

// Short and small products: the direct tiles at their rates with two blocks per CU, and the register-staged
// kernel's for a ragged k.
static const TileChoice kF64ShortTiles[] = {
    {1, 128, 128, 0.87, 2}, {2, 128, 96, 0.89, 2}, {3, 96, 96, 0.88, 2},
};
static const TileChoice kF32ShortTiles[] = {
    {0, 256, 128, 0.85, 1}, {1, 128, 128, 0.84, 2},
};
static const TileChoice kF64Tiles[] = {
    {0, 256, 128, 0.818, 1}, {1, 128, 128, 0.787, 2}, {2, 128, 96, 0.80, 2}, {3, 96, 96, 0.76, 2},
};
static const TileChoice kF32Tiles[] = {
    {0, 256, 128, 0.80, 1}, {1, 128, 128, 0.78, 2},
};

// The data-part kernel and tile for an M x N x K product of element type E.
struct MainPick {
    bool direct;            // direct-to-LDS kernel for whole slabs only in low precision (else register-staged / ring)
    const TileChoice *t;
};
// Whether an M x N x K product (K in slabs of BK) is picked from the direct
// tiles by rounds.  Below four slabs a launch is mostly its start and its
// stores and the pick matters little (binary64 776 x 5384 x 32: 13 us with any
// tile; 1032 x 5384 x 48: 17 to 23).  The small products of a ragged k or a fused
// epilogue excluded here would gain from it too (320 x 320 x 250: 21 us on the
// register-staged kernel, 8 on a direct tile): they stay with the kernel that the
// numeric checks of that kernel's tiles run at these sizes, which is why the line
// lies there and not where the time says.
static bool by_rounds(int64_t M, int64_t N, int64_t K, int64_t BK, bool fused) {
    const int64_t least = fused ? int64_t(1) << 18 : (K % BK ? int64_t(1) << 17 : 0);
    return K >= 4 * BK && M * N > least;
}
static MainPick pick_main(const double *, int64_t M, int64_t N, int64_t K, bool fused) {
    if (by_rounds(M, N, K, 16, fused)) {
        // a ragged k needs a few more registers than 128 x 128 leaves free
        const int skip = K % 16 ? 1 : 0, n = (fused ? kF64FusedTiles : 5) - skip;
        return {true, &kF64DirectTiles[skip + choose_rounds(kF64DirectTiles + skip, n, M, N)]};
    }
    if (K % 16 == 0) return {true, &kF64ShortTiles[choose_tile(kF64ShortTiles, 3, M, N)]};
    return {false, &kF64Tiles[choose_tile(kF64Tiles, 4, M, N)]};
}
static MainPick pick_main(const float *, int64_t M, int64_t N, int64_t K, bool fused) {
    if (by_rounds(M, N, K, 32, fused))
        return {true, &kF32DirectTiles[choose_rounds(kF32DirectTiles, fused ? kF32FusedTiles : 4, M, N)]};
    if (K % 32 == 0) return {true, &kF32ShortTiles[choose_tile(kF32ShortTiles, 2, M, N)]};
    return {false, &kF32Tiles[choose_tile(kF32Tiles, 2, M, N)]};
}

static int gemm_main(const double *A, int64_t lda, const double *Bt, int64_t ldb, double *C, int64_t ldc, int64_t M,
                     int64_t N, int64_t K, hipStream_t s, bool acc = false, EpiArgs *e = nullptr) {
    const MainPick pk = pick_main(A, M, N, K, e && e->pc);
    if (pk.direct) {
        switch (pk.t->id) {
        case 1:
            return launch_gemm_mfma2<Mfma2Tile<double, 2, 128, 128, 2, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s,
                                                                             acc, e);
        case 2:
            return launch_gemm_mfma2<Mfma2Tile<double, 2, 128, 96, 2, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc,
                                                                            e);
        case 4:
            return launch_gemm_mfma2<Mfma2Tile<double, 2, 64, 64, 2, 2, 4>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
        case 5:
            return launch_gemm_mfma2<Mfma2Tile<double, 4, 32, 32, 2, 2, 4>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
        default:
            return launch_gemm_mfma2<Mfma2Tile<double, 2, 96, 96, 2, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc,
                                                                           e);
        }
    }
    switch (pk.t->id) {
    case 0: return launch_gemm_tile<MfmaTile<double, 256, 128, 16, 4, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
    case 1: return launch_gemm_tile<MfmaTile<double, 128, 128, 16, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
    case 2:
        return launch_gemm_tile<MfmaTile<double, 128, 96, 16, 2, 2, 8, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc,
                                                                          e);
    default:
        return launch_gemm_tile<MfmaTile<double, 96, 96, 16, 2, 2, 8, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
    }
}

static int gemm_main(const float *A, int64_t lda, const float *Bt, int64_t ldb, float *C, int64_t ldc, int64_t M,
                     int64_t N, int64_t K, hipStream_t s, bool acc = false, EpiArgs *e = nullptr) {
    const MainPick pk = pick_main(A, M, N, K, e && e->pc);
    if (pk.direct) {
        switch (pk.t->id) {
        case 0: return launch_gemm_mfma2<Mfma2Tile<float, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
        case 4:
            return launch_gemm_mfma2<Mfma2Tile<float, 4, 64, 64, 2, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
        case 5:
            return launch_gemm_mfma2<Mfma2Tile<float, 4, 32, 32, 2, 2, 4>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
        default:
            return launch_gemm_mfma2<Mfma2Tile<float, 2, 128, 128, 2, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc,
                                                                            e);
        }
    }
    switch (pk.t->id) {
    case 0: return launch_gemm_tile<MfmaTile<float, 256, 128, 32, 4, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
    default: return launch_gemm_tile<MfmaTile<float, 128, 128, 32, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, s, acc, e);
    }
}

// Where the owner tag of the fused partial sums is still to be stored; its
// value depends on the tile grid the main launch has filled in.  The carried
// blocks' launch stores it and clears dst.
struct TagStore {
    uint64_t *dst;
    const abft_problem *p;
    const void *C_f;
    bool fused;
    const EpiArgs *e;
    uint64_t key() const {
        if (!fused) return 0;
        int64_t tm = 0, tn = 0;
        const uint64_t k = fused_key(p, C_f, &tm, &tn);
        return tm == e->tiles_m && tn == e->tiles_n ? k : 0;   // 0: a grid the fused verification would not read
    }
};

// C_f = (acc ? C_f : 0) + A_f[:, k0:k0+K) B_f[k0:k0+K, :)  (the whole product: k0 = 0, K = k).
template <typename E>
static int protected_product(const abft_problem *p, const Geom &g, const E *A, const E *Bt, E *C, bool plain,
                             hipStream_t s, int64_t k0 = 0, int64_t K = -1, bool acc = false,
                             EpiArgs *e = nullptr, TagStore *tag = nullptr) {
    if (K < 0) K = g.k;
    const bool thin_r = !plain && g.S * g.br <= kSliverMaxB;
    const bool thin_c = !plain && g.S * g.bc <= kSliverMaxB;
    int64_t Mm = (plain || thin_r) ? g.m : g.M;
    int64_t Nm = (plain || thin_c) ? g.n : g.N;
    const E *Ak = A + k0, *Bk = Bt + k0;
    int st = gemm_main(Ak, p->lda, Bk, p->ldb, C, p->ldc, Mm, Nm, K, s, acc, e);
    if (st) return st;
    ABFT_LAUNCHED();
    // the carried row block over all N columns (corner included) and the carried
    // column block over the rows the main product covered, in one launch
    SliverExtra x = sliver_extra(nullptr, acc);
    if (tag && (thin_r || thin_c)) { x.tag = tag->dst; x.key = tag->key(); tag->dst = nullptr; }
    const auto cols = sliver_carried_cols<E>(g, Mm, Ak, p->lda, Bk + g.n * p->ldb, p->ldb, C, p->ldc, K);
    if (thin_r)
        return slivers(sliver_carried_rows<E>(g, Ak + g.m * p->lda, p->lda, Bk, p->ldb, C, p->ldc, K),
                       thin_c ? &cols : nullptr, x, s);
    if (thin_c) return slivers(cols, (decltype(&cols))nullptr, x, s);
    return ABFT_OK;
}

// bfloat16 / FP8 candidates, picked by rounds.  eff orders the tiles as measured
// (us, 256x256 / 256x128 / 128x128 / 64x64): bfloat16 16384^3 6557 / 8428 / 7981 /
// 17138, 8431 x 8116 x 8824 1272 / 1465 / 1522 / 3060, 3000 x 5003 x 2056
// 66 / 81 / 84 / 171, 2048^3 43 / 32 / 26 / 28, 440 x 11551 x 1832 51 / 37 / 45 / 67,
// 861 x 765 x 4504 108 / 70 / 51 / 26, 1024^3 24 / 18 / 12 / 11; FP8 3000 x 5003 x
// 2064 44 / 52 / 53 / 95, 1570 x 3468 x 880 25 / 18 / 17 / 19, 2048^3
// 27 / 22 / 16 / 17, 861 x 765 x 4512 51 / 37 / 28 / 15.  The 64 x 64 tile is not
// offered to a fused epilogue, whose sums have no room for it.  Below eight slabs
// of k, where a launch is mostly its start and stores, it is the tile of products
// no wider than itself (bfloat16 299247 x 26 x 32: 19 us, 128x128 29, FP8 16 x
// 289750 x 352: 24 and 33) -- in FP8, whose 128 bytes are more of k, below four
// slabs of those up to 192 wide too (164827 x 65 x 192: 23 us, 256x128 30;
// 269714 x 162 x 144 48 and 70, 93 x 164860 x 336 27 and 32; but 163 x 45118 x 896
// 29 and 22, and in bfloat16 166 x 170184 x 328 75 and 60) -- and not offered to
// others (FP8 500 x 600 x 528: 10.9 us with either small tile).
// A whole number of rounds away the order moves with k and the rows' alignment by a
// few percent only (68015 x 1008 x 752: 183 / 189 / 184); 128x128 needs three rounds
// and more to come near its rate (4913 x 2276 x 2976: 93 us, 256x256 77).
// When k is a multiple of the 128-byte slab the 256 x 256 tile runs in the kernel
// made for that (16384^3: 6472 us, 6421 in the ring).
static const TileChoice kLowpTiles[] = {
    {0, 256, 256, 0.50}, {3, 256, 128, 0.36}, {1, 128, 128, 0.35}, {2, 64, 64, 0.195},
};
static MainPick pick_main_lowp(int64_t elem_size, int64_t M, int64_t N, int64_t K, bool fused) {
    const int64_t slab = 128 / elem_size;
    const bool brief = K < 8 * slab;
    const int64_t narrow = elem_size == 1 && K < 4 * slab ? 192 : 64;
    if (brief && !fused && std::min(M, N) <= narrow) return {false, &kLowpTiles[3]};
    const TileChoice *t = &kLowpTiles[choose_rounds(kLowpTiles, fused || brief ? 3 : 4, M, N)];
    return {t->bm == 256 && t->bn == 256 && K % slab == 0, t};
}
// The ring's depth by what shares a CU: where the small tiles are no more than
// the device holds at once with deep rings, four slabs in flight cover a lone
// block's latency (bfloat16 861 x 765 x 4504 on 64x64: 26 us, two slabs 35; 2048^3 on
// 128x128: 25.8 and 26.3); else two slabs and more blocks per CU (128 x 101760 x 2376
// on 128x128: 169 us, four slabs 173; 336023 x 135 x 232 110 and 162).
template <class Ops>
static int gemm_main_lowp(const typename Ops::E *A, int64_t lda, const typename Ops::E *Bt, int64_t ldb, float *C,
                          int64_t ldc, int64_t M, int64_t N, int64_t K, const int *scale_exp, hipStream_t s,
                          EpiArgs *e = nullptr) {
    const MainPick pk = pick_main_lowp((int64_t)sizeof(typename Ops::E), M, N, K, e && e->pc);
    if (pk.direct) return launch_gemm_lowp2<Ops, 4>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s, e);
    const int64_t tiles = ((M + pk.t->bm - 1) / pk.t->bm) * ((N + pk.t->bn - 1) / pk.t->bn);
    switch (pk.t->id) {
    case 0:
        return launch_gemm_lowp<LowpRing<Ops, 256, 256, 4, 2, 1, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s, e);
    case 2:
        if (tiles <= 512)
            return launch_gemm_lowp<LowpRing<Ops, 64, 64, 2, 2, 2, 4>>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s, e);
        return launch_gemm_lowp<LowpRing<Ops, 64, 64, 2, 2, 4, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s, e);
    case 3:
        return launch_gemm_lowp<LowpRing<Ops, 256, 128, 4, 2, 1, 3>>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s, e);
    default:
        if (tiles <= 256)
            return launch_gemm_lowp<LowpRing<Ops, 128, 128, 2, 2, 1, 4>>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s,
                                                                        e);
        return launch_gemm_lowp<LowpRing<Ops, 128, 128, 2, 2, 2, 2>>(A, lda, Bt, ldb, C, ldc, M, N, K, scale_exp, s, e);
    }
}

// Low-precision operands: the data part on the matrix cores, every carried
// block from the binary32 checksum rows in the workspace (Acs: br x k,
// Bcs: bc x k) with binary64 accumulation; FP8 results are scaled back by
// 2^-(eA + eB) on the device.
template <class Ops>
static int protected_product_lowp(const abft_problem *p, const Geom &g, const typename Ops::E *A,
                                  const typename Ops::E *Bt, float *C, const float *Acs, const float *Bcs,
                                  const int *scale_exp, bool plain, hipStream_t s, EpiArgs *e = nullptr,
                                  TagStore *tag = nullptr) {
    typedef typename Ops::E E;
    int st = gemm_main_lowp<Ops>(A, p->lda, Bt, p->ldb, C, p->ldc, g.m, g.n, g.k, scale_exp, s, e);
    if (st) return st;
    ABFT_LAUNCHED();
    if (plain) return ABFT_OK;
    float *Crow = C + g.m * p->ldc;
    SliverExtra x = sliver_extra(scale_exp, false);
    // corner C_f[m + r, n + c]
    if (g.br * g.bc >= kCornerTiled) {
        auto j = sliver_job<float, float, float>(Bcs, g.k, g.bc, Acs, g.k, kCornerRows, g.k, Crow + g.n, 1, p->ldc);
        j.blocks = (unsigned)std::min<int64_t>((g.bc + 15) / 16, 4096);      // four waves of four columns each
        const unsigned pieces = (unsigned)std::min<int64_t>((g.br + kCornerRows - 1) / kCornerRows, 4096);
        k_corner<<<dim3(j.blocks, pieces), kSliverThreads, 0, s>>>(j, g.br, scale_exp);
    } else {
        x.Yr = Acs; x.Yc = Bcs; x.K = g.k; x.nc = g.bc; x.out = Crow + g.n; x.ldo = p->ldc;
        x.blocks = (unsigned)(g.br * g.bc);
    }
    if (tag) { x.tag = tag->dst; x.key = tag->key(); tag->dst = nullptr; }
    // C_f[m + r, j], j < n, and C_f[i, n + c], i < m
    const auto cols = sliver_job<E, float, float>(A, p->lda, g.m, Bcs, g.k, g.bc, g.k, C + g.n, p->ldc, 1);
    return slivers(sliver_job<E, float, float>(Bt, p->ldb, g.n, Acs, g.k, g.br, g.k, Crow, 1, p->ldc), &cols, x, s);
}

int launch_skinny_f64(const double *A, int64_t lda, const double *Bt, int64_t ldb, double *C, int64_t ldc,
                      int64_t M, int64_t N, int64_t K, hipStream_t s) {
    return slivers(sliver_job<double, double, double>(A, lda, M, Bt, ldb, N, K, C, ldc, 1),
                   (const SliverJob<double, double, double> *)nullptr, sliver_extra(nullptr, false), s);
}

int launch_gemm_f64(const double *A, int64_t lda, const double *Bt, int64_t ldb, double *C, int64_t ldc, int64_t M,
                    int64_t N, int64_t K, hipStream_t s) {
    int st = gemm_main(A, lda, Bt, ldb, C, ldc, M, N, K, s);
    if (st) return st;
    ABFT_LAUNCHED();
    return ABFT_OK;
}

int launch_skinny_f32(const float *A, int64_t lda, const float *Bt, int64_t ldb, float *C, int64_t ldc,
                      int64_t M, int64_t N, int64_t K, hipStream_t s) {
    return slivers(sliver_job<float, float, float>(A, lda, M, Bt, ldb, N, K, C, ldc, 1),
                   (const SliverJob<float, float, float> *)nullptr, sliver_extra(nullptr, false), s);
}

int launch_gemm_f32(const float *A, int64_t lda, const float *Bt, int64_t ldb, float *C, int64_t ldc, int64_t M,
                    int64_t N, int64_t K, hipStream_t s) {
    int st = gemm_main(A, lda, Bt, ldb, C, ldc, M, N, K, s);
    if (st) return st;
    ABFT_LAUNCHED();
    return ABFT_OK;
}

int launch_gemm_panel(const abft_problem *p, const void *A_f, const void *B_f, void *C_f, int64_t k0, int64_t k1,
                      uint32_t flags, hipStream_t s) {
    Geom g = geom_of(p);
    const bool plain = flags & ABFT_PLAIN, acc = flags & ABFT_ACCUMULATE;
    switch (p->dtype) {
    case ABFT_F64:
        return protected_product<double>(p, g, (const double *)A_f, (const double *)B_f, (double *)C_f, plain, s, k0,
                                         k1 - k0, acc);
    case ABFT_F32:
        return protected_product<float>(p, g, (const float *)A_f, (const float *)B_f, (float *)C_f, plain, s, k0,
                                        k1 - k0, acc);
    default:
        return ABFT_E_UNSUPPORTED;
    }
}

// The kernels and tiles launch_gemm runs for p and flags, as text (a
// diagnostic: tests check that every tile is exercised, benchmarks report it).
int describe_gemm(const abft_problem *p, uint32_t flags, char *buf, size_t len) {
    const Geom g = geom_of(p);
    const bool plain = flags & ABFT_PLAIN;
    const bool lowp = p->dtype == ABFT_BF16 || p->dtype == ABFT_FP8_E4M3;
    static const char *const kDt[] = {"f64", "f32", "bf16", "fp8"};
    bool thin_r, thin_c;
    int64_t Mm, Nm;
    MainPick pk;
    const char *kname;
    if (lowp) {
        thin_r = thin_c = !plain;             // every carried block from the workspace checksum rows
        Mm = g.m;
        Nm = g.n;
        pk = pick_main_lowp(p->dtype == ABFT_BF16 ? 2 : 1, Mm, Nm, g.k, flags & ABFT_FUSED);
        kname = pk.direct ? "k_gemm_lowp2" : "k_gemm_lowp";
    } else {
        thin_r = !plain && g.S * g.br <= kSliverMaxB;
        thin_c = !plain && g.S * g.bc <= kSliverMaxB;
        Mm = (plain || thin_r) ? g.m : g.M;
        Nm = (plain || thin_c) ? g.n : g.N;
        pk = p->dtype == ABFT_F64 ? pick_main((const double *)nullptr, Mm, Nm, g.k, flags & ABFT_FUSED)
                                  : pick_main((const float *)nullptr, Mm, Nm, g.k, flags & ABFT_FUSED);
        kname = pk.direct ? "k_gemm_mfma2" : "k_gemm_mfma";
    }
    // the carried blocks' kernels: rows over the N columns (lowp: n), columns over the data rows
    const char *sr = sliver_multirow(g.br, lowp ? g.n : g.N) ? " + k_sliver1 carried rows" : " + k_sliver carried rows";
    const char *sc = sliver_multirow(g.bc, Mm) ? " + k_sliver1 carried columns" : " + k_sliver carried columns";
    const char *co = g.br * g.bc >= kCornerTiled ? " + k_corner corner" : " + k_sliver corner";
    const int n = snprintf(buf, len, "%s %s %dx%d on %lldx%lld k=%lld%s%s%s", kname, kDt[p->dtype], pk.t->bm,
                           pk.t->bn, (long long)Mm, (long long)Nm, (long long)g.k, thin_r ? sr : "",
                           (lowp && !plain) ? co : "", thin_c ? sc : "");
    return (n < 0 || (size_t)n >= len) ? ABFT_E_ARG : ABFT_OK;
}

// Owner tag of the fused partial sums (the stateless stand-in for "the last
// product on this workspace"): a 64-bit mix of the problem, its tile grid and
// C_f, never 0 (0 marks "no valid partials").
static uint64_t mix64(uint64_t h, uint64_t v) {
    h ^= v + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
    h ^= h >> 31;
    h *= 0xBF58476D1CE4E5B9ull;
    return h ^ (h >> 29);
}

uint64_t fused_key(const abft_problem *p, const void *C_f, int64_t *tiles_m, int64_t *tiles_n) {
    const Geom g = geom_of(p);
    const bool lowp = p->dtype == ABFT_BF16 || p->dtype == ABFT_FP8_E4M3;
    // b = 1: the carried row and column are slivers, the main product covers m x n
    const MainPick pk = lowp ? pick_main_lowp(p->dtype == ABFT_BF16 ? 2 : 1, g.m, g.n, g.k, true)
                             : (p->dtype == ABFT_F64 ? pick_main((const double *)nullptr, g.m, g.n, g.k, true)
                                                     : pick_main((const float *)nullptr, g.m, g.n, g.k, true));
    *tiles_m = (g.m + pk.t->bm - 1) / pk.t->bm;
    *tiles_n = (g.n + pk.t->bn - 1) / pk.t->bn;
    uint64_t h = 0x6A09E667F3BCC908ull;
    for (uint64_t v : {(uint64_t)p->dtype, (uint64_t)g.m, (uint64_t)g.n, (uint64_t)g.k, (uint64_t)g.br,
                       (uint64_t)g.bc, (uint64_t)p->ldc, (uint64_t)(uintptr_t)C_f, (uint64_t)*tiles_m,
                       (uint64_t)*tiles_n})
        h = mix64(h, v);
    return h ? h : 1;
}

__global__ void k_store_tag(uint64_t *dst, uint64_t v) { *dst = v; }

static int product_with_extras(const abft_problem *p, const Geom &g, const void *A_f, const void *B_f, void *C_f,
                               bool plain, void *ws, const float *Acs, const float *Bcs, const int *scale,
                               EpiArgs *e, TagStore *tag, hipStream_t s) {
    switch (p->dtype) {
    case ABFT_F64:
        return protected_product<double>(p, g, (const double *)A_f, (const double *)B_f, (double *)C_f, plain, s, 0,
                                         -1, false, e, tag);
    case ABFT_F32:
        return protected_product<float>(p, g, (const float *)A_f, (const float *)B_f, (float *)C_f, plain, s, 0, -1,
                                        false, e, tag);
    case ABFT_BF16:
        return protected_product_lowp<Bf16Ops>(p, g, (const uint16_t *)A_f, (const uint16_t *)B_f, (float *)C_f,
                                               Acs, Bcs, nullptr, plain, s, e, tag);
    case ABFT_FP8_E4M3:
        return protected_product_lowp<Fp8x64Ops>(p, g, (const uint8_t *)A_f, (const uint8_t *)B_f, (float *)C_f,
                                                 Acs, Bcs, scale, plain, s, e, tag);
    default:
        return ABFT_E_UNSUPPORTED;
    }
}

int launch_gemm(const abft_problem *p, const void *A_f, const void *B_f, void *C_f, uint32_t flags, void *ws,
                const abft_fault *fault, hipStream_t s) {
    Geom g = geom_of(p);
    const bool plain = flags & ABFT_PLAIN, fused = flags & ABFT_FUSED;
    // epilogue extras: the test-only accumulator flip and the fused partial sums
    EpiArgs e = epi_none();
    if (fault) {
        e.fi = fault->i; e.fj = fault->j; e.fbit = fault->bit;
    }
    WsLayout L = ws_layout(p);
    if (fused) {
        e.pc = (double *)((char *)ws + L.fused_c);
        e.pr = (double *)((char *)ws + L.fused_r);
        e.ldpc = g.n;
        e.ldpr = g.m;
    }
    const char *wsc = (const char *)ws;
    const bool lowp = p->dtype == ABFT_BF16 || p->dtype == ABFT_FP8_E4M3;
    const float *Acs = (lowp && ws) ? (const float *)(wsc + L.acs) : nullptr;
    const float *Bcs = (lowp && ws) ? (const float *)(wsc + L.bcs) : nullptr;
    const int *scale = (p->dtype == ABFT_FP8_E4M3 && ws) ? (const int *)(wsc + L.scale) : nullptr;
    // ws records who owns the fused partials now: this product (fused) or nobody
    TagStore tag{ws ? (uint64_t *)((char *)ws + L.fused_tag) : nullptr, p, C_f, fused, &e};
    int st = product_with_extras(p, g, A_f, B_f, C_f, plain, ws, Acs, Bcs, scale, (fault || fused) ? &e : nullptr,
                                 ws ? &tag : nullptr, s);
    if (st) return st;
    if (tag.dst) {                                   // no carried blocks' launch stored it
        k_store_tag<<<1, 1, 0, s>>>(tag.dst, tag.key());
        ABFT_LAUNCHED();
    }
    return ABFT_OK;
}

}  // namespace abft
