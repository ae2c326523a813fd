// Encode (checksum rows/columns + threshold statistics) and verify (relation
// residuals, thresholds, flags) for gfx950.  Both are HBM-bound row-group
// sums: every element is read once per pass, lanes walk contiguous columns,
// sums are binary64, and the per-block maxima/counts are folded with
// wavefront shuffles before one atomic per block.
#include <cmath>
#include <type_traits>

#include "common.h"

namespace abft {

constexpr int kThreads = 256;
constexpr int kWave = 64;

// ------------------------------------------------------------------ block reductions
__device__ inline double wave_max(double v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
    return v;
}
__device__ inline unsigned long long wave_sum_u64(unsigned long long v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}
__device__ inline double wave_sum(double v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Fold one value per thread into the report: max ratio and excluded count.
__device__ inline void fold_block(double ratio, unsigned long long excl, double *rep_ratio, int64_t *rep_excl) {
    __shared__ double s_r[kThreads / kWave];
    __shared__ unsigned long long s_e[kThreads / kWave];
    ratio = wave_max(ratio);
    excl = wave_sum_u64(excl);
    int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    if (lane == 0) { s_r[w] = ratio; s_e[w] = excl; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = s_r[0];
        unsigned long long e = s_e[0];
        for (int q = 1; q < kThreads / kWave; ++q) { r = fmax(r, s_r[q]); e += s_e[q]; }
        if (r > 0) {
            // ordering of non-negative doubles = ordering of their bits; the maximum only grows, so a block
            // that cannot raise it leaves it alone (thousands of blocks' atomics on one address took 40 us).
            // Not so where blocks count exclusions: a look at the maximum then waits behind their additions to
            // the same line, which an unconditional maximum does not (binary64 8192^2, blocks of 1024, one of
            // them known lost: 224 us with the look, 179 without; nothing lost 130 and 135)
            unsigned long long bits;
            __builtin_memcpy(&bits, &r, 8);
            unsigned long long *dst = (unsigned long long *)rep_ratio;
            if (e || bits > __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(dst, bits);
        }
        if (e) atomicAdd((unsigned long long *)rep_excl, e);
    }
}

// Record a relation residual; returns the ratio |d|/tau for the block maximum (0 if not finite).
__device__ inline double record(abft_report *rep, bool col, int64_t a, int64_t b, double d, double tau) {
    if (!(fabs(d) <= tau)) {
        unsigned long long *cnt = (unsigned long long *)(col ? &rep->n_flag_c : &rep->n_flag_r);
        unsigned long long q = atomicAdd(cnt, 1ull);
        if (q < ABFT_MAX_FLAGS) {
            abft_flag *f = col ? &rep->flag_c[q] : &rep->flag_r[q];
            f->a = a; f->b = b; f->d = d; f->tau = tau;
        }
        if (!isfinite(d)) atomicAdd((unsigned long long *)&rep->n_nonfinite, 1ull);
    }
    if (isfinite(d) && tau > 0) return fabs(d) / tau;
    return 0.0;
}

__device__ inline void clear_report(abft_report *rep) {
    uint64_t *w = (uint64_t *)rep;
    const int nw = sizeof(abft_report) / 8;
    for (int q = threadIdx.x; q < nw; q += blockDim.x) w[q] = 0;
}
__global__ void k_report_init(abft_report *rep) { clear_report(rep); }

// Report of a fused verification: cleared, with status ABFT_E_STALE when the
// owner tag in ws does not name this problem and C_f (the verify kernels then
// record nothing).
__global__ void k_report_init_tag(abft_report *rep, const uint64_t *tag, uint64_t key) {
    clear_report(rep);
    __syncthreads();
    if (threadIdx.x == 0 && *tag != key) rep->status = ABFT_E_STALE;
}

// ------------------------------------------------------------------ encode
// Checksum rows of an operand X (R data rows, row-major, ld; the B operand is
// passed as its transpose, so both sides are the same row-group sum):
//   CS[r, l] = sum_{g<G} X[g*b + r, l]       (binary64 sum, rounded once to TC)
// and the per-residue statistic grp[r, l] of the threshold:
//   det:  sum_g |X[g*b + r, l]|               (row r of C_C^T |X|)
//   stat: sum_g X[g*b + r, l]^2 + CS[r, l]^2  (the squares of every member of the relation)
template <typename TC> __device__ inline void finish_encode(double sv, double ssv, bool stat, TC *cs, double *grp) {
    TC c = (TC)sv;
    *cs = c;
    *grp = stat ? ssv + (double)c * (double)c : ssv;
}

// Per-row statistics of the thresholds:
//   ROW_L2:  ||x||_2              ROW_W: sum_l x_l^2 w_l          ROW_L4SQ: ||x||_4^2
enum { ROW_L2 = 0, ROW_W = 1, ROW_L4SQ = 2 };
__device__ inline double row_term(int mode, double x, double w) {
    const double x2 = x * x;
    return mode == ROW_W ? x2 * w : (mode == ROW_L4SQ ? x2 * x2 : x2);
}

static bool operands_stream(const abft_problem *p) {
    return streams((p->m + p->n) * p->k * (int64_t)dtype_size(p->dtype));
}

// Where the encode pass takes an operand's values from: the stored operand,
// or binary32 values quantized to bfloat16 on the way (round to nearest even),
// which are written to the operand's storage and used as stored.  fetch
// requests the V values X[row, l0 .. l0+V) (raw words, so that several rows
// are in flight), take fills them in as binary64.
template <typename T, bool NT> struct SrcStored {
    static constexpr int V = kEncVec<T>;
    typedef typename std::conditional<V * sizeof(T) == 16, v4u32, uint64_t>::type Raw;
    const T *X;
    int64_t ld;
    __device__ Raw fetch(int64_t row, int64_t l0) const { return load_raw<NT, Raw>(X + row * ld + l0); }
    __device__ void take(const Raw &w, int64_t, int64_t, double *v) const {
        if constexpr (V * sizeof(T) == 16) {
            vec16<T>::widen(w, v);
        } else {
            static_assert(sizeof(T) == 1 && V == 8, "two E4M3 words");
            e4m3x4_to_f64((uint32_t)w, v);
            e4m3x4_to_f64((uint32_t)(w >> 32), v + 4);
        }
    }
};
template <bool NT> struct SrcQuantBf16 {
    static constexpr int V = kEncVec<uint16_t>;
    typedef float v4 __attribute__((ext_vector_type(4)));
    struct Raw { v4 x0, x1; };
    const float *X;
    int64_t ldx;
    uint16_t *Q;
    int64_t ldq;
    __device__ Raw fetch(int64_t row, int64_t l0) const {
        const v4 *x = (const v4 *)(X + row * ldx + l0);
        return Raw{x[0], x[1]};
    }
    __device__ void take(const Raw &w, int64_t row, int64_t l0, double *v) const {
        uint16_t h[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            h[q] = f32_to_bf16_rne(w.x0[q]);
            h[4 + q] = f32_to_bf16_rne(w.x1[q]);
        }
        v4u32 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = (uint32_t)h[2 * q] | ((uint32_t)h[2 * q + 1] << 16);
        if constexpr (NT) __builtin_nontemporal_store(o, (v4u32 *)(Q + row * ldq + l0));
        else *(v4u32 *)(Q + row * ldq + l0) = o;
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = (double)bf16_to_f32(h[q]);
    }
};

// The same to E4M3 under the operand's scale exponent (written by k_scale_exp before the pass).
struct SrcQuantFp8 {
    static constexpr int V = kEncVec<uint8_t>;
    typedef float v4 __attribute__((ext_vector_type(4)));
    struct Raw { v4 x0, x1; };
    const float *X;
    int64_t ldx;
    uint8_t *Q;
    int64_t ldq;
    const int *scale_exp;            // this operand's exponent
    __device__ Raw fetch(int64_t row, int64_t l0) const {
        const v4 *x = (const v4 *)(X + row * ldx + l0);
        return Raw{x[0], x[1]};
    }
    __device__ void take(const Raw &w, int64_t row, int64_t l0, double *v) const {
        const int e = *scale_exp;
        auto sc = [e](float x) { return __builtin_ldexpf(x, e); };
        const uint32_t lo = f32x4_to_e4m3(sc(w.x0[0]), sc(w.x0[1]), sc(w.x0[2]), sc(w.x0[3]));
        const uint32_t hi = f32x4_to_e4m3(sc(w.x1[0]), sc(w.x1[1]), sc(w.x1[2]), sc(w.x1[3]));
        *(uint64_t *)(Q + row * ldq + l0) = (uint64_t)lo | ((uint64_t)hi << 32);
        e4m3x4_to_f64(lo, v);
        e4m3x4_to_f64(hi, v + 4);
    }
};

// One operand in the encode pass.  A block of 256 threads covers a strip of
// CW column vectors (CW = 64 or 16 lanes of V columns) with 256 / CW row
// lanes; how the row lanes and blocks share the groups is EncSplit's choice.
//   rp:  partials of the data rows' statistic, rp[row * strips + strip]
//   rpt: partials of the checksum and group rows' statistics, rpt[row * nt + .],
//        rows 0 .. b-1 the checksum rows, b .. 2b-1 the group rows
template <class Src, typename TC> struct EncSide {
    Src src;
    int64_t b, G, k, strips, P, chunk;
    double *part;
    TC *CS;
    int64_t ldcs;
    double *grp, *rp, *rpt;
    int64_t nt;
    const double *rw;
};
constexpr int kRowNone = -1;     // no fused row statistic
constexpr int kEncRows = 4;      // rows requested together per lane

// Sums of rows g*b + r, g = g0, g0 + step, ... < g1, over the strip's columns
// of one lane (V sums and V group statistics), and the rows' statistic RM
// folded over the CW lanes of the strip: four rows' partials by a
// reduce-scatter (2 + 1 exchanges, then within CW / 4 lanes).  Lanes past the
// last column (ok false) take no loads and add zeros.
template <int CW, class Src, typename TC, bool STAT, int RM>
__device__ __attribute__((always_inline)) inline void enc_rows(const EncSide<Src, TC> &o, int64_t r, int64_t g0,
                                                               int64_t g1, int64_t step, int64_t strip, int c, bool ok,
                                                               int64_t l0, const double *wv, double *s, double *ss) {
    constexpr int V = Src::V, U = kEncRows;
    auto add = [&](const typename Src::Raw &w, int64_t row) {
        double q2 = 0.0;
        if (ok) {
            double v[V];
            o.src.take(w, row, l0, v);
#pragma unroll
            for (int q = 0; q < V; ++q) {
                s[q] += v[q];
                ss[q] += STAT ? v[q] * v[q] : fabs(v[q]);
                if constexpr (RM != kRowNone) q2 += row_term(RM, v[q], wv[q]);
            }
        }
        return q2;
    };
    int64_t g = g0;
    for (; g + (U - 1) * step < g1; g += U * step) {
        typename Src::Raw w[U];
        if (ok) {
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = o.src.fetch((g + u * step) * o.b + r, l0);
        }
        double q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) q[u] = add(w[u], (g + u * step) * o.b + r);
        if constexpr (RM != kRowNone) {
            static_assert(U == 4, "reduce-scatter of four rows");
            const bool hi = c & (CW / 2), lo = c & (CW / 4);
            double k0 = hi ? q[2] : q[0], k1 = hi ? q[3] : q[1];
            k0 += __shfl_xor(hi ? q[0] : q[2], CW / 2);
            k1 += __shfl_xor(hi ? q[1] : q[3], CW / 2);
            double x = lo ? k1 : k0;
            x += __shfl_xor(lo ? k0 : k1, CW / 4);
#pragma unroll
            for (int off = CW / 8; off > 0; off >>= 1) x += __shfl_xor(x, off);
            if (c % (CW / 4) == 0) o.rp[((g + (c / (CW / 4)) * step) * o.b + r) * o.strips + strip] = x;
        }
    }
    for (; g < g1; g += step) {
        typename Src::Raw w;
        if (ok) w = o.src.fetch(g * o.b + r, l0);
        double x = add(w, g * o.b + r);
        if constexpr (RM != kRowNone) {
#pragma unroll
            for (int off = CW / 2; off > 0; off >>= 1) x += __shfl_xor(x, off);
            if (c == 0) o.rp[(g * o.b + r) * o.strips + strip] = x;
        }
    }
}

template <class Src, int RM> __device__ inline void enc_weights(const double *rw, int64_t l0, double *wv) {
#pragma unroll
    for (int q = 0; q < Src::V; ++q) wv[q] = RM == ROW_W ? rw[l0 + q] : 0.0;
}

// Direct: each row lane owns a residue and sums all its groups, so the sums
// are finished here (no partials).  Blocks [0, na) work on x, the rest on y.
template <int CW, class Src, typename TC, bool STAT, int RM>
__global__ __launch_bounds__(kThreads) void k_encode_direct(EncSide<Src, TC> x, EncSide<Src, TC> y, unsigned na) {
    constexpr int V = Src::V, RW = kThreads / CW;
    const EncSide<Src, TC> &o = blockIdx.x < na ? x : y;
    const int64_t idx = blockIdx.x < na ? blockIdx.x : blockIdx.x - na;
    const int64_t strip = idx % o.strips, r = idx / o.strips * RW + threadIdx.x / CW;
    if (r >= o.b) return;
    const int c = threadIdx.x % CW;
    const int64_t kv = o.k / V, cv = strip * CW + c, l0 = min(cv, kv - 1) * V;
    const bool ok = cv < kv;
    double s[V] = {}, ss[V] = {}, wv[V];
    enc_weights<Src, RM>(o.rw, l0, wv);
    enc_rows<CW, Src, TC, STAT, RM>(o, r, 0, o.G, 1, strip, c, ok, l0, wv, s, ss);
    double c2 = 0.0, g2 = 0.0;
    if (ok) {
#pragma unroll
        for (int q = 0; q < V; ++q) {
            finish_encode<TC>(s[q], ss[q], STAT, o.CS + r * o.ldcs + l0 + q, o.grp + r * o.k + l0 + q);
            if constexpr (RM != kRowNone) {
                const double cs = (double)(TC)s[q], gv = STAT ? ss[q] + cs * cs : ss[q];
                c2 += row_term(RM, cs, wv[q]);
                g2 += gv * gv;
            }
        }
    }
    if constexpr (RM != kRowNone) {
#pragma unroll
        for (int off = CW / 2; off > 0; off >>= 1) {
            c2 += __shfl_xor(c2, off);
            g2 += __shfl_xor(g2, off);
        }
        if (c == 0) {
            o.rpt[r * o.nt + strip] = c2;
            o.rpt[(o.b + r) * o.nt + strip] = g2;
        }
    }
}

// Partitioned: a block sums one partition (chunk groups) of one residue, its
// row lanes taking the groups in turn and adding up through LDS in lane order.
// HBM-bound; the block, not the thread, owns a partition, so the partials are
// a small share of the operand (a thread per partition wrote more bytes of
// partials than it read of a 3000 x 2056 bfloat16 operand: both operands of a
// 3000 x 5003 x 2056 product took 36 + 41 us here and 141 + 141 us in the
// finish, now 23 and 5; 16384 x 16384 quantized from binary32: 331 + 39 us,
// now 321 + 11, 5.0 TB/s, the rate of a large copy).
template <int CW, class Src, typename TC, bool STAT, int RM>
__global__ __launch_bounds__(kThreads) void k_encode_partial(EncSide<Src, TC> x, EncSide<Src, TC> y, unsigned na) {
    constexpr int V = Src::V, RW = kThreads / CW;
    __shared__ double sh[RW][CW * V];
    const EncSide<Src, TC> &o = blockIdx.x < na ? x : y;
    const int64_t idx = blockIdx.x < na ? blockIdx.x : blockIdx.x - na;
    const int64_t strip = idx % o.strips, pr = idx / o.strips, r = pr % o.b, p = pr / o.b;
    const int c = threadIdx.x % CW, w = threadIdx.x / CW;
    const int64_t kv = o.k / V, cv = strip * CW + c, l0 = min(cv, kv - 1) * V;
    const int64_t g0 = p * o.chunk, g1 = min(o.G, g0 + o.chunk);
    double s[V] = {}, ss[V] = {}, wv[V];
    enc_weights<Src, RM>(o.rw, l0, wv);
    enc_rows<CW, Src, TC, STAT, RM>(o, r, g0 + w, g1, RW, strip, c, cv < kv, l0, wv, s, ss);
    const int64_t rel = o.b * o.k;
    double *out = o.part + 2 * p * rel + r * o.k + strip * CW * V;
    auto combine = [&](const double *v, double *dst) {
#pragma unroll
        for (int q = 0; q < V; ++q) sh[w][q * CW + c] = v[q];
        __syncthreads();
        for (int t = threadIdx.x; t < CW * V; t += kThreads) {
            double a = 0.0;
#pragma unroll
            for (int u = 0; u < RW; ++u) a += sh[u][(t % V) * CW + t / V];
            if (strip * CW * V + t < o.k) dst[t] = a;
        }
        __syncthreads();
    };
    combine(s, out);
    combine(ss, out + rel);
}

// Finish of the partitioned sums: a block takes 64 columns of one residue, its
// four waves every fourth partition (four running sums each, eight loads in
// flight), added through LDS in a fixed order.
template <typename TC> struct FinSide {
    int64_t b, k, P;
    const double *part;
    TC *CS;
    int64_t ldcs;
    double *grp, *rpt;               // rpt null: no fused row statistics
    int64_t nt;
    int rmode;
    const double *rw;
};
template <typename TC>
__global__ __launch_bounds__(kThreads) void k_encode_finish(FinSide<TC> x, FinSide<TC> y, unsigned na, bool stat) {
    constexpr int NW = kThreads / kWave;
    __shared__ double sh[2][NW][kWave];
    const FinSide<TC> &o = blockIdx.x < na ? x : y;
    const int64_t idx = blockIdx.x < na ? blockIdx.x : blockIdx.x - na;
    const int64_t cbs = (o.k + kWave - 1) / kWave, cb = idx % cbs, r = idx / cbs;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t l = cb * kWave + lane, rel = o.b * o.k;
    const bool ok = l < o.k;
    double s4[4] = {}, ss4[4] = {};
    if (ok) {
        const double *src = o.part + r * o.k + l;
        int64_t p = w;
        for (; p + 3 * NW < o.P; p += 4 * NW) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s4[q] += src[2 * (p + q * NW) * rel];
                ss4[q] += src[(2 * (p + q * NW) + 1) * rel];
            }
        }
        for (int q = 0; p < o.P; p += NW, ++q) {
            s4[q] += src[2 * p * rel];
            ss4[q] += src[(2 * p + 1) * rel];
        }
    }
    sh[0][w][lane] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    sh[1][w][lane] = (ss4[0] + ss4[1]) + (ss4[2] + ss4[3]);
    __syncthreads();
    if (w) return;
    const double sv = (sh[0][0][lane] + sh[0][1][lane]) + (sh[0][2][lane] + sh[0][3][lane]);
    const double ssv = (sh[1][0][lane] + sh[1][1][lane]) + (sh[1][2][lane] + sh[1][3][lane]);
    if (ok) finish_encode<TC>(sv, ssv, stat, o.CS + r * o.ldcs + l, o.grp + r * o.k + l);
    if (o.rpt) {
        const double cs = (double)(TC)sv, gv = stat ? ssv + cs * cs : ssv;
        const double c2 = wave_sum(ok ? row_term(o.rmode, cs, o.rmode == ROW_W ? o.rw[l] : 0.0) : 0.0);
        const double g2 = wave_sum(ok ? gv * gv : 0.0);
        if (lane == 0) {
            o.rpt[r * o.nt + cb] = c2;
            o.rpt[(o.b + r) * o.nt + cb] = g2;
        }
    }
}

constexpr int kRowThreads = 512;       // 8 waves
// Per-row statistic of X[i, 0:k), one wave per row (grid-stride over rows),
// 16-byte loads, eight in flight per lane, kept as raw words until each is
// widened and summed in column order (the statistics are listed above the
// encode kernels).
template <typename T, int MODE, bool NT>
__device__ __attribute__((always_inline)) inline void row_stats_rows(const T *X, int64_t ld, int64_t rows, int64_t k,
                                                                     double *out, int64_t blk, int64_t nblk) {
    static_assert(MODE != ROW_W, "weighted rows: row_w_rows");
    constexpr int V = vec16<T>::N;
    constexpr int NW = kRowThreads / kWave;
    constexpr int64_t step = (int64_t)kWave * V;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    auto term = [&](const double *v, double &acc) {
#pragma unroll
        for (int q = 0; q < V; ++q) acc += row_term(MODE, v[q], 0.0);
    };
    for (int64_t i = blk * NW + wave; i < rows; i += nblk * NW) {
        const T *row = X + i * ld;
        double acc = 0.0;
        int64_t l0 = (int64_t)lane * V;
        for (; l0 + 7 * step < k; l0 += 8 * step) {
            v4u32 raw[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) raw[u] = load_raw<NT, v4u32>(row + l0 + u * step);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                double v[V];
                vec16<T>::widen(raw[u], v);
                term(v, acc);
            }
        }
        for (; l0 < k; l0 += step) {
            double v0[V];
            vec16<T>::load(row + l0, v0);
            term(v0, acc);
        }
        acc = wave_sum(acc);
        if (lane == 0) out[i] = sqrt(acc);
    }
}

// ROW_W, sum_l x_l^2 w_l: the weights stay binary64 -- they are sums of squares,
// which leave binary32's range for operands of 2^64 and beyond, or 2^-75 and
// below.  A block stages kWSlab of them in LDS at a time (32 KB; any k),
// permuted so that the lanes of a wave read consecutive words: lane L needs
// w[l0 + q] with l0 = 64 V c + V L (chunk c of 64 V columns), stored at
// 64 V c + 64 q + L.  One slab that holds all of k is staged once for all of the
// block's rows; otherwise the next slab's words are requested a slab ahead.  A
// wave takes R rows together and U chunks at a time, the next ones requested
// before these are summed; per row the terms are added in column order per lane,
// then by the butterfly.  HBM-bound; the weights' reads of LDS are shared by the
// R rows.  Whole encodes (us, binary32 weights of all of k in LDS and a row per
// wave against this): bfloat16 16384 x 16384 twice 335 and 331, FP8 8192 x 8192
// twice 100 and 95, binary32 8192 and 4096 x 16384 265 and 255, bfloat16 3000
// and 5003 x 2056 29.6 and 28.5; 300 and 300 x 16384, four slabs in turn for
// few rows, 31.5 and 34.3.
constexpr int kWSlab = 4096;
// Rows per wave: four where they still give every CU two blocks, else two
// (11077 and 2631 x 5456 binary32: 128 us with four, 123 with two; 16384 x 1000
// and 2000 62 with two, 59 with four).
constexpr int kRowWRows = 4, kRowWFewRows = 2;
__host__ __device__ inline bool row_w_multi(int64_t rows) { return rows >= 16384; }
template <typename T, int R, int U, bool NT>
__device__ __attribute__((always_inline)) inline void row_w_rows(const T *X, int64_t ld, int64_t rows, int64_t k,
                                                                 const double *w, double *wsh, double *out, int64_t blk,
                                                                 int64_t nblk) {
    constexpr int V = vec16<T>::N;
    constexpr int NW = kRowThreads / kWave;
    constexpr int CH = kWave * V, STEP = U * CH;
    static_assert(kWSlab % STEP == 0, "whole steps in a slab");
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // weights of one slab to LDS, each thread's words requested into wn before
    constexpr int WT = kWSlab / kRowThreads;
    double wn[WT];
    auto request_w = [&](int64_t s) {
#pragma unroll
        for (int e = 0; e < WT; ++e) {
            const int64_t l = s + e * kRowThreads + threadIdx.x;
            wn[e] = l < k ? w[l] : 0.0;
        }
    };
    auto stage_w = [&](int64_t s) {
        const int lim = (int)min((k - s + CH - 1) / CH * CH, (int64_t)kWSlab);
#pragma unroll
        for (int e = 0; e < WT; ++e) {
            const int l = e * kRowThreads + threadIdx.x;
            if (l < lim) wsh[l / CH * CH + l % V * kWave + l % CH / V] = wn[e];
        }
    };
    const bool once = k <= kWSlab;                                       // one slab serves every row
    request_w(0);
    if (once) {
        stage_w(0);
        __syncthreads();
    }
    for (int64_t b0 = blk * NW * R; b0 < rows; b0 += nblk * NW * R) {    // every wave: the barriers are the block's
        const int64_t i0 = b0 + wave * R;
        const T *row[R];
        double acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            row[r] = X + min(i0 + r, rows - 1) * ld + lane * V;          // rows past the last re-read it (not stored)
            acc[r] = 0.0;
        }
        auto request = [&](v4u32 (&raw)[U][R], int64_t s) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (s + u * CH + lane * V < k) raw[u][r] = load_raw<NT, v4u32>(row[r] + s + u * CH);
        };
        v4u32 next[U][R];
        request(next, 0);
        for (int64_t s = 0; s < k; s += STEP) {
            v4u32 raw[U][R];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r) raw[u][r] = next[u][r];
            if (s + STEP < k) request(next, s + STEP);
            if (!once && s % kWSlab == 0) {
                __syncthreads();                                         // every wave is done with the last slab
                stage_w(s);
                request_w(s + kWSlab < k ? s + kWSlab : 0);              // the next, or the next rows' first
                __syncthreads();
            }
            const double *ws = wsh + s % kWSlab + lane;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s + u * CH + lane * V >= k) break;
                constexpr int P = vec16<T>::P;
#pragma unroll
                for (int p = 0; p < V / P; ++p) {
                    double wq[P];
#pragma unroll
                    for (int q = 0; q < P; ++q) wq[q] = ws[u * CH + (p * P + q) * kWave];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        double v[P];
                        vec16<T>::widen_part(raw[u][r], p, v);
#pragma unroll
                        for (int q = 0; q < P; ++q) acc[r] += row_term(ROW_W, v[q], wq[q]);
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc[r] = wave_sum(acc[r]);
            if (lane == 0 && i0 + r < rows) out[i0 + r] = acc[r];
        }
    }
}

// Everything an encode still owes once the sums are finished, in one launch:
// a list of jobs, each with its own run of blocks.
//   JOB_ROWS: statistic `mode` of `rows` rows of X (k columns of T), a wave per row
//   JOB_TAIL_C / JOB_TAIL_D: the same of checksum rows (TC) / group rows
//     (double), a block per row: they are few and long
//   JOB_SUM: rows' statistics from their partials X[row * ld + 0 .. k), eight lanes per row
//   JOB_ZERO: out[0 .. rows) = 0
enum { JOB_ROWS, JOB_TAIL_C, JOB_TAIL_D, JOB_SUM, JOB_ZERO };
struct EncJob {
    int kind, mode;
    unsigned blocks;
    const void *X;
    int64_t ld, rows, k;
    const double *w;
    double *out;
};
constexpr int kMaxJobs = 8;
struct EncJobs {
    int n;
    EncJob j[kMaxJobs];
};

template <typename T>
__device__ inline void tail_row(const EncJob &o, int64_t i) {
    __shared__ double sh[kRowThreads / kWave];
    constexpr int V = vec16<T>::N;
    const T *row = (const T *)o.X + i * o.ld;
    double acc = 0.0;
    for (int64_t l = (int64_t)threadIdx.x * V; l < o.k; l += kRowThreads * V) {
        double v[V];
        vec16<T>::load(row + l, v);
#pragma unroll
        for (int q = 0; q < V; ++q) acc += row_term(o.mode, v[q], o.mode == ROW_W ? o.w[l + q] : 0.0);
    }
    acc = wave_sum(acc);
    if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kRowThreads / kWave; ++q) acc += sh[q];
        o.out[i] = o.mode == ROW_W ? acc : sqrt(acc);
    }
}

template <typename T, typename TC, bool NT>
__global__ __launch_bounds__(kRowThreads, 4) void k_encode_jobs(EncJobs jobs) {
    extern __shared__ double wsh[];                    // a ROW_W job's weights: kWSlab, or k if less
    int64_t blk = blockIdx.x;
    int q = 0;
    while (q + 1 < jobs.n && blk >= jobs.j[q].blocks) blk -= jobs.j[q++].blocks;
    const EncJob &o = jobs.j[q];
    switch (o.kind) {
    case JOB_ROWS: {
        const T *X = (const T *)o.X;
        if (o.mode == ROW_W) {
            // four loads and the next four in flight per lane either way
            if (row_w_multi(o.rows)) row_w_rows<T, kRowWRows, 1, NT>(X, o.ld, o.rows, o.k, o.w, wsh, o.out, blk, o.blocks);
            else row_w_rows<T, kRowWFewRows, 2, NT>(X, o.ld, o.rows, o.k, o.w, wsh, o.out, blk, o.blocks);
        } else if (o.mode == ROW_L4SQ) {
            row_stats_rows<T, ROW_L4SQ, NT>(X, o.ld, o.rows, o.k, o.out, blk, o.blocks);
        } else {
            row_stats_rows<T, ROW_L2, NT>(X, o.ld, o.rows, o.k, o.out, blk, o.blocks);
        }
        break;
    }
    case JOB_TAIL_C: tail_row<TC>(o, blk); break;
    case JOB_TAIL_D: tail_row<double>(o, blk); break;
    case JOB_SUM: {
        const int64_t i = blk * (kRowThreads / 8) + threadIdx.x / 8;
        if (i >= o.rows) break;
        const double *x = (const double *)o.X + i * o.ld;
        double acc = 0.0;
        for (int64_t c = threadIdx.x % 8; c < o.k; c += 8) acc += x[c];
        acc += __shfl_xor(acc, 4);
        acc += __shfl_xor(acc, 2);
        acc += __shfl_xor(acc, 1);
        if (threadIdx.x % 8 == 0) o.out[i] = o.mode == ROW_W ? acc : sqrt(acc);
        break;
    }
    default:
        for (int64_t t = blk * kRowThreads + threadIdx.x; t < o.rows; t += (int64_t)o.blocks * kRowThreads) o.out[t] = 0.0;
        break;
    }
}

// The job list of one launch.
struct JobList {
    EncJobs a{};
    size_t lds = 0;
    unsigned blocks = 0;
    void add(int kind, int mode, int64_t nblk, const void *X, int64_t ld, int64_t rows, int64_t k, const double *w,
             double *out) {
        if (rows <= 0) return;
        a.j[a.n++] = EncJob{kind, mode, (unsigned)nblk, X, ld, rows, k, w, out};
        blocks += (unsigned)nblk;
    }
    template <typename T> void rows(const T *X, int64_t ld, int64_t rows, int64_t k, int mode, const double *w,
                                    double *out) {
        constexpr int64_t CH = (int64_t)kWave * vec16<T>::N;   // the permuted weights fill whole chunks
        if (mode == ROW_W) lds = std::max(lds, sizeof(double) * (size_t)std::min<int64_t>((k + CH - 1) / CH * CH, kWSlab));
        const int64_t per_block = kRowThreads / kWave * (mode != ROW_W ? 1 : row_w_multi(rows) ? kRowWRows : kRowWFewRows);
        add(JOB_ROWS, mode, std::min<int64_t>((rows + per_block - 1) / per_block, mode == ROW_W ? 512 : 65536), X, ld, rows, k, w, out);
    }
    void sums(const double *X, int64_t ld, int64_t rows, int64_t n, int mode, double *out) {
        add(JOB_SUM, mode, (rows + kRowThreads / 8 - 1) / (kRowThreads / 8), X, ld, rows, n, nullptr, out);
    }
    void zero(double *out, int64_t n) {
        add(JOB_ZERO, 0, std::min<int64_t>((n + kRowThreads - 1) / kRowThreads, 64), nullptr, 0, n, 0, nullptr, out);
    }
    template <typename T, typename TC> void launch(bool nt, hipStream_t s) {
        if (!blocks) return;
        if (nt) k_encode_jobs<T, TC, true><<<blocks, kRowThreads, lds, s>>>(a);
        else k_encode_jobs<T, TC, false><<<blocks, kRowThreads, lds, s>>>(a);
    }
};

// One side of the encode pass: its split, buffers and statistics.
template <class Src, typename TC> struct EncJobSide {
    EncSide<Src, TC> o;
    EncSplit sp;
    int rmode;
    double *rows_out, *grp_out;      // statistic of the R + b rows, norms of the group rows
    bool fused;                      // row statistics from the pass's partials
    int64_t R;
};
template <class Src, typename TC>
static EncJobSide<Src, TC> enc_side(Src src, int64_t R, int64_t b, int64_t k, TC *CS, int64_t ldcs, double *grp,
                                    double *part, double *rowpart, bool fused, int rmode, const double *rw,
                                    double *rows_out, double *grp_out) {
    EncJobSide<Src, TC> x;
    x.sp = enc_split(R, b, k, Src::V);
    x.R = R;
    x.rmode = rmode;
    x.fused = fused;
    x.rows_out = rows_out;
    x.grp_out = grp_out;
    x.o = EncSide<Src, TC>{src, b, R / b, k, x.sp.strips, x.sp.P, x.sp.chunk, part, CS, ldcs, grp, rowpart,
                           rowpart + R * x.sp.strips, x.sp.tail_slots, rw};
    return x;
}

// The pass over one side (y null) or both in one launch (the same split form
// and statistic), then the finish of the partitioned sums.
template <class Src, typename TC>
static void enc_launch(const EncJobSide<Src, TC> &x, const EncJobSide<Src, TC> *y, bool stat, hipStream_t s) {
    auto pass = [&](auto cw, auto st, auto rm, const EncJobSide<Src, TC> &u, const EncJobSide<Src, TC> *v) {
        constexpr int CW = decltype(cw)::value, RM = decltype(rm)::value;
        constexpr bool ST = decltype(st)::value;
        const EncSide<Src, TC> &vo = v ? v->o : u.o;
        const int64_t nb = v ? v->sp.blocks : 0;
        if (u.sp.direct)
            k_encode_direct<CW, Src, TC, ST, RM><<<(unsigned)(u.sp.blocks + nb), kThreads, 0, s>>>(
                u.o, vo, (unsigned)u.sp.blocks);
        else
            k_encode_partial<CW, Src, TC, ST, RM><<<(unsigned)(u.sp.blocks + nb), kThreads, 0, s>>>(
                u.o, vo, (unsigned)u.sp.blocks);
    };
    auto by_mode = [&](const EncJobSide<Src, TC> &u, const EncJobSide<Src, TC> *v) {
        const int rm = u.fused ? u.rmode : kRowNone;
        auto by_rm = [&](auto cw, auto st) {
            if (rm == kRowNone) pass(cw, st, std::integral_constant<int, kRowNone>{}, u, v);
            else if constexpr (!decltype(st)::value) pass(cw, st, std::integral_constant<int, ROW_L2>{}, u, v);
            else if (rm == ROW_W) pass(cw, st, std::integral_constant<int, ROW_W>{}, u, v);
            else pass(cw, st, std::integral_constant<int, ROW_L4SQ>{}, u, v);
        };
        auto by_stat = [&](auto cw) {
            if (stat) by_rm(cw, std::true_type{});
            else by_rm(cw, std::false_type{});
        };
        if (u.sp.cw == 64) by_stat(std::integral_constant<int, 64>{});
        else by_stat(std::integral_constant<int, 16>{});
    };
    const bool one = y && x.sp.direct == y->sp.direct && x.sp.cw == y->sp.cw && x.fused == y->fused &&
                     (!x.fused || x.rmode == y->rmode);
    by_mode(x, one ? y : nullptr);
    if (y && !one) by_mode(*y, nullptr);
    auto fin = [](const EncJobSide<Src, TC> &u) {
        return FinSide<TC>{u.o.b, u.o.k, u.o.P, u.o.part, u.o.CS, u.o.ldcs, u.o.grp, u.fused ? u.o.rpt : nullptr,
                           u.o.nt, u.rmode, u.o.rw};
    };
    auto nfin = [](const EncJobSide<Src, TC> *u) {
        return u && !u->sp.direct ? (unsigned)(u->o.b * ((u->o.k + kWave - 1) / kWave)) : 0u;
    };
    const unsigned nx = nfin(&x), ny = nfin(y);
    if (nx + ny) k_encode_finish<TC><<<nx + ny, kThreads, 0, s>>>(fin(x), fin(y ? *y : x), nx, stat);
}

// Row statistics of one side: sums of the pass's partials, or a pass of their
// own over the stored operand and the checksum and group rows.
template <typename T, class Src, typename TC>
static void enc_rows_jobs(JobList &jl, const EncJobSide<Src, TC> &x, const T *X, int64_t ld) {
    const EncSide<Src, TC> &o = x.o;
    if (x.fused) {
        const int64_t nt = x.sp.direct ? x.sp.strips : (o.k + kWave - 1) / kWave;
        jl.sums(o.rp, o.strips, x.R, o.strips, x.rmode, x.rows_out);
        jl.sums(o.rpt, o.nt, o.b, nt, x.rmode, x.rows_out + x.R);
        jl.sums(o.rpt + o.b * o.nt, o.nt, o.b, nt, ROW_L2, x.grp_out);
    } else {
        jl.rows<T>(X, ld, x.R, o.k, x.rmode, o.rw, x.rows_out);
        jl.add(JOB_TAIL_C, x.rmode, o.b, o.CS, o.ldcs, o.b, o.k, o.rw, x.rows_out + x.R);
        jl.add(JOB_TAIL_D, ROW_L2, o.b, o.grp, o.k, o.b, o.k, nullptr, x.grp_out);
    }
}

template <typename T, typename TC, class Src>
static int encode_typed(const abft_problem *p, Src srcA, Src srcB, T *A, T *Bt, TC *Acs, int64_t ldacs, TC *Bcs,
                        int64_t ldbcs, char *ws, hipStream_t s) {
    Geom g = geom_of(p);
    WsLayout L = ws_layout(p);
    double *grpA = (double *)(ws + L.grpA), *grpB = (double *)(ws + L.grpB);
    const bool stat = p->tau_mode == ABFT_TAU_STAT;
    // row statistics (det: na, nb; stat: qr, qc) and the norms of the grp rows
    // (det: na_abs, nb_abs; stat: nv, nw)
    double *ra = (double *)(ws + (stat ? L.qr : L.na)), *rb = (double *)(ws + (stat ? L.qc : L.nb));
    double *ga = (double *)(ws + (stat ? L.nv : L.na_abs)), *gb = (double *)(ws + (stat ? L.nw : L.nb_abs));
    // det: ||row||_2; stat with the other side thin: sum_l row_l^2 w_l (w = the other side's grp); stat
    // otherwise: ||row||_4^2
    const int modeA = !stat ? ROW_L2 : (g.bc == 1 ? ROW_W : ROW_L4SQ);
    const int modeB = !stat ? ROW_L2 : (g.br == 1 ? ROW_W : ROW_L4SQ);
    // The pass produces the row statistics too, unless their weights do not exist yet: A's weights are B's
    // grp and B's are A's.  B's can still be fused by running A's pass first, in launches of their own; that
    // saves reading B again and costs two launches and the overlap of the two passes, so it pays from about
    // kEncRereadBytes of B on (a re-read at 5 TB/s against 10 us).
    const bool serial = modeB == ROW_W && g.n * g.k * (int64_t)sizeof(T) > kEncRereadBytes;
    const bool fuseA = modeA != ROW_W, fuseB = modeB != ROW_W || serial;
    auto a = enc_side<Src, TC>(srcA, g.m, g.br, g.k, Acs, ldacs, grpA, (double *)(ws + L.partial),
                                (double *)(ws + L.rowpart), fuseA, modeA, grpB, ra, ga);
    auto b = enc_side<Src, TC>(srcB, g.n, g.bc, g.k, Bcs, ldbcs, grpB, (double *)(ws + L.partial_b),
                                (double *)(ws + L.rowpart_b), fuseB, modeB, grpA, rb, gb);
    if (serial) {
        enc_launch<Src, TC>(a, nullptr, stat, s);
        enc_launch<Src, TC>(b, nullptr, stat, s);
    } else {
        enc_launch<Src, TC>(a, &b, stat, s);
    }
    JobList jl;
    enc_rows_jobs<T>(jl, a, A, p->lda);
    enc_rows_jobs<T>(jl, b, Bt, p->ldb);
    // an operand encoded here carries no inherited residual
    jl.zero((double *)(ws + L.chain_a), g.br);
    jl.zero((double *)(ws + L.chain_w), g.N);
    jl.launch<T, TC>(operands_stream(p), s);
    ABFT_LAUNCHED();
    return ABFT_OK;
}

// Chained product (the result of a product fed to the next one, F64 or F32,
// det or exact): A_f is the previous C_f, whose carried rows are used as they are.
// Its checksum rows are recomputed only into scratch, for the group statistic;
// the row statistics are taken over the rows that enter the product (the
// carried ones).  B_f is encoded as usual.  The previous column relations hold
// up to their residual, at most tau_prev(r, l) = cc_prev na_abs_prev[r]
// nb_prev[l]; through the product it contributes at most
// sum_l tau_prev(r, l) |B_f[l, j]| to relation (r, j): stored as
// chain_a[r] = cc_prev na_abs_prev[r] and chain_w[j] = sum_l nb_prev[l] |B_f[l, j]|.
__global__ __launch_bounds__(kThreads) void k_chain_a(const double *na_abs_prev, double cc_prev, int64_t br,
                                                      double *chain_a) {
    for (int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x; r < br; r += (int64_t)gridDim.x * kThreads)
        chain_a[r] = cc_prev * na_abs_prev[r];
}

// out[j] = sum_l w[l] |X[j, l]|: one wave per row, binary64.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_row_absdot(const T *X, int64_t ld, int64_t rows, int64_t k,
                                                         const double *w, double *out) {
    constexpr int V = vec16<T>::N;
    const int lane = threadIdx.x % kWave;
    const int64_t w0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gridDim.x * kThreads / kWave;
    for (int64_t j = w0; j < rows; j += nw) {
        const T *row = X + j * ld;
        double acc = 0.0;
        for (int64_t l = V * lane; l < k; l += V * kWave) {
            double v[V];
            vec16<T>::load(row + l, v);
#pragma unroll
            for (int e = 0; e < V; ++e) acc += w[l + e] * fabs(v[e]);
        }
        for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
        if (lane == 0) out[j] = acc;
    }
}

template <typename T>
static int encode_chained_typed(const abft_problem *p, const T *A, T *Bt, char *ws, const abft_problem *prev,
                                const char *ws_prev, double cc_prev, hipStream_t s) {
    Geom g = geom_of(p);
    WsLayout L = ws_layout(p), Lp = ws_layout(prev);
    double *grpA = (double *)(ws + L.grpA), *grpB = (double *)(ws + L.grpB);
    typedef SrcStored<T, false> Src;
    // the A side: group statistic (checksum rows into scratch); the B side as in a plain encode
    auto a = enc_side<Src, T>(Src{A, p->lda}, g.m, g.br, g.k, (T *)(ws + L.chain_cs), g.k, grpA,
                              (double *)(ws + L.partial), (double *)(ws + L.rowpart), false, ROW_L2, nullptr, nullptr,
                              nullptr);
    auto b = enc_side<Src, T>(Src{Bt, p->ldb}, g.n, g.bc, g.k, Bt + g.n * p->ldb, p->ldb, grpB,
                              (double *)(ws + L.partial_b), (double *)(ws + L.rowpart_b), false, ROW_L2, nullptr,
                              nullptr, nullptr);
    enc_launch<Src, T>(a, &b, false, s);
    // row norms of the rows that enter the product (A's carried rows as they are), norms of the group rows
    JobList jl;
    jl.rows<T>(A, p->lda, g.M, g.k, ROW_L2, nullptr, (double *)(ws + L.na));
    jl.rows<T>(Bt, p->ldb, g.N, g.k, ROW_L2, nullptr, (double *)(ws + L.nb));
    jl.add(JOB_TAIL_D, ROW_L2, g.br, grpA, g.k, g.br, g.k, nullptr, (double *)(ws + L.na_abs));
    jl.add(JOB_TAIL_D, ROW_L2, g.bc, grpB, g.k, g.bc, g.k, nullptr, (double *)(ws + L.nb_abs));
    jl.launch<T, T>(operands_stream(p), s);
    // the inherited term
    k_chain_a<<<1, kThreads, 0, s>>>((const double *)(ws_prev + Lp.na_abs), cc_prev, g.br, (double *)(ws + L.chain_a));
    k_row_absdot<T><<<(unsigned)std::min<int64_t>((g.N + 3) / 4, 65536), kThreads, 0, s>>>(
        Bt, p->ldb, g.N, g.k, (const double *)(ws_prev + Lp.nb), (double *)(ws + L.chain_w));
    ABFT_LAUNCHED();
    return ABFT_OK;
}

int launch_encode_chained(const abft_problem *p, const void *A_f, void *B_f, char *ws, const abft_problem *prev,
                          const char *ws_prev, double cc_prev, hipStream_t s) {
    if (p->dtype == ABFT_F32)
        return encode_chained_typed(p, (const float *)A_f, (float *)B_f, ws, prev, ws_prev, cc_prev, s);
    return encode_chained_typed(p, (const double *)A_f, (double *)B_f, ws, prev, ws_prev, cc_prev, s);
}

// Operands already stored as T: checksum rows after the data rows, or (low
// precision: E4M3 in the scaled domain) binary32 checksum rows in the workspace.
template <typename T, typename TC, bool NT>
static int encode_stored(const abft_problem *p, void *A_f, void *B_f, char *ws, hipStream_t s) {
    const Geom g = geom_of(p);
    T *A = (T *)A_f, *Bt = (T *)B_f;
    const SrcStored<T, NT> a{A, p->lda}, b{Bt, p->ldb};
    if constexpr (std::is_same<T, TC>::value) {
        return encode_typed<T, TC>(p, a, b, A, Bt, A + g.m * p->lda, p->lda, Bt + g.n * p->ldb, p->ldb, ws, s);
    } else {
        const WsLayout L = ws_layout(p);
        return encode_typed<T, TC>(p, a, b, A, Bt, (TC *)(ws + L.acs), g.k, (TC *)(ws + L.bcs), g.k, ws, s);
    }
}

int launch_encode(const abft_problem *p, void *A_f, void *B_f, char *ws, hipStream_t s) {
    auto run = [&](auto nt) {
        constexpr bool NT = decltype(nt)::value;
        switch (p->dtype) {
        case ABFT_F64: return encode_stored<double, double, NT>(p, A_f, B_f, ws, s);
        case ABFT_F32: return encode_stored<float, float, NT>(p, A_f, B_f, ws, s);
        case ABFT_BF16: return encode_stored<uint16_t, float, NT>(p, A_f, B_f, ws, s);
        case ABFT_FP8_E4M3: return encode_stored<uint8_t, float, NT>(p, A_f, B_f, ws, s);
        default: return (int)ABFT_E_UNSUPPORTED;
        }
    };
    return operands_stream(p) ? run(std::true_type{}) : run(std::false_type{});
}

static unsigned grid_for(int64_t work) { return (unsigned)std::min<int64_t>((work + kThreads - 1) / kThreads, 65536); }

// ------------------------------------------------------------------ quantize
// binary32 -> bfloat16, round to nearest even; 8 values per thread and step.
__global__ __launch_bounds__(kThreads) void k_quantize_bf16(const float *X, int64_t ldx, int64_t rows, int64_t k,
                                                            uint16_t *Q, int64_t ldq) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    const int64_t per_row = k / 8, total = rows * per_row;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads) {
        int64_t i = t / per_row, c = (t - i * per_row) * 8;
        v4 x0 = *(const v4 *)(X + i * ldx + c), x1 = *(const v4 *)(X + i * ldx + c + 4);
        v4u o;
        o[0] = f32_to_bf16_rne(x0[0]) | ((uint32_t)f32_to_bf16_rne(x0[1]) << 16);
        o[1] = f32_to_bf16_rne(x0[2]) | ((uint32_t)f32_to_bf16_rne(x0[3]) << 16);
        o[2] = f32_to_bf16_rne(x1[0]) | ((uint32_t)f32_to_bf16_rne(x1[1]) << 16);
        o[3] = f32_to_bf16_rne(x1[2]) | ((uint32_t)f32_to_bf16_rne(x1[3]) << 16);
        *(v4u *)(Q + i * ldq + c) = o;
    }
}

// FP8 per-tensor scaling, kept on the device (no host synchronisation):
// amax = max |x| over the finite entries (binary32 bit patterns of
// non-negative values order like unsigned integers), then the scale exponent
// e = the largest e with amax * 2^e <= 448 (0 when amax is 0), then x * 2^e
// (ldexp: exact wherever the result can round to a non-zero code, also where
// 2^e itself is beyond binary32) rounded to E4M3;
// NaN stays NaN and an infinity saturates to +-448 like any |x 2^e| >= 464.
// ws scale words: [0] = e_A, [1] = e_B, [2] = amax_A bits, [3] = amax_B bits.

// 16-byte loads: rows of X are 16-byte aligned and k is a multiple of 4 (as for the quantizer).
// |x| for finite x, else 0 (NaN and infinities take no part in the scale)
__device__ inline float fin_abs(float x) {
    const float a = fabsf(x);
    return a <= 3.40282347e38f ? a : 0.0f;
}

// One or both operands: blocks [0, nx) on x, the rest on y; each block's
// maximum goes to its slot.  A load instruction takes 64 vectors of four columns:
// a piece of one row, or several rows of a short k side by side (one row at a
// time left most lanes idle: 379665 x 48 quantized in 121 us, 31 here); a wave
// takes runs of eight, all in flight, with no division per load (one per element
// vector held the pass at 3.5 TB/s).
struct AmaxSide {
    const float *X;
    int64_t ldx, rows, k;
    float *out;
    int shift;               // log2 of the lanes across a row
    int64_t pieces, total;   // load instructions across a row; in all
};
constexpr int kAmaxRun = 8;
static AmaxSide amax_side(const float *X, int64_t ldx, int64_t rows, int64_t k, float *out) {
    int shift = 0;
    while (shift < 6 && (int64_t(4) << shift) < k) ++shift;
    const int64_t across = int64_t(4) << shift, pieces = (k + across - 1) / across, per = kWave >> shift;
    return AmaxSide{X, ldx, rows, k, out, shift, pieces, (rows + per - 1) / per * pieces};
}
template <bool NT>
__global__ __launch_bounds__(kThreads) void k_amax(AmaxSide x, AmaxSide y, unsigned nx) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    __shared__ float sh[kThreads / kWave];
    const AmaxSide &o = blockIdx.x < nx ? x : y;
    const unsigned blk = blockIdx.x < nx ? blockIdx.x : blockIdx.x - nx, nblk = blockIdx.x < nx ? nx : gridDim.x - nx;
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r = lane >> o.shift, c = (lane & ((1 << o.shift) - 1)) * 4;      // this lane's row and column of a piece
    float mx = 0.0f;
    for (int64_t t = ((int64_t)blk * (kThreads / kWave) + wave) * kAmaxRun; t < o.total;
         t += (int64_t)nblk * (kThreads / kWave) * kAmaxRun) {
        int64_t g = t / o.pieces, p = t - g * o.pieces;                        // row group and piece of the next load
        v4 v[kAmaxRun];
#pragma unroll
        for (int u = 0; u < kAmaxRun; ++u) {
            const int64_t i = (g << (6 - o.shift)) + r, l = (p << (o.shift + 2)) + c;
            v[u] = i < o.rows && l < o.k ? load_raw<NT, v4>(o.X + i * o.ldx + l) : v4{0.f, 0.f, 0.f, 0.f};
            if (++p == o.pieces) { p = 0; ++g; }
        }
#pragma unroll
        for (int u = 0; u < kAmaxRun; ++u)
            mx = fmaxf(mx, fmaxf(fmaxf(fin_abs(v[u][0]), fin_abs(v[u][1])), fmaxf(fin_abs(v[u][2]), fin_abs(v[u][3]))));
    }
    for (int off = kWave / 2; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
    if (lane == 0) sh[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kThreads / kWave; ++q) mx = fmaxf(mx, sh[q]);
        o.out[blk] = mx;
    }
}

// Block b: operand which + b, from its nx (b = 0) or ny block maxima.
__global__ __launch_bounds__(kThreads) void k_scale_exp(const float *amax, int *scale, int which, unsigned nx,
                                                        unsigned ny) {
    __shared__ float sh[kThreads / kWave];
    const int w = which + (int)blockIdx.x;
    const unsigned n = blockIdx.x == 0 ? nx : ny;
    float mx = 0.0f;
    for (unsigned t = threadIdx.x; t < n; t += kThreads) mx = fmaxf(mx, amax[w * kAmaxBlocks + t]);
    for (int off = kWave / 2; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
    if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = mx;
    __syncthreads();
    if (threadIdx.x) return;
    for (int q = 1; q < kThreads / kWave; ++q) mx = fmaxf(mx, sh[q]);
    // mx = f 2^x with 0.5 <= f < 1 and 448 = 0.875 * 2^9
    int e = 0, x = 0;
    if (mx > 0.0f) e = (frexp((double)mx, &x) <= 0.875 ? 9 : 8) - x;
    scale[2 + w] = (int)__float_as_uint(mx);
    scale[w] = e;
}

__global__ __launch_bounds__(kThreads) void k_quantize_fp8(const float *X, int64_t ldx, int64_t rows, int64_t k,
                                                           uint8_t *Q, int64_t ldq, const int *scale, int which) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    const int e = scale[which];
    const int64_t per_row = k / 4, total = rows * per_row;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads) {
        int64_t i = t / per_row, c = (t - i * per_row) * 4;
        v4 x = *(const v4 *)(X + i * ldx + c);
        const uint32_t o = f32x4_to_e4m3(__builtin_ldexpf(x[0], e), __builtin_ldexpf(x[1], e), __builtin_ldexpf(x[2], e),
                                         __builtin_ldexpf(x[3], e));
        *(uint32_t *)(Q + i * ldq + c) = o;
    }
}

// Scale exponents of one operand (which) or of both (Y set, which = 0).
static void scale_exponents(const abft_problem *p, int which, const float *X, int64_t ldx, const float *Y, int64_t ldy,
                            char *ws, hipStream_t s) {
    const WsLayout L = ws_layout(p);
    float *amax = (float *)(ws + L.amax);
    // the quantizing pass reads the operands again: kept in cache where both fit
    const bool nt = streams((p->m + p->n) * p->k * 4);
    auto side = [&](int w, const float *P, int64_t ld) {
        return amax_side(P, ld, w == 0 ? p->m : p->n, p->k, amax + w * kAmaxBlocks);
    };
    auto blocks = [](const AmaxSide &a) {
        constexpr int64_t per = kAmaxRun * (kThreads / kWave);
        return (unsigned)std::min<int64_t>((a.total + per - 1) / per, kAmaxBlocks);
    };
    const AmaxSide x = side(which, X, ldx), y = Y ? side(1, Y, ldy) : x;
    const unsigned nx = blocks(x), ny = Y ? blocks(y) : 0;
    if (nt) k_amax<true><<<nx + ny, kThreads, 0, s>>>(x, y, nx);
    else k_amax<false><<<nx + ny, kThreads, 0, s>>>(x, y, nx);
    k_scale_exp<<<Y ? 2 : 1, kThreads, 0, s>>>(amax, (int *)(ws + L.scale), which, nx, ny);
}

int launch_quantize(const abft_problem *p, int which, const float *X, int64_t ldx, void *dst, char *ws, hipStream_t s) {
    int64_t rows = which == 0 ? p->m : p->n;
    int64_t ldq = which == 0 ? p->lda : p->ldb;
    if (p->dtype == ABFT_BF16) {
        k_quantize_bf16<<<grid_for(rows * p->k / 8), kThreads, 0, s>>>(X, ldx, rows, p->k, (uint16_t *)dst, ldq);
        ABFT_LAUNCHED();
        return ABFT_OK;
    }
    if (p->dtype == ABFT_FP8_E4M3) {
        WsLayout L = ws_layout(p);
        int *scale = (int *)(ws + L.scale);
        scale_exponents(p, which, X, ldx, nullptr, 0, ws, s);
        k_quantize_fp8<<<grid_for(rows * p->k / 4), kThreads, 0, s>>>(X, ldx, rows, p->k, (uint8_t *)dst, ldq, scale,
                                                                      which);
        ABFT_LAUNCHED();
        return ABFT_OK;
    }
    return ABFT_E_UNSUPPORTED;
}

// Quantize both binary32 operands and encode them in the same pass (the values
// abft_quantize would store are written and the encode uses them as stored),
// so the result equals quantize + quantize + encode bit for bit.  FP8 reads
// each operand once before that, for its scale.
int launch_quantize_encode(const abft_problem *p, const float *A32, int64_t lda32, const float *B32, int64_t ldb32,
                           void *A_f, void *B_f, char *ws, hipStream_t s) {
    if (p->dtype == ABFT_BF16) {
        WsLayout L = ws_layout(p);
        uint16_t *A = (uint16_t *)A_f, *Bt = (uint16_t *)B_f;
        auto run = [&](auto nt) {
            typedef SrcQuantBf16<decltype(nt)::value> Src;
            return encode_typed<uint16_t, float>(p, Src{A32, lda32, A, p->lda}, Src{B32, ldb32, Bt, p->ldb}, A, Bt,
                                                 (float *)(ws + L.acs), p->k, (float *)(ws + L.bcs), p->k, ws, s);
        };
        return operands_stream(p) ? run(std::true_type{}) : run(std::false_type{});
    }
    if (p->dtype == ABFT_FP8_E4M3) {
        WsLayout L = ws_layout(p);
        uint8_t *A = (uint8_t *)A_f, *Bt = (uint8_t *)B_f;
        const int *scale = (const int *)(ws + L.scale);
        scale_exponents(p, 0, A32, lda32, B32, ldb32, ws, s);
        return encode_typed<uint8_t, float>(p, SrcQuantFp8{A32, lda32, A, p->lda, scale},
                                            SrcQuantFp8{B32, ldb32, Bt, p->ldb, scale + 1}, A, Bt,
                                            (float *)(ws + L.acs), p->k, (float *)(ws + L.bcs), p->k, ws, s);
    }
    return ABFT_E_UNSUPPORTED;
}

// ------------------------------------------------------------------ verify
struct VerifyArgs {
    int64_t m, n, br, bc, S, Gr, Gc, M, N, ldc;
    int mode;
    double cc, cr;                  // det coefficients; stat: cc = lambda^2 (u^2/3)(T/2 + s)
    double cst;                     // stat: lambda^2 u^2 / 3 (the stored total's binary32 rounding)
    const double *na, *na_abs, *nb, *nb_abs;
    const double *chain_a, *chain_w; // det: inherited term of a chained product (zero otherwise)
    const double *qr, *qc, *nv, *nw;
    const int *scale_exp;           // FP8: statistics are in the scaled domain, C is not
    abft_report *rep;
    Erasures er;
    const uint64_t *tag;            // fused verification: the owner tag the product wrote into ws (null: none)
    uint64_t key;                   // and the value it must hold for this problem and C_f
};

// det:  tau_c = cc ||(C_C^T|A|)[r,:]||_2 ||B_f[:,j]||_2
// stat: tau_c = sqrt(s^2 cc Q_c[r,j] + cst tot^2),  Q_c = qc[j] (br = 1, exact) or nv[r] qc[j]
//       (Cauchy-Schwarz bound), s the FP8 result scale (Q is in the scaled domain), tot the
//       relation's stored total as read from C_f; a non-finite total adds no term (its
//       residual is then non-finite and the relation fails, as it must)
__device__ inline double tau_scale(const VerifyArgs &a) {
    return a.scale_exp ? ldexp(1.0, -(a.scale_exp[0] + a.scale_exp[1])) : 1.0;
}
__device__ inline double tau_col(const VerifyArgs &a, int64_t r, int64_t j, double tot) {
    if (a.mode == ABFT_TAU_DET) return tau_scale(a) * a.cc * a.na_abs[r] * a.nb[j] + a.chain_a[r] * a.chain_w[j];
    if (a.mode == ABFT_TAU_STAT) {
        const double sc = tau_scale(a), t = isfinite(tot) ? tot : 0.0;
        return sqrt(sc * sc * a.cc * (a.br == 1 ? a.qc[j] : a.nv[r] * a.qc[j]) + a.cst * t * t);
    }
    return 0.0;
}
__device__ inline double tau_row(const VerifyArgs &a, int64_t i, int64_t c, double tot) {
    if (a.mode == ABFT_TAU_DET) return tau_scale(a) * a.cr * a.na[i] * a.nb_abs[c];
    if (a.mode == ABFT_TAU_STAT) {
        const double sc = tau_scale(a), t = isfinite(tot) ? tot : 0.0;
        return sqrt(sc * sc * a.cr * (a.bc == 1 ? a.qr[i] : a.qr[i] * a.nw[c]) + a.cst * t * t);
    }
    return 0.0;
}

// Column relation (r, j): sum_{g<Gr} C[g*br + r, j] - sum_{s<S} C[m + s*br + r, j]
template <typename T>
__device__ inline void finish_col(const VerifyArgs &a, const T *C, int64_t r, int64_t j, double s, double &ratio,
                                  unsigned long long &excl) {
    double tot = 0.0;
    for (int64_t q = 0; q < a.S; ++q) tot += elem<T>::load(C + (a.m + q * a.br + r) * a.ldc + j);
    if (col_rel_erased(a.er, r, j, a.br)) { excl++; return; }
    ratio = fmax(ratio, record(a.rep, true, r, j, s - tot, tau_col(a, r, j, tot)));
}

// V consecutive elements of a C row: one 16-byte load (V > 1, aligned rows) or one element.
template <typename T, int V> __device__ inline void load_c(const T *p, double *v) {
    if constexpr (V == 1) v[0] = elem<T>::load(p);
    else vec16<T>::load(p, v);
}

// Column relations, one thread per residue r and V consecutive columns.  With
// V > 1 the rows of C are 16-byte aligned and ldc is a multiple of V, so the
// last vector of a row stays inside the row's ldc elements; columns >= N are
// read but not used.
template <typename T, int V>
__device__ inline void vcol_direct(const VerifyArgs &a, const T *C, int64_t blk, int64_t nblk) {
    const int64_t nv = (a.N + V - 1) / V, total = a.br * nv;
    double ratio = 0.0;
    unsigned long long excl = 0;
    for (int64_t t = blk * kThreads + threadIdx.x; t < total; t += nblk * kThreads) {
        int64_t r = t / nv, j0 = (t - r * nv) * V;
        const T *p = C + r * a.ldc + j0;
        double s[V], v[V];
#pragma unroll
        for (int q = 0; q < V; ++q) s[q] = 0.0;
        const int64_t rs = a.br * a.ldc;
        int64_t g = 0;
        for (; g + 3 < a.Gr; g += 4) {                 // four rows requested together
            double w[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) load_c<T, V>(p + (g + u) * rs, w[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < V; ++q) s[q] += w[u][q];
        }
        for (; g < a.Gr; ++g) {
            load_c<T, V>(p + g * rs, v);
#pragma unroll
            for (int q = 0; q < V; ++q) s[q] += v[q];
        }
#pragma unroll
        for (int q = 0; q < V; ++q)
            if (j0 + q < a.N) finish_col<T>(a, C, r, j0 + q, s[q], ratio, excl);
    }
    fold_block(ratio, excl, &a.rep->max_ratio_c, &a.rep->n_excl_c);
}

// Partitioned: a block sums one partition of one residue over a strip of 64
// vectors, its four waves taking the groups in turn (four rows requested
// together) and adding up through LDS.  The first block also clears the
// report: nothing is recorded before the next launch.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void k_vcol_partial(const T *C, VerifyArgs a, VcolSplit sp, double *part) {
    constexpr int NW = kThreads / kWave;
    __shared__ double sh[NW][kWave * V];
    if (blockIdx.x == 0) clear_report(a.rep);
    const int64_t strip = blockIdx.x % sp.strips, pr = blockIdx.x / sp.strips, r = pr % a.br, p = pr / a.br;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t j0 = (strip * kWave + lane) * V;
    const bool ok = j0 < a.N;
    const int64_t g1 = min(a.Gr, (p + 1) * sp.chunk), rs = a.br * a.ldc;
    const T *src = C + r * a.ldc + (ok ? j0 : 0);
    double s[V] = {}, v[4][V];
    int64_t g = p * sp.chunk + w;
    for (; g + 3 * NW < g1; g += 4 * NW) {
#pragma unroll
        for (int u = 0; u < 4; ++u) load_c<T, V>(src + (g + u * NW) * rs, v[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e) s[e] += v[u][e];
    }
    for (; g < g1; g += NW) {
        load_c<T, V>(src + g * rs, v[0]);
#pragma unroll
        for (int e = 0; e < V; ++e) s[e] += v[0][e];
    }
#pragma unroll
    for (int e = 0; e < V; ++e) sh[w][e * kWave + lane] = s[e];
    __syncthreads();
    for (int t = threadIdx.x; t < kWave * V; t += kThreads) {
        const int64_t j = strip * kWave * V + t;
        const int q = (t % V) * kWave + t / V;
        if (j < a.N) part[p * a.br * a.N + r * a.N + j] = (sh[0][q] + sh[1][q]) + (sh[2][q] + sh[3][q]);
    }
}

// Columns' finish: a block takes 64 columns of one residue, its waves every
// fourth partition.
template <typename T>
__device__ inline void vcol_finish(const VerifyArgs &a, const T *C, int64_t blk, int64_t P, const double *part) {
    __shared__ double sh[kThreads / kWave][kWave];
    const int64_t cbs = (a.N + kWave - 1) / kWave, r = blk / cbs, j = (blk - r * cbs) * kWave + threadIdx.x % kWave;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    double s = 0.0;
    if (j < a.N)
        for (int64_t p = w; p < P; p += kThreads / kWave) s += part[p * a.br * a.N + r * a.N + j];
    sh[w][lane] = s;
    __syncthreads();
    double ratio = 0.0;
    unsigned long long excl = 0;
    if (w == 0 && j < a.N)
        finish_col<T>(a, C, r, j, (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]), ratio, excl);
    fold_block(ratio, excl, &a.rep->max_ratio_c, &a.rep->n_excl_c);
}

// Row relation (i, c): sum_{h<Gc} C[i, h*bc + c] - sum_{s<S} C[i, n + s*bc + c]
__device__ inline void finish_row_total(const VerifyArgs &a, int64_t i, int64_t c, double s, double tot, double &ratio,
                                        unsigned long long &excl) {
    if (row_rel_erased(a.er, i, c, a.bc)) { excl++; return; }
    ratio = fmax(ratio, record(a.rep, false, i, c, s - tot, tau_row(a, i, c, tot)));
}
template <typename T>
__device__ inline void finish_row(const VerifyArgs &a, const T *C, int64_t i, int64_t c, double s, double &ratio,
                                  unsigned long long &excl) {
    double tot = 0.0;
    for (int64_t q = 0; q < a.S; ++q) tot += elem<T>::load(C + i * a.ldc + a.n + q * a.bc + c);
    finish_row_total(a, i, c, s, tot, ratio, excl);
}

// One thread per V row relations of consecutive residues (V > 1: 16-byte rows
// and bc a multiple of V); lanes take consecutive residues (coalesced when
// bc >= 64 V), four loads in flight.  HBM-bound: a load per relation kept the
// lanes waiting (both directions of a 264704 x 1024 binary32 C_f with blocks of
// 256: 860 us with one residue per thread, 555 with four).
template <typename T, int V>
__device__ inline void vrow_strided(const VerifyArgs &a, const T *C, int64_t blk, int64_t nblk) {
    const int64_t cv = a.bc / V, total = a.M * cv;
    double ratio = 0.0;
    unsigned long long excl = 0;
    for (int64_t t = blk * kThreads + threadIdx.x; t < total; t += nblk * kThreads) {
        const int64_t i = t / cv, c = (t - i * cv) * V;
        const T *p = C + i * a.ldc + c;
        double s[V] = {}, tot[V] = {};
        auto sum = [&](double *d, int64_t h, int64_t n) {
            for (; h + 3 < n; h += 4) {
                double w[4][V];
#pragma unroll
                for (int u = 0; u < 4; ++u) load_c<T, V>(p + (h + u) * a.bc, w[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int q = 0; q < V; ++q) d[q] += w[u][q];
            }
            for (; h < n; ++h) {
                double w[V];
                load_c<T, V>(p + h * a.bc, w);
#pragma unroll
                for (int q = 0; q < V; ++q) d[q] += w[q];
            }
        };
        sum(s, 0, a.Gc);
        sum(tot, a.Gc, a.Gc + a.S);                        // the carried columns follow the data columns
#pragma unroll
        for (int q = 0; q < V; ++q) finish_row_total(a, i, c + q, s[q], tot[q], ratio, excl);
    }
    fold_block(ratio, excl, &a.rep->max_ratio_r, &a.rep->n_excl_r);
}

// One block per row for bc < 64 dividing 256, any alignment: thread t sums the
// columns j = t mod 256, all of residue t mod bc; a fixed-order tree then
// combines the 256/bc partial sums of each residue.
template <typename T>
__device__ inline void vrow_block(const VerifyArgs &a, const T *C, int64_t blk, int64_t nblk) {
    __shared__ double sh[kThreads];
    double ratio = 0.0;
    unsigned long long excl = 0;
    for (int64_t i = blk; i < a.M; i += nblk) {
        const T *row = C + i * a.ldc;
        double s0 = 0.0, s1 = 0.0;
        int64_t j = threadIdx.x;
        for (; j + kThreads < a.n; j += 2 * kThreads) {
            s0 += elem<T>::load(row + j);
            s1 += elem<T>::load(row + j + kThreads);
        }
        if (j < a.n) s0 += elem<T>::load(row + j);
        sh[threadIdx.x] = s0 + s1;
        __syncthreads();
        for (int wd = kThreads / 2; wd >= a.bc; wd >>= 1) {
            if (threadIdx.x < wd) sh[threadIdx.x] += sh[threadIdx.x + wd];
            __syncthreads();
        }
        if (threadIdx.x < a.bc) finish_row<T>(a, C, i, threadIdx.x, sh[threadIdx.x], ratio, excl);
        __syncthreads();
    }
    fold_block(ratio, excl, &a.rep->max_ratio_r, &a.rep->n_excl_r);
}

// The same with 16-byte loads (aligned rows): a wave per row, or the block's four
// waves (WR = 4) where few rows are long, four loads in flight per lane.  A
// lane's V columns keep their residues from load to load (64 V is a multiple of
// bc), so it holds V sums, folded at the end within the lane (bc < V) and across
// the lanes that share them; lane c < bc then finishes residue c.
template <typename T, int V, int WR>
__device__ inline void vrow_wave(const VerifyArgs &a, const T *C, int64_t blk, int64_t nblk) {
    constexpr int NW = kThreads / kWave, RB = NW / WR, STEP = WR * kWave * V;       // rows per block; columns per load
    __shared__ double sh[WR > 1 ? NW : 1][kWave];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, bc = (int)a.bc;
    double ratio = 0.0;
    unsigned long long excl = 0;
    for (int64_t i = blk * RB + w / WR; i < a.M; i += nblk * RB) {
        const T *row = C + i * a.ldc;
        double s[V] = {}, v[4][V];
        // a vector that starts before n stays inside its row; its elements at n and beyond are not summed
        auto add = [&](const double (&x)[V], int64_t j) {
#pragma unroll
            for (int q = 0; q < V; ++q) s[q] += j + q < a.n ? x[q] : 0.0;
        };
        int64_t j = (int64_t)(w % WR * kWave + lane) * V;
        for (; j + 3 * STEP < a.n; j += 4 * STEP) {
#pragma unroll
            for (int u = 0; u < 4; ++u) load_c<T, V>(row + j + u * STEP, v[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) add(v[u], j + u * STEP);
        }
        for (; j < a.n; j += STEP) {
            load_c<T, V>(row + j, v[0]);
            add(v[0], j);
        }
        for (int h = V / 2; h >= bc; h >>= 1) {
#pragma unroll
            for (int q = 0; q < V / 2; ++q)
                if (q < h) s[q] += s[q + h < V ? q + h : q];
        }
        const int lanes = bc > V ? bc / V : 1;
        for (int off = kWave / 2; off >= lanes; off >>= 1)
#pragma unroll
            for (int q = 0; q < V; ++q) s[q] += __shfl_xor(s[q], off);
        // lane c takes residue c, sum c % V of lane c / V: the stored totals are read side by side, and failed
        // relations are counted once per wave, not once per sum of a lane
        double mine = 0.0;
#pragma unroll
        for (int q = 0; q < V; ++q) {
            const double t = __shfl(s[q], lane / V);
            if (lane % V == q) mine = t;
        }
        if constexpr (WR > 1) {                            // every wave of the block is on this row
            sh[w][lane] = mine;
            __syncthreads();
            if (w == 0 && lane < bc)
                finish_row<T>(a, C, i, lane, (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]), ratio, excl);
            __syncthreads();
        } else if (lane < bc) {
            finish_row<T>(a, C, i, lane, mine, ratio, excl);
        }
    }
    fold_block(ratio, excl, &a.rep->max_ratio_r, &a.rep->n_excl_r);
}

// Both directions' relations in one launch: blocks [0, nc) the columns (summed
// here, or finished from P partitions' sums), the rest the rows.
enum { ROWS_WAVE, ROWS_WAVES, ROWS_BLOCK, ROWS_VECTORS, ROWS_STRIDED };
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void k_vrelations(const T *C, VerifyArgs a, int64_t P, const double *part,
                                                         unsigned nc, int rows) {
    if (blockIdx.x < nc) {
        if (part) vcol_finish<T>(a, C, blockIdx.x, P, part);
        else vcol_direct<T, V>(a, C, blockIdx.x, nc);
        return;
    }
    const int64_t blk = blockIdx.x - nc, nblk = gridDim.x - nc;
    if (V > 1 && rows == ROWS_WAVE) vrow_wave<T, V, 1>(a, C, blk, nblk);
    else if (V > 1 && rows == ROWS_WAVES) vrow_wave<T, V, 4>(a, C, blk, nblk);
    else if (rows == ROWS_BLOCK) vrow_block<T>(a, C, blk, nblk);
    else if (V > 1 && rows == ROWS_VECTORS) vrow_strided<T, V>(a, C, blk, nblk);
    else vrow_strided<T, 1>(a, C, blk, nblk);
}

// Erasure tests of the one-pass kernel: the residues of each known
// rectangle's first row (mod br) and first column (mod bc) are taken on the
// host, so a test is a few comparisons on kernel arguments (the same answer as
// col_rel_erased / row_rel_erased for 0 <= r < br and 0 <= c < bc).
struct ErasureRes {
    int n;
    int64_t i0[4], j0[4], h[4], w[4], ri[4], cj[4];
};
static ErasureRes erasure_res(const Erasures &e, int64_t br, int64_t bc) {
    ErasureRes x{};
    x.n = e.n;
    for (int q = 0; q < e.n && q < 4; ++q) {
        x.i0[q] = e.i0[q]; x.j0[q] = e.j0[q]; x.h[q] = e.h[q]; x.w[q] = e.w[q];
        x.ri[q] = e.i0[q] % br;
        x.cj[q] = e.j0[q] % bc;
    }
    return x;
}
__device__ inline bool col_erased_res(const ErasureRes &e, int64_t r, int64_t j, int64_t br) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q >= e.n) break;
        if (j < e.j0[q] || j >= e.j0[q] + e.w[q]) continue;
        if (e.h[q] >= br) return true;
        const int64_t off = r >= e.ri[q] ? r - e.ri[q] : r - e.ri[q] + br;
        if (off < e.h[q]) return true;
    }
    return false;
}
__device__ inline bool row_erased_res(const ErasureRes &e, int64_t i, int64_t c, int64_t bc) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q >= e.n) break;
        if (i < e.i0[q] || i >= e.i0[q] + e.h[q]) continue;
        if (e.w[q] >= bc) return true;
        const int64_t off = c >= e.cj[q] ? c - e.cj[q] : c - e.cj[q] + bc;
        if (off < e.w[q]) return true;
    }
    return false;
}

// One pass over C_f for wide checksum blocks: thread t owns residue r and the
// V consecutive residues c0..c0+V-1 and walks the (Gr+1) x (Gc+1) grid of
// blocks (the last block row / column is the carried one), so it holds every
// member of the column relations (r, h*bc + c) and of the row relations
// (g*br + r, c): both directions from one read of C_f.  Sums run over the
// groups in increasing order with the carried term subtracted last, as in the
// two-pass kernels, so the residuals are the same numbers.  GC = Gc, 1..8.
constexpr int kBlockPassMaxG = 8;    // data block columns: up to 8 (the carried one makes 9)
// The thresholds of this pass with their row-, column- and problem-dependent
// factors loaded ahead of the sums (the same arithmetic as tau_row / tau_col).
struct VbFac {
    double sc, rowc, colc;          // tau_scale; per-residue factors of the row (c) and column (r) relations
};
__device__ inline double vb_row_fac(const VerifyArgs &a, int64_t i) {
    return a.mode == ABFT_TAU_DET ? a.na[i] : (a.mode == ABFT_TAU_STAT ? a.qr[i] : 0.0);
}
__device__ inline double vb_tau_row(const VerifyArgs &a, double sc, double fi, double fc, double tot) {
    if (a.mode == ABFT_TAU_DET) return sc * a.cr * fi * fc;
    if (a.mode == ABFT_TAU_STAT) {
        const double t = isfinite(tot) ? tot : 0.0;
        return sqrt(sc * sc * a.cr * (a.bc == 1 ? fi : fi * fc) + a.cst * t * t);
    }
    return 0.0;
}
__device__ inline double vb_tau_col(const VerifyArgs &a, double sc, double fr, double chr, double fj, double cwj,
                                    double tot) {
    if (a.mode == ABFT_TAU_DET) return sc * a.cc * fr * fj + chr * cwj;
    if (a.mode == ABFT_TAU_STAT) {
        const double t = isfinite(tot) ? tot : 0.0;
        return sqrt(sc * sc * a.cc * (a.br == 1 ? fj : fr * fj) + a.cst * t * t);
    }
    return 0.0;
}

template <typename T, int V, int GC>
__global__ __launch_bounds__(kThreads) void k_vblock(const T *C, VerifyArgs a, ErasureRes er) {
    const int64_t cv = a.bc / V, total = a.br * cv;
    const bool det = a.mode == ABFT_TAU_DET, stat = a.mode == ABFT_TAU_STAT;
    const double sc = (det || stat) ? tau_scale(a) : 0.0;
    double ratio_c = 0.0, ratio_r = 0.0;
    unsigned long long excl_c = 0, excl_r = 0;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads) {
        const int64_t r = t / cv, c0 = (t - r * cv) * V;
        // residue factors, loaded once: row relations (i, c0 + q), column relations (r, .)
        double fc[V];
#pragma unroll
        for (int q = 0; q < V; ++q) fc[q] = det ? a.nb_abs[c0 + q] : ((stat && a.bc > 1) ? a.nw[c0 + q] : 0.0);
        const double fr = det ? a.na_abs[r] : ((stat && a.br > 1) ? a.nv[r] : 0.0);
        const double chr = det ? a.chain_a[r] : 0.0;
        double cs[GC + 1][V];
#pragma unroll
        for (int h = 0; h <= GC; ++h)
#pragma unroll
            for (int q = 0; q < V; ++q) cs[h][q] = 0.0;
        // row relations (i, c0 + q): data columns summed, the carried column last
        auto rows_of = [&](int64_t i, double fi, const double (&v)[GC + 1][V]) {
#pragma unroll
            for (int q = 0; q < V; ++q) {
                double rs = 0.0;
#pragma unroll
                for (int h = 0; h < GC; ++h) rs += v[h][q];
                if (er.n && row_erased_res(er, i, c0 + q, a.bc)) excl_r++;
                else ratio_r = fmax(ratio_r, record(a.rep, false, i, c0 + q, rs - v[GC][q],
                                                    vb_tau_row(a, sc, fi, fc[q], v[GC][q])));
            }
        };
        auto add_col = [&](const double (&v)[GC + 1][V]) {
#pragma unroll
            for (int h = 0; h <= GC; ++h)
#pragma unroll
                for (int q = 0; q < V; ++q) cs[h][q] += v[h][q];
        };
        // two rows of blocks at a time: both rows' loads (and their row factors) in flight together
        int64_t g = 0;
        for (; g + 1 < a.Gr; g += 2) {
            const int64_t i0 = g * a.br + r, i1 = i0 + a.br;
            const double f0 = vb_row_fac(a, i0), f1 = vb_row_fac(a, i1);
            double v0[GC + 1][V], v1[GC + 1][V];
#pragma unroll
            for (int h = 0; h <= GC; ++h) {
                load_c<T, V>(C + i0 * a.ldc + h * a.bc + c0, v0[h]);
                load_c<T, V>(C + i1 * a.ldc + h * a.bc + c0, v1[h]);
            }
            rows_of(i0, f0, v0);
            add_col(v0);
            rows_of(i1, f1, v1);
            add_col(v1);
        }
        if (g < a.Gr) {
            const int64_t i0 = g * a.br + r;
            const double f0 = vb_row_fac(a, i0);
            double v0[GC + 1][V];
#pragma unroll
            for (int h = 0; h <= GC; ++h) load_c<T, V>(C + i0 * a.ldc + h * a.bc + c0, v0[h]);
            rows_of(i0, f0, v0);
            add_col(v0);
        }
        // the carried row: its row relations, then the column relations (r, j),
        // data rows summed, the carried row last
        const int64_t i = a.m + r;
        const double fi = vb_row_fac(a, i);
        double fj[GC + 1][V], cw[GC + 1][V], v[GC + 1][V];
#pragma unroll
        for (int h = 0; h <= GC; ++h)
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const int64_t j = h * a.bc + c0 + q;
                fj[h][q] = det ? a.nb[j] : (stat ? a.qc[j] : 0.0);
                cw[h][q] = det ? a.chain_w[j] : 0.0;
            }
#pragma unroll
        for (int h = 0; h <= GC; ++h) load_c<T, V>(C + i * a.ldc + h * a.bc + c0, v[h]);
        rows_of(i, fi, v);
#pragma unroll
        for (int h = 0; h <= GC; ++h)
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const int64_t j = h * a.bc + c0 + q;
                if (er.n && col_erased_res(er, r, j, a.br)) excl_c++;
                else ratio_c = fmax(ratio_c, record(a.rep, true, r, j, cs[h][q] - v[h][q],
                                                    vb_tau_col(a, sc, fr, chr, fj[h][q], cw[h][q], v[h][q])));
            }
    }
    fold_block(ratio_c, excl_c, &a.rep->max_ratio_c, &a.rep->n_excl_c);
    __syncthreads();   // fold_block's shared slots are reused
    fold_block(ratio_r, excl_r, &a.rep->max_ratio_r, &a.rep->n_excl_r);
}
template <int GC>
static void launch_vblock(const double *C, const VerifyArgs &a, const ErasureRes &er, unsigned grid, hipStream_t s) {
    k_vblock<double, 2, GC><<<grid, kThreads, 0, s>>>(C, a, er);
}

// Re-read verification for b = 1 in one pass over C: tile partial sums of the
// data part, column sums of each kPartRows-row tile (pc[tile row][j]) and row
// sums of each 64V-column tile (pr[tile column][i]), the layout the product
// epilogue writes for the fused verification; k_vfused then finishes the
// relations.  A wave takes rows w, w + 4, ... of its tile, four at a time.
constexpr int64_t kPartRows = kVerifyPartRows;
template <typename T, int V, bool NT>
__global__ __launch_bounds__(kThreads) void k_vpartials(const T *C, int64_t ldc, int64_t m, int64_t n, double *pc,
                                                        double *pr, abft_report *rep) {
    constexpr int NW = kThreads / kWave;
    constexpr int64_t TCW = (int64_t)kWave * V;
    __shared__ double sh[NW][TCW];
    if (blockIdx.x == 0) clear_report(rep);            // nothing is recorded before the next launch
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t tiles_n = (n + TCW - 1) / TCW, tiles = ((m + kPartRows - 1) / kPartRows) * tiles_n;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t tm = tile / tiles_n, tn = tile - tm * tiles_n;
        const int64_t i0 = tm * kPartRows, i1 = min(m, i0 + kPartRows), j0 = tn * TCW + lane * V;
        double cs[V] = {};
        // rows of C are 16-byte aligned and ldc is a multiple of V: a vector that starts before n stays
        // inside its row; its elements at n and beyond are not summed
        const bool ok = j0 < n;
        const T *src = C + (ok ? j0 : 0);
        auto add_row = [&](const v4u32 &raw) {
            double v[V], rs = 0.0;
            vec16<T>::widen(raw, v);
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const double x = j0 + q < n ? v[q] : 0.0;
                cs[q] += x;
                rs += x;
            }
            return rs;
        };
        // four rows of the wave at a time, the next four requested before these are summed
        auto request = [&](v4u32 (&raw)[4], int64_t i) {
#pragma unroll
            for (int u = 0; u < 4; ++u) raw[u] = load_raw<NT, v4u32>(src + (i + u * NW) * ldc);
        };
        int64_t i = i0 + w;
        v4u32 next[4];
        if (i + 3 * NW < i1) request(next, i);
        for (; i + 3 * NW < i1; i += 4 * NW) {
            v4u32 raw[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) raw[u] = next[u];
            if (i + 7 * NW < i1) request(next, i + 4 * NW);
            double q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = add_row(raw[u]);
            // the four rows' sums by a reduce-scatter: 2 + 1 exchanges, then within 16 lanes
            const bool hi = lane & 32, lo = lane & 16;
            double k0 = hi ? q[2] : q[0], k1 = hi ? q[3] : q[1];
            k0 += __shfl_xor(hi ? q[0] : q[2], 32);
            k1 += __shfl_xor(hi ? q[1] : q[3], 32);
            double x = lo ? k1 : k0;
            x += __shfl_xor(lo ? k0 : k1, 16);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) x += __shfl_xor(x, o);
            if (lane % 16 == 0) pr[tn * m + i + (lane / 16) * NW] = x;
        }
        for (; i < i1; i += NW) {
            const double x = wave_sum(add_row(load_raw<NT, v4u32>(src + i * ldc)));
            if (lane == 0) pr[tn * m + i] = x;
        }
#pragma unroll
        for (int q = 0; q < V; ++q) sh[w][q * kWave + lane] = cs[q];
        __syncthreads();
        for (int64_t c = threadIdx.x; c < TCW; c += kThreads) {
            const int64_t j = tn * TCW + c, q = (c % V) * kWave + c / V;
            if (j < n) pc[tm * n + j] = (sh[0][q] + sh[1][q]) + (sh[2][q] + sh[3][q]);
        }
        __syncthreads();
    }
}

// Verification from partial sums (b = 1): the column relations of the data
// columns and the row relations of the data rows from tile sums (pc: tiles_m x
// n, pr: tiles_n x m), added in a fixed order -- a block takes 64 relations, its
// four waves every fourth tile; the first two blocks, the longest, sum the carried
// column C_f[0:m, n] and the carried row C_f[m, 0:n] against the corner.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_vfused(const T *C, VerifyArgs a, const double *pc, const double *pr,
                                                     int64_t tiles_m, int64_t tiles_n) {
    if (a.tag && *a.tag != a.key) return;     // partials of another product: nothing is recorded
    constexpr int NW = kThreads / kWave;
    __shared__ double sh[kThreads];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t nbc = (a.n + kWave - 1) / kWave, blk = (int64_t)blockIdx.x - 2;
    double ratio = 0.0;
    unsigned long long excl = 0;
    bool col;
    if (blk >= 0) {
        col = blk < nbc;
        const int64_t len = col ? a.n : a.m, t = (col ? blk : blk - nbc) * kWave + lane;
        const int64_t tiles = col ? tiles_m : tiles_n;
        const double *x = (col ? pc : pr) + t;
        double s4[4] = {};
        if (t < len) {
            int64_t q = w;
            for (; q + 3 * NW < tiles; q += 4 * NW) {
#pragma unroll
                for (int e = 0; e < 4; ++e) s4[e] += x[(q + e * NW) * len];
            }
            for (int e = 0; q < tiles; q += NW, ++e) s4[e] += x[q * len];
        }
        sh[threadIdx.x] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        __syncthreads();
        if (w == 0 && t < len) {
            const double s = (sh[lane] + sh[kWave + lane]) + (sh[2 * kWave + lane] + sh[3 * kWave + lane]);
            if (col) finish_col<T>(a, C, 0, t, s, ratio, excl);
            else finish_row<T>(a, C, t, 0, s, ratio, excl);
        }
    } else {
        col = blk == -2;
        const int64_t len = col ? a.m : a.n;
        // element t of the carried column (row); sixteen loads in flight (the column's are a line each)
        auto at = [&](int64_t t) { return col ? elem<T>::load(C + t * a.ldc + a.n) : elem<T>::load(C + a.m * a.ldc + t); };
        double s8[8] = {};
        int64_t t = threadIdx.x;
        for (; t + 15 * kThreads < len; t += 16 * kThreads) {
            double x[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = at(t + e * kThreads);
#pragma unroll
            for (int e = 0; e < 16; ++e) s8[e % 8] += x[e];
        }
        for (; t + 3 * kThreads < len; t += 4 * kThreads) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s8[e] += at(t + e * kThreads);
        }
        for (; t < len; t += kThreads) s8[0] += at(t);
        sh[threadIdx.x] = ((s8[0] + s8[1]) + (s8[2] + s8[3])) + ((s8[4] + s8[5]) + (s8[6] + s8[7]));
        __syncthreads();
        for (int h = kThreads / 2; h > 0; h >>= 1) {
            if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            if (col) finish_col<T>(a, C, 0, a.n, sh[0], ratio, excl);
            else finish_row<T>(a, C, a.m, 0, sh[0], ratio, excl);
        }
    }
    if (col) fold_block(ratio, excl, &a.rep->max_ratio_c, &a.rep->n_excl_c);
    else fold_block(ratio, excl, &a.rep->max_ratio_r, &a.rep->n_excl_r);
}
template <typename T>
static void launch_vfused(const T *C, const VerifyArgs &a, const double *pc, const double *pr, int64_t tiles_m,
                          int64_t tiles_n, hipStream_t s) {
    const unsigned blocks = (unsigned)((a.n + kWave - 1) / kWave + (a.m + kWave - 1) / kWave + 2);
    k_vfused<T><<<blocks, kThreads, 0, s>>>(C, a, pc, pr, tiles_m, tiles_n);
}

// Whether a problem's relations are verified by k_vblock (wide checksum blocks,
// few of them per row: both directions from one read of C).  Its threads walk
// the block rows two at a time, so with fewer threads it pays while there are few
// block rows: 2304 x 2304 binary64 with 256-blocks 72 us by columns and by rows,
// 21 here; 320 x 320 with 64-blocks 10 in one launch of both, 12 here.
static bool block_pass(const Geom &g, bool f64, bool vec) {
    const int64_t threads = g.br * (g.bc / 2);
    return f64 && vec && g.bc % 2 == 0 && g.bc >= 64 && g.Gc <= kBlockPassMaxG &&
           (threads >= 65536 || (threads >= 16384 && g.Gr <= 16));
}

template <typename T>
static int verify_typed(const abft_problem *p, const T *C, const Erasures &er, const char *ws, const VerifyScratch &sc,
                        hipStream_t s) {
    Geom g = geom_of(p);
    WsLayout L = ws_layout(p);
    TauCoef tc = tau_coef(p);
    VerifyArgs a{};
    a.m = g.m; a.n = g.n; a.br = g.br; a.bc = g.bc; a.S = g.S; a.Gr = g.Gr; a.Gc = g.Gc; a.M = g.M; a.N = g.N;
    a.ldc = p->ldc;
    a.mode = tc.mode; a.cc = tc.cc; a.cr = tc.cr; a.cst = tc.cst;
    a.na = (const double *)(ws + L.na); a.na_abs = (const double *)(ws + L.na_abs);
    a.nb = (const double *)(ws + L.nb); a.nb_abs = (const double *)(ws + L.nb_abs);
    a.chain_a = (const double *)(ws + L.chain_a); a.chain_w = (const double *)(ws + L.chain_w);
    a.qr = (const double *)(ws + L.qr); a.qc = (const double *)(ws + L.qc);
    a.nv = (const double *)(ws + L.nv); a.nw = (const double *)(ws + L.nw);
    a.scale_exp = p->dtype == ABFT_FP8_E4M3 ? (const int *)(ws + L.scale) : nullptr;
    a.rep = sc.rep;
    a.er = er;
    auto blocks = [](int64_t work) { return (unsigned)std::min<int64_t>((work + kThreads - 1) / kThreads, 4096); };
    // 16-byte loads when every row of C starts on a 16-byte boundary
    constexpr int VV = 16 / (int)sizeof(T);
    const bool vec = ((uintptr_t)C % 16 == 0) && (p->ldc % VV == 0);
    // wide checksum blocks with few groups per row: one pass for both directions
    if (block_pass(g, sizeof(T) == 8, vec)) {
        k_report_init<<<1, kThreads, 0, s>>>(a.rep);
        const double *Cd = (const double *)C;
        const ErasureRes ex = erasure_res(er, g.br, g.bc);
        const unsigned grid = blocks(g.br * (g.bc / 2));
        switch (g.Gc) {
        case 1: launch_vblock<1>(Cd, a, ex, grid, s); break;
        case 2: launch_vblock<2>(Cd, a, ex, grid, s); break;
        case 3: launch_vblock<3>(Cd, a, ex, grid, s); break;
        case 4: launch_vblock<4>(Cd, a, ex, grid, s); break;
        case 5: launch_vblock<5>(Cd, a, ex, grid, s); break;
        case 6: launch_vblock<6>(Cd, a, ex, grid, s); break;
        case 7: launch_vblock<7>(Cd, a, ex, grid, s); break;
        default: launch_vblock<8>(Cd, a, ex, grid, s); break;
        }
        ABFT_LAUNCHED();
        return ABFT_OK;
    }
    // b = 1: tile partials in one pass, then the relations from them
    if (g.br == 1 && g.bc == 1 && vec) {
        double *pc = sc.vpart_c, *pr = sc.vpart_r;
        const int64_t tiles_m = (g.m + kPartRows - 1) / kPartRows, tiles_n = (g.n + kWave * VV - 1) / (kWave * VV);
        const unsigned grid = (unsigned)std::min<int64_t>(tiles_m * tiles_n, 8192);
        if (streams(g.m * g.n * (int64_t)sizeof(T)))
            k_vpartials<T, VV, true><<<grid, kThreads, 0, s>>>(C, p->ldc, g.m, g.n, pc, pr, a.rep);
        else
            k_vpartials<T, VV, false><<<grid, kThreads, 0, s>>>(C, p->ldc, g.m, g.n, pc, pr, a.rep);
        launch_vfused<T>(C, a, pc, pr, tiles_m, tiles_n, s);
        ABFT_LAUNCHED();
        return ABFT_OK;
    }
    const VcolSplit sp = vcol_split(g, vec ? VV : 1);
    unsigned nc;
    if (sp.direct) {
        k_report_init<<<1, kThreads, 0, s>>>(a.rep);
        nc = blocks(g.br * (vec ? (g.N + VV - 1) / VV : g.N));
    } else {
        const unsigned grid = (unsigned)(sp.strips * g.br * sp.P);
        if (vec) k_vcol_partial<T, VV><<<grid, kThreads, 0, s>>>(C, a, sp, sc.partial);
        else k_vcol_partial<T, 1><<<grid, kThreads, 0, s>>>(C, a, sp, sc.partial);
        nc = (unsigned)(g.br * ((g.N + kWave - 1) / kWave));
    }
    // the block's waves share a row where a wave per row leaves most of the device idle over rows that take each
    // wave four rounds of its loads and more
    const bool few = g.M <= 1024 && g.n >= 4 * 4 * kWave * VV;
    const int rows = g.bc < 64 && kThreads % g.bc == 0 ? (vec ? (few ? ROWS_WAVES : ROWS_WAVE) : ROWS_BLOCK)
                     : (vec && g.bc % VV == 0 ? ROWS_VECTORS : ROWS_STRIDED);
    const unsigned nr = rows == ROWS_STRIDED || rows == ROWS_VECTORS
                            ? blocks(g.M * (g.bc / (rows == ROWS_VECTORS ? VV : 1)))
                            : (unsigned)std::min<int64_t>(rows == ROWS_WAVE ? (g.M + 3) / 4 : g.M, 4096);
    const double *part = sp.direct ? nullptr : sc.partial;
    if (vec) k_vrelations<T, VV><<<nc + nr, kThreads, 0, s>>>(C, a, sp.P, part, nc, rows);
    else k_vrelations<T, 1><<<nc + nr, kThreads, 0, s>>>(C, a, sp.P, part, nc, rows);
    ABFT_LAUNCHED();
    return ABFT_OK;
}

template <typename T>
static int verify_fused_typed(const abft_problem *p, const T *C, char *ws, int64_t tiles_m, int64_t tiles_n,
                              uint64_t key, hipStream_t s) {
    Geom g = geom_of(p);
    WsLayout L = ws_layout(p);
    TauCoef tc = tau_coef(p);
    VerifyArgs a{};
    a.m = g.m; a.n = g.n; a.br = g.br; a.bc = g.bc; a.S = g.S; a.Gr = g.Gr; a.Gc = g.Gc; a.M = g.M; a.N = g.N;
    a.ldc = p->ldc;
    a.mode = tc.mode; a.cc = tc.cc; a.cr = tc.cr; a.cst = tc.cst;
    a.na = (const double *)(ws + L.na); a.na_abs = (const double *)(ws + L.na_abs);
    a.nb = (const double *)(ws + L.nb); a.nb_abs = (const double *)(ws + L.nb_abs);
    a.chain_a = (const double *)(ws + L.chain_a); a.chain_w = (const double *)(ws + L.chain_w);
    a.qr = (const double *)(ws + L.qr); a.qc = (const double *)(ws + L.qc);
    a.nv = (const double *)(ws + L.nv); a.nw = (const double *)(ws + L.nw);
    a.scale_exp = p->dtype == ABFT_FP8_E4M3 ? (const int *)(ws + L.scale) : nullptr;
    a.rep = (abft_report *)(ws + L.report);
    a.er.n = 0;
    a.tag = (const uint64_t *)(ws + L.fused_tag);
    a.key = key;
    k_report_init_tag<<<1, kThreads, 0, s>>>(a.rep, a.tag, key);
    launch_vfused<T>(C, a, (const double *)(ws + L.fused_c), (const double *)(ws + L.fused_r), tiles_m, tiles_n, s);
    ABFT_LAUNCHED();
    return ABFT_OK;
}

int launch_verify_fused(const abft_problem *p, const void *C_f, char *ws, int64_t tiles_m, int64_t tiles_n,
                        uint64_t key, hipStream_t s) {
    if (p->dtype == ABFT_F64) return verify_fused_typed<double>(p, (const double *)C_f, ws, tiles_m, tiles_n, key, s);
    return verify_fused_typed<float>(p, (const float *)C_f, ws, tiles_m, tiles_n, key, s);
}

int launch_verify(const abft_problem *p, const void *C_f, const Erasures &er, char *ws, hipStream_t s) {
    const WsLayout L = ws_layout(p);
    VerifyScratch sc;
    sc.rep = (abft_report *)(ws + L.report);
    sc.vpart_c = (double *)(ws + L.vpart_c);
    sc.vpart_r = (double *)(ws + L.vpart_r);
    sc.partial = (double *)(ws + L.partial);
    return launch_verify_scratch(p, C_f, er, ws, sc, s);
}

// Bytes of scratch the verification of p on this C_f writes, by the path it
// takes (as verify_typed decides it), laid out from base (256-byte aligned
// parts; base may be null to size only).
size_t verify_scratch_layout(const abft_problem *p, const void *C_f, char *base, VerifyScratch *sc) {
    const Geom g = geom_of(p);
    const bool f64 = p->dtype == ABFT_F64;
    const int64_t VV = f64 ? 2 : 4;
    const bool vec = ((uintptr_t)C_f % 16 == 0) && (p->ldc % VV == 0);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = (off + bytes + 255) & ~(size_t)255; return o; };
    const size_t rep = take(sizeof(abft_report));
    size_t pc = 0, pr = 0, part = 0;
    bool use_pc = false, use_part = false;
    if (!block_pass(g, f64, vec)) {
        if (g.br == 1 && g.bc == 1 && vec) {
            const int64_t tiles_m = (g.m + kPartRows - 1) / kPartRows, tiles_n = (g.n + kWave * VV - 1) / (kWave * VV);
            pc = take(sizeof(double) * tiles_m * g.n);
            pr = take(sizeof(double) * tiles_n * g.m);
            use_pc = true;
        } else {
            const VcolSplit sp = vcol_split(g, vec ? (int)VV : 1);
            if (!sp.direct) {
                part = take(sizeof(double) * sp.P * g.br * g.N);
                use_part = true;
            }
        }
    }
    if (sc) {
        sc->rep = (abft_report *)(base + rep);
        sc->vpart_c = use_pc ? (double *)(base + pc) : nullptr;
        sc->vpart_r = use_pc ? (double *)(base + pr) : nullptr;
        sc->partial = use_part ? (double *)(base + part) : nullptr;
    }
    return off;
}

int launch_verify_scratch(const abft_problem *p, const void *C_f, const Erasures &er, const char *ws,
                          const VerifyScratch &sc, hipStream_t s) {
    if (p->dtype == ABFT_F64) return verify_typed<double>(p, (const double *)C_f, er, ws, sc, s);
    return verify_typed<float>(p, (const float *)C_f, er, ws, sc, s);
}

}  // namespace abft
