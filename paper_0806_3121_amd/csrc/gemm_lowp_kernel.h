// The matrix-core instructions of the low-precision products, with binary32
// accumulation:
//   bfloat16: v_mfma_f32_16x16x32_bf16 (16 x 16 x 32 per instruction)
//   FP8 E4M3 (OCP e4m3fn): v_mfma_scale_f32_32x32x64_f8f6f4
// A is row-major and B column-major (Bt row-major), both k-contiguous.  Each
// lane reads 16-byte chunks of its row; A and B use the same k mapping, so every
// product is formed exactly once.  bfloat16: lane l of a 16-row block holds row
// l % 16 and the 8 values at chunk l / 16 of a 64-byte k group, and accumulator
// value v of lane l is C[4 * (l / 16) + v][l % 16] (measured on gfx950).
#pragma once

#include "gemm_mfma_kernel.h"

namespace abft {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Each Ops feeds one MFMA from CPM 16-byte chunks per lane.
struct Bf16Ops {
    typedef uint16_t E;
    static constexpr int CPM = 1;
    static constexpr int MT = 16;       // output tile of one instruction: MT x MT
    __device__ static void mfma(const v4u &a, const v4u &b, v4f &c) {
        v8bf x, y;
        __builtin_memcpy(&x, &a, 16);
        __builtin_memcpy(&y, &b, 16);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
    }
};

// FP8 E4M3 through v_mfma_scale_f32_32x32x64_f8f6f4 (unit E8M0 scales): a 32 x 32
// output tile over 64 k per instruction.  Lane l holds row (column) l % 32 and
// 32 bytes of k, lanes 32-63 the second half of the 64; accumulator value v of
// lane l is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 (measured on
// gfx950 with integer-valued data, whose products and sums are exact).  The 64
// products of an instruction share its sum's window; against 32-deep groups
// (v_mfma_f32_16x16x32_fp8_fp8) the error to binary64 measured the same, 60 random
// problems each with k from 256 to 16384: root mean square equal to 6 digits for
// uniform and normal data of both signs, within 0.06 % either way for positive data
// and within 0.01 % with 1 % outliers of a hundred times the size.
typedef float v16f __attribute__((ext_vector_type(16)));
struct Fp8x64Ops {
    typedef uint8_t E;
    static constexpr int CPM = 2;
    static constexpr int MT = 32;
    typedef int v8i __attribute__((ext_vector_type(8)));
    __device__ static void mfma(const v8i &a, const v8i &b, v16f &c) {
        c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
    }
};

}  // namespace abft
