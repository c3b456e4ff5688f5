// MX-FP8 conversion shared by the block-scaled kernels.
#pragma once

#include "common.hpp"

namespace espace {

typedef int i32x8_t __attribute__((ext_vector_type(8)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// MX-FP8 code byte of x (already divided by its block scale): clamp to the
// largest E4M3 magnitude, then the hardware's round-to-nearest-even
// conversion (which turns magnitudes past 464 into NaN, hence the clamp).
__device__ __forceinline__ uint32_t mx_pack4(float x0, float x1, float x2, float x3) {
    x0 = fminf(fmaxf(x0, -448.f), 448.f);
    x1 = fminf(fmaxf(x1, -448.f), 448.f);
    x2 = fminf(fmaxf(x2, -448.f), 448.f);
    x3 = fminf(fmaxf(x3, -448.f), 448.f);
    uint32_t r = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x2, x3, (int)r, true);
}

// Scale exponent S of a block with largest magnitude amax: floor(log2 amax)
// - 8 with the byte S + 127 clamped to [0, 254]; byte 0 for a zero block.
__device__ __forceinline__ int mx_scale_byte(float amax) {
    if (!(amax > 0.f)) return 0;
    const int e = __builtin_amdgcn_frexp_expf(amax) - 1;   // floor(log2 amax)
    const int b = e - 8 + 127;
    return b < 0 ? 0 : (b > 254 ? 254 : b);
}

// The order in which a workgroup walks the depth steps: each XCD starts an
// eighth of the whole groups of four steps further on (groups, so that the
// steps that share a scale load stay together; a last partial group keeps its
// place), so that the XCDs read different columns of the operands at a time
// (measured in proj_mxfp8.hip).  A row's sums are added in the order of the XCD its
// tile falls to, so equal rows of one call may differ in the last bits; the same call
// gives the same bits again.
struct MxDepthOrder {
    int whole, rot;
    __device__ __forceinline__ explicit MxDepthOrder(int steps) {
        whole = steps & ~3;
        rot = (int)(blockIdx.x & 7) * (steps >> 2) / 8 * 4;
    }
    __device__ __forceinline__ int operator()(int t) const {
        if (t >= whole) return t;
        const int r = t + rot;
        return r >= whole ? r - whole : r;
    }
};

}  // namespace espace
