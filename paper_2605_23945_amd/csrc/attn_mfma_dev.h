// Matrix-core helpers of the attention kernels whose K and V tiles pass through LDS (attn_prefill.hip, attn_gqa.hip).
#pragma once
#include "pat_dev.h"

namespace pat {

typedef short shortx4_t __attribute__((ext_vector_type(4)));

// four 16-bit elements per lane, transposed among the 16 lanes of a group: element j of lane i is element i % 4 of the
// 8 bytes that lane i / 4 + 4 j addresses
__device__ __forceinline__ uint2 lds_read_tr(const char *p)
{
    typedef __attribute__((address_space(3))) shortx4_t *ptr_t;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr_t)p));
}

// the upper 16 bits of x and of y: two truncated bf16 values, x in the lower half
__device__ __forceinline__ uint32_t upper_halves(float x, float y) { return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u); }

// p = h + m + l exactly, for eight values: truncated to the upper 8 significant bits, the remainder likewise, and what is left
__device__ __forceinline__ void split3_bf16(const float *p, u32x4_t &h, u32x4_t &m, u32x4_t &l)
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float x = p[2 * w], y = p[2 * w + 1];
        const float xr = x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u), yr = y - __uint_as_float(__float_as_uint(y) & 0xFFFF0000u);
        const float xl = xr - __uint_as_float(__float_as_uint(xr) & 0xFFFF0000u), yl = yr - __uint_as_float(__float_as_uint(yr) & 0xFFFF0000u);
        h[w] = upper_halves(x, y); m[w] = upper_halves(xr, yr); l[w] = upper_halves(xl, yl);
    }
}

// eight fp32 values times `scale` as split-bf16 operand fragments
__device__ __forceinline__ void split_fragment(float4 q0, float4 q1, float scale, u32x4_t &hi, u32x4_t &lo)
{
    const float v[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
    uint16_t hh[8], ll[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) split_bf16(v[j] * scale, hh[j], ll[j]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        hi[w] = (uint32_t)hh[2 * w] | ((uint32_t)hh[2 * w + 1] << 16);
        lo[w] = (uint32_t)ll[2 * w] | ((uint32_t)ll[2 * w + 1] << 16);
    }
}

__device__ __forceinline__ floatx4_t mfma_16x16x32(u32x4_t a, u32x4_t b, floatx4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

}  // namespace pat
