// The embedding gather of a small batch, shared by its own kernel and the launch that plans the step beside it.
#pragma once
#include "pat_dev.h"

namespace pat {

constexpr int kEmbedThreads = 256;

// Row b of the embedding as fp32, its sum of squares (one part per row), and the row times the first layer's RMSNorm
// gains as the packed split-bf16 operand of its QKV projection.  Called by kEmbedThreads threads of a workgroup; the sum
// has a fixed order (per thread, per wave by shuffles, the waves in order).
__device__ __forceinline__ void embed_stats_row(const uint16_t *table, int H, const int32_t *tok, const uint16_t *gains, int b, float *x,
                                                float *stats, uint4 *pk_hi, uint4 *pk_lo, float *part)
{
    const uint16_t *row = table + (int64_t)tok[b] * H;
    float ss = 0.f;
    for (int k0 = threadIdx.x * 8; k0 < H; k0 += kEmbedThreads * 8) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row + k0);
        const uint4 gv = *reinterpret_cast<const uint4 *>(gains + k0);
        const float4 p = make_float4(bf16lo(v.x), bf16hi(v.x), bf16lo(v.y), bf16hi(v.y));
        const float4 q = make_float4(bf16lo(v.z), bf16hi(v.z), bf16lo(v.w), bf16hi(v.w));
        float *o = x + (int64_t)b * H + k0;
        *reinterpret_cast<float4 *>(o) = p;
        *reinterpret_cast<float4 *>(o + 4) = q;
        ss += (p.x * p.x + p.y * p.y) + (p.z * p.z + p.w * p.w) + (q.x * q.x + q.y * q.y) + (q.z * q.z + q.w * q.w);
        const float xg[8] = {p.x * bf16lo(gv.x), p.y * bf16hi(gv.x), p.z * bf16lo(gv.y), p.w * bf16hi(gv.y),
                             q.x * bf16lo(gv.z), q.y * bf16hi(gv.z), q.z * bf16lo(gv.w), q.w * bf16hi(gv.w)};
        uint16_t hh[8], ll[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) split_bf16(xg[j], hh[j], ll[j]);
        const int64_t vi = packed_elem_offset(b, k0, H >> 5) >> 3;
        pk_hi[vi] = make_uint4(hh[0] | (uint32_t)hh[1] << 16, hh[2] | (uint32_t)hh[3] << 16, hh[4] | (uint32_t)hh[5] << 16, hh[6] | (uint32_t)hh[7] << 16);
        pk_lo[vi] = make_uint4(ll[0] | (uint32_t)ll[1] << 16, ll[2] | (uint32_t)ll[3] << 16, ll[4] | (uint32_t)ll[5] << 16, ll[6] | (uint32_t)ll[7] << 16);
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) stats[b] = (part[0] + part[1]) + (part[2] + part[3]);
}

}  // namespace pat
