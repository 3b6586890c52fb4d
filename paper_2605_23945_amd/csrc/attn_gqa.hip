// Decode attention of 4 or 8 query heads per KV head (grouped queries) over the paged cache.
//
// An item is (sequence, chunk of its keys, KV head), one workgroup.  Its waves take tiles of 32 keys in turn (wave w:
// tiles w, w + W, ...) and never wait for each other while they stream: a wave brings its K and V tiles by asynchronous
// loads into two LDS slots of its own, requesting a slot's K half anew as soon as its fragments are in registers and the
// V half as soon as it is read, and waits by counting its own loads.  Both products run on the matrix cores with a
// head per operand column (columns G .. 15 repeat heads, their results are dropped):
//   S^T[key, head] = K q^T    K rows as the A operand, split-bf16 q as the B operand (registers);
//   O^T[feature, head] += V^T p^T   V read transposed from LDS (ds_read_b64_tr_b16), p from the lane's own scores,
// as in the prefill kernel (attn_prefill.hip): p never crosses lanes and is split into three bf16 terms (no rounding).
// K and V rows lie in LDS with their 16-byte pieces permuted (piece c of key k at c ^ k): K's fragments are read without bank
// conflicts, in V's transposed reads keys k and k ^ 1 share banks (conflict cycles: 6 % of the busy ones at 256 sequences of
// 8192 tokens, where memory bounds the kernel at 5.7 TB/s).
//
// What bounds it: HBM once an item is long (180 sequences of about 2100 tokens, 8 heads on one KV head of 128 features,
// 194 MB: 37.6 us, 5.1 TB/s; 59 us with the scores alone on the matrix cores and p V on the vector ALU), and an item's
// 4 us of dependent loads before and combination after its stream where the batch gives few items (11 sequences of about
// 6000: 11.0 us, before 18.1).  Four waves with two slots of 32 keys each put 128 KiB in flight on a compute unit; two
// waves per workgroup, two workgroups on a compute unit, measured 39.1 and 11.7 us at their best chunk lengths.
#include "attn_mfma_dev.h"
#include "pat_kernels.h"

namespace pat {

namespace {

constexpr int kKeys = 32;       // keys per tile

template <int N>
__device__ __forceinline__ void wait_newer() { asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory"); }     // all but the N newest loads have arrived

// Leading scalar arguments: what the first loads depend on (see gemm_xs_kernel).
template <int D, int G, int W>
__global__ __launch_bounds__(W * 64) void attn_gqa_kernel(const int32_t *meta, const uint16_t *kbase, const uint16_t *vbase, const float *qkv, uint32_t hkv, int ldq, int lgP,
                                                          int C, AttnArgs a)
{
    static_assert(G == 4 || G == 8, "heads per operand column");
    constexpr int KST = D / 32, FT = D / 16, PC = D / 8;       // k-steps of a score, 16-feature tiles, 16-byte pieces per row
    constexpr int KPI = 64 / PC, NI = kKeys / KPI;             // keys per load instruction, load instructions per K (or V) tile
    constexpr int kHalf = kKeys * D * 2;                       // bytes of a K (or V) tile
    constexpr int NQ = G * D / 256;                            // 1-KiB load instructions of the item's query heads
    extern __shared__ __align__(16) char lds[];                // [W][slot 2][K | V] tiles, then the query heads (fp32)
    __shared__ float wml[W][G][2];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g4 = lane >> 4;
    const int P = 1 << lgP;
    const uint32_t ce = blockIdx.x / hkv, h = blockIdx.x - ce * hkv;
    int4 m0 = reinterpret_cast<const int4 *>(meta)[2 * (int64_t)ce];
    int4 m1 = reinterpret_cast<const int4 *>(meta)[2 * (int64_t)ce + 1];
    asm volatile("" : "+s"(m0.x), "+s"(m0.y), "+s"(m0.z), "+s"(m1.x), "+s"(m1.y), "+s"(m1.z), "+s"(m1.w));     // one load, not two in turn
    const int b = __builtin_amdgcn_readfirstlane(m0.x), t0 = __builtin_amdgcn_readfirstlane(m0.y),
              cnt = __builtin_amdgcn_readfirstlane(m0.z);
    const int last = t0 + cnt - 1, tiles = (cnt + kKeys - 1) / kKeys;
    const int n = tiles > wave ? (tiles - wave + W - 1) / W : 0;            // this wave's tiles

    // Lane i holds the page of the wave's i-th half tile (16 keys lie in one page): from the chunk record when it covers
    // the chunk, so that no second dependent look-up precedes the first loads.
    int page;
    {
        const int j = (min(t0 + ((lane >> 1) * W + wave) * kKeys + (lane & 1) * 16, last) >> lgP) - (t0 >> lgP);
        if (C <= 4 * P) page = j == 0 ? m1.x : j == 1 ? m1.y : j == 2 ? m1.z : m1.w;
        else page = a.page_table[(int64_t)(a.row_slot ? a.row_slot[b] : b) * a.max_pages + (t0 >> lgP) + j];
        asm volatile("" : "+v"(page));                         // here, or the compiler waits for all loads at every later use
    }
    const int64_t page_bytes = (int64_t)(hkv << lgP) * D * 2, head_bytes = (int64_t)(h << lgP) * D * 2;
    const char *kpool = reinterpret_cast<const char *>(kbase) + head_bytes, *vpool = reinterpret_cast<const char *>(vbase) + head_bytes;
    char *const ring = lds + wave * 4 * kHalf;
    const uint32_t ring0 = lds_offset(ring), q0 = lds_offset(lds + W * 4 * kHalf);

    // the i-th tile's keys from K or V into their place; keys past the chunk repeat its last one (finite values, weight 0)
    auto request = [&](const char *pool, int i, uint32_t to) {
        const int key0 = t0 + (i * W + wave) * kKeys;
#pragma unroll
        for (int u = 0; u < NI; ++u) {
            const int half = u * KPI / 16, key = u * KPI + lane / PC, src = min(key0 + key, last);
            const uint32_t off = (uint32_t)((src & (P - 1)) * (D * 2)) + (uint32_t)(((lane % PC) ^ (key & (PC - 1))) * 16);
            load_to_lds_stream(pool + __builtin_amdgcn_readlane(page, 2 * i + half) * page_bytes, off, to + u * 1024);
        }
    };
    {
        const char *qp = reinterpret_cast<const char *>(qkv + (int64_t)b * ldq + h * G * D);
#pragma unroll
        for (int i = 0; i < (NQ + W - 1) / W; ++i)
            if (i * W + wave < NQ) load_to_lds(qp, (uint32_t)((i * W + wave) * 1024 + lane * 16), q0 + (uint32_t)((i * W + wave) * 1024));
    }
    if (n > 0) { request(kpool, 0, ring0); request(vpool, 0, ring0 + kHalf); }
    if (n > 1) { request(kpool, 1, ring0 + 2 * kHalf); request(vpool, 1, ring0 + 3 * kHalf); }
    if (n > 1) wait_newer<4 * NI>(); else if (n > 0) wait_newer<2 * NI>(); else wait_newer<0>();
    asm volatile("s_barrier" ::: "memory");                    // the query heads are in LDS

    u32x4_t qh[KST], ql[KST];
    {
        const float scale = rsqrtf((float)D) * 1.44269504f;    // scores in units of log2: p is one exp2 instruction
        const float4 *qr = reinterpret_cast<const float4 *>(lds + W * 4 * kHalf) + ((col % G) * D + g4 * 8) / 4;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) split_fragment(qr[ks * 8], qr[ks * 8 + 1], scale, qh[ks], ql[ks]);
    }
    floatx4_t o[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) o[f] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    float M = -INFINITY, den = 0.f;
    for (int i = 0; i < n; ++i) {
        const int slot = i & 1, key0 = t0 + (i * W + wave) * kKeys;
        const char *kt = ring + slot * 2 * kHalf, *vt = kt + kHalf;
        const uint32_t to = ring0 + slot * 2 * kHalf;
        // newer than this tile's K: its V and the next tile
        if (i + 1 < n) wait_newer<3 * NI>(); else wait_newer<NI>();
        u32x4_t kf[2][KST];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                const int key = j * 16 + col;
                kf[j][ks] = *reinterpret_cast<const u32x4_t *>(kt + (key * PC + ((ks * 4 + g4) ^ (key & (PC - 1)))) * 16);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // read: the place can be requested anew
        if (i + 2 < n) request(kpool, i + 2, to);
        floatx4_t s[2] = {floatx4_t{0.f, 0.f, 0.f, 0.f}, floatx4_t{0.f, 0.f, 0.f, 0.f}};
        floatx4_t sl[2] = {floatx4_t{0.f, 0.f, 0.f, 0.f}, floatx4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {                     // four independent accumulators
#pragma unroll
            for (int j = 0; j < 2; ++j) s[j] = mfma_16x16x32(kf[j][ks], qh[ks], s[j]);
#pragma unroll
            for (int j = 0; j < 2; ++j) sl[j] = mfma_16x16x32(kf[j][ks], ql[ks], sl[j]);
        }
        float p[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) p[j] = s[j >> 2][j & 3] + sl[j >> 2][j & 3];
        if (key0 + kKeys - 1 > last) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (key0 + (j >> 2) * 16 + g4 * 4 + (j & 3) > last) p[j] = -INFINITY;
        }
        float mt = p[0];
#pragma unroll
        for (int j = 1; j < 8; ++j) mt = fmaxf(mt, p[j]);
        mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
        mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
        const float Mn = fmaxf(M, mt);
        if (__any(Mn > M)) {                                   // some head of the wave has a new maximum
            const float corr = M == Mn ? 1.f : __builtin_amdgcn_exp2f(M - Mn);     // exp2(-inf) = 0 on the wave's first keys
            M = Mn;
            den *= corr;
#pragma unroll
            for (int f = 0; f < FT; ++f) { o[f][0] *= corr; o[f][1] *= corr; o[f][2] *= corr; o[f][3] *= corr; }
        }
        const float m0_ = M == -INFINITY ? 0.f : M;            // a head whose scores so far all overflowed to -inf: p = 0
#pragma unroll
        for (int j = 0; j < 8; ++j) { p[j] = __builtin_amdgcn_exp2f(p[j] - m0_); den += p[j]; }
        u32x4_t ph, pm, pl;
        split3_bf16(p, ph, pm, pl);
        // newer than this tile's V: the next tile, and the K half requested above
        if (i + 2 < n) wait_newer<3 * NI>(); else if (i + 1 < n) wait_newer<2 * NI>(); else wait_newer<0>();
        const int ka = g4 * 4 + (col >> 2), kb = ka + 16;      // keys whose pieces this lane addresses
        u32x4_t vf[FT];
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const int piece = f * 2 + ((col & 3) >> 1), half = (col & 1) * 8;
            const uint2 va = lds_read_tr(vt + (ka * PC + (piece ^ (ka & (PC - 1)))) * 16 + half);
            const uint2 vb = lds_read_tr(vt + (kb * PC + (piece ^ (kb & (PC - 1)))) * 16 + half);
            vf[f] = u32x4_t{va.x, va.y, vb.x, vb.y};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + 2 < n) request(vpool, i + 2, to + kHalf);
#pragma unroll
        for (int f = 0; f < FT; ++f) o[f] = mfma_16x16x32(vf[f], ph, o[f]);
#pragma unroll
        for (int f = 0; f < FT; ++f) o[f] = mfma_16x16x32(vf[f], pm, o[f]);
#pragma unroll
        for (int f = 0; f < FT; ++f) o[f] = mfma_16x16x32(vf[f], pl, o[f]);
    }
    den += __shfl_xor(den, 16, 64);
    den += __shfl_xor(den, 32, 64);

    // the waves' states meet in LDS (a wave's tiles are read: its ring is free) and are combined in wave order
    float *red = reinterpret_cast<float *>(ring);
    if (col < G) {
#pragma unroll
        for (int f = 0; f < FT; ++f) *reinterpret_cast<float4 *>(red + col * D + f * 16 + g4 * 4) = make_float4(o[f][0], o[f][1], o[f][2], o[f][3]);
        if (g4 == 0) { wml[wave][col][0] = M; wml[wave][col][1] = den; }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < G * D / 4; e += W * 64) {
        const int g = e / (D / 4);
        float mw[W], Mc = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) { mw[w] = wml[w][g][0]; Mc = fmaxf(Mc, mw[w]); }
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float sw = mw[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[w] - Mc);     // a wave without tiles, or whose scores all are -inf
            const float4 t = reinterpret_cast<const float4 *>(lds + w * 4 * kHalf)[e];
            v.x = fmaf(t.x, sw, v.x); v.y = fmaf(t.y, sw, v.y); v.z = fmaf(t.z, sw, v.z); v.w = fmaf(t.w, sw, v.w);
            l = fmaf(wml[w][g][1], sw, l);
        }
        if (a.direct) {
            // the row's only chunk: four features of the O projection's operand, as the merge of one chunk would write them
            const float inv = 1.0f / l;
            uint16_t hh[4], ll[4];
            split_bf16(v.x * inv, hh[0], ll[0]); split_bf16(v.y * inv, hh[1], ll[1]);
            split_bf16(v.z * inv, hh[2], ll[2]); split_bf16(v.w * inv, hh[3], ll[3]);
            const int64_t off = packed_elem_offset(b, (h * G + g) * D + e % (D / 4) * 4, a.hq * D / 32);
            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.ohi) + off) = make_uint2(hh[0] | (uint32_t)hh[1] << 16, hh[2] | (uint32_t)hh[3] << 16);
            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.olo) + off) = make_uint2(ll[0] | (uint32_t)ll[1] << 16, ll[2] | (uint32_t)ll[3] << 16);
            continue;
        }
        const int64_t row = (int64_t)ce * a.hq + h * G + g;
        reinterpret_cast<float4 *>(a.part_acc + row * D)[e % (D / 4)] = v;
        if (e % (D / 4) == 0) *reinterpret_cast<float2 *>(a.part_ml + row * 2) = make_float2(Mc, l);
    }
}

constexpr int kWaves = 4;
template <int D, int G> constexpr size_t gqa_lds() { return (size_t)kWaves * 4 * kKeys * D * 2 + (size_t)G * D * 4; }

template <int D, int G>
hipError_t launch_gqa(const AttnArgs &a, hipStream_t s)
{
    attn_gqa_kernel<D, G, kWaves><<<a.n_items, kWaves * 64, gqa_lds<D, G>(), s>>>(a.chunk_meta, a.kv.pool + a.kv.base(a.layer, 0), a.kv.pool + a.kv.base(a.layer, 1), a.qkv,
                                                                                  (uint32_t)a.kv.hkv, a.ldq, __builtin_ctz(a.kv.P), a.chunk_tokens, a);
    return hipGetLastError();
}

template <int D, int G>
hipError_t gqa_limit() { return hipFuncSetAttribute((const void *)attn_gqa_kernel<D, G, kWaves>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)gqa_lds<D, G>()); }

}  // namespace

hipError_t attn_gqa_prepare_device()
{
    hipError_t e = gqa_limit<128, 8>();
    if (e == hipSuccess) e = gqa_limit<128, 4>();
    if (e == hipSuccess) e = gqa_limit<64, 8>();
    if (e == hipSuccess) e = gqa_limit<64, 4>();
    return e;
}

hipError_t launch_attn_gqa(const AttnArgs &a, hipStream_t s)
{
    const int G = a.hq / a.kv.hkv;
    { const hipError_t e = gemm_prepare_device(); if (e != hipSuccess) return e; }
    if (a.kv.d == 128) return G == 8 ? launch_gqa<128, 8>(a, s) : launch_gqa<128, 4>(a, s);
    return G == 8 ? launch_gqa<64, 8>(a, s) : launch_gqa<64, 4>(a, s);
}

}  // namespace pat
