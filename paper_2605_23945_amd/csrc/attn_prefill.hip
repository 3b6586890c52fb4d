// Causal attention of a prefill pass over the paged cache.
//
// An item is (block of 64 / G consecutive positions of ONE sequence, chunk of its keys, KV head): its 64 operand rows
// are the block's positions times the G query heads of the KV head, 16 per wave.  K and V tiles of 64 keys come by
// asynchronous loads straight into LDS, one tile ahead, shared by the four waves; both products run on the matrix
// cores, transposed, so that everything about a row sits in the lanes of its column:
//   S^T[key, row] = K q^T    K rows as the A operand, split-bf16 q as the B operand (registers);
//   O^T[feature, row] += V^T p^T   V read transposed from LDS (ds_read_b64_tr_b16), p from the lane's own scores.
// A lane's scores of two 16-key tiles, keys 4 g .. 4 g + 3 and 16 + 4 g .. (g = lane / 16), are exactly one operand
// fragment when the V fragment takes its keys in the same order, so p never crosses lanes; the running maximum, the
// denominator and the rescaling of O are per-lane values (the maximum over a row's keys needs two shuffles).
// p is split into three bf16 terms (24 bits: no rounding), q into two as everywhere in this path.
// K and V rows are stored with their 16-byte pieces permuted (piece c of key k at c ^ k), which the loads do on their
// way in by permuting the source addresses: without it the 16 rows of a fragment would share their LDS banks.
//
// What bounds it: at long contexts the matrix cores and the vector ALU about equally (per wave and tile 80 products of
// 16 clocks against 16 exponentials and splits per lane); at short ones the latency of an item's first loads.
#include "attn_mfma_dev.h"
#include "pat_kernels.h"

namespace pat {

namespace {

constexpr int kRows = 64;       // operand rows per item
constexpr int kTile = 64;       // keys per tile

// DIRECT: every row has one chunk; the finished output goes to the packed operand of the O projection instead of the
// partial (m, l, acc) of the row's chunk list.
template <int D, int G, bool DIRECT>
__global__ __launch_bounds__(256, 2) void attn_prefill_kernel(const int32_t *meta, const uint16_t *kbase, const uint16_t *vbase, const float *qkv, const int32_t *page_table,
                                                              uint32_t hkv, int ldq, int lgP, int C, int max_pages, AttnArgs a)
{
    static_assert(G == 1 || G == 2 || G == 4 || G == 8, "the 64 operand rows are 64 / G positions x G heads");
    constexpr int KST = D / 32, FT = D / 16, PC = D / 8;       // k-steps of a score, 16-feature tiles, 16-byte pieces per row
    constexpr int KPI = 64 / PC, NI = kTile / KPI / 4;         // keys per load instruction, instructions per wave for one K (or V) tile
    __shared__ u32x4_t kv[2][2][kTile * PC];                   // [buffer][K | V][key][piece, permuted]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g4 = lane >> 4;
    const int P = 1 << lgP;
    const uint32_t ce = blockIdx.x / hkv, h = blockIdx.x - ce * hkv;
    const int4 m0 = reinterpret_cast<const int4 *>(meta)[2 * (int64_t)ce];
    const int4 m1 = reinterpret_cast<const int4 *>(meta)[2 * (int64_t)ce + 1];
    const int row0 = __builtin_amdgcn_readfirstlane(m0.x), n = __builtin_amdgcn_readfirstlane(m0.y),
              slot = __builtin_amdgcn_readfirstlane(m0.z), pos0 = __builtin_amdgcn_readfirstlane(m0.w),
              t0 = __builtin_amdgcn_readfirstlane(m1.x);
    const int last = min(t0 + C, pos0 + n) - 1;   // last key of the item
    const int32_t *pt = page_table + (int64_t)slot * max_pages;
    const int64_t page_bytes = (int64_t)(hkv << lgP) * D * 2, head_bytes = (int64_t)(h << lgP) * D * 2;
    const char *pool[2] = {reinterpret_cast<const char *>(kbase) + head_bytes, reinterpret_cast<const char *>(vbase) + head_bytes};
    const uint32_t lds0 = lds_offset(kv);

    // Tile of 64 keys from `key0` into buffer `buf`: wave w loads keys 16 w .. 16 w + 15 of K and of V, KPI per instruction.
    // Keys past the item's last one repeat it (finite values under weights of zero); a group of KPI keys lies in one
    // page, whose id was looked up a tile ahead (a look-up between the loads would wait for them).
    int page[NI];
    auto look_up = [&](int key0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) page[i] = pt[min(key0 + (wave * NI + i) * KPI, last) >> lgP];
    };
    auto request = [&](int key0, int buf) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int kb = (wave * NI + i) * KPI;              // first key of the instruction inside the tile
            const int64_t at = __builtin_amdgcn_readfirstlane(page[i]) * page_bytes;
            const int key = kb + lane / PC, src = min(key0 + key, last);
            const uint32_t off = (uint32_t)((src & (P - 1)) * (D * 2)) + (uint32_t)(((lane % PC) ^ (key & (PC - 1))) * 16);
            load_to_lds(pool[0] + at, off, lds0 + (uint32_t)(((buf * 2 + 0) * kTile + kb) * PC) * 16);
            load_to_lds(pool[1] + at, off, lds0 + (uint32_t)(((buf * 2 + 1) * kTile + kb) * PC) * 16);
        }
    };
    look_up(t0);
    request(t0, 0);

    // this lane's operand row and its query head as B operand fragments
    const int i = wave * 16 + col, pi = i / G, head = h * G + i % G;
    const bool live = pi < n;
    const int pos = live ? pos0 + pi : -1;                     // last key the row sees
    const int wave_last = (wave * 16) / G < n ? pos0 + min((wave * 16 + 15) / G, n - 1) : -1;   // last key any row of the wave sees
    const int wave_first = (wave * 16 + 15) / G < n ? pos0 + (wave * 16) / G : -1;              // last key that every row of the wave sees (-1: a dead row)
    u32x4_t qh[KST], ql[KST];
    {
        const float scale = rsqrtf((float)D) * 1.44269504f;              // scores in units of log2: p is one exp2 instruction
        const float *qp = qkv + (int64_t)(row0 + min(pi, n - 1)) * ldq + head * D + g4 * 8;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {
            const float4 q0 = *reinterpret_cast<const float4 *>(qp + ks * 32), q1 = *reinterpret_cast<const float4 *>(qp + ks * 32 + 4);
            split_fragment(q0, q1, scale, qh[ks], ql[ks]);
        }
    }
    look_up(t0 + kTile);
    // Sums in blocks: `o` starts anew at every tile and is added to `sum`.  One chain over a whole context rounds so often at
    // the size of the result that the output's distance from float64 (2.56e-6, 2-norm; the two bf16 terms that it is stored in
    // round it too) grew by 1.3 % at 1756 keys; blocks of 4 tiles leave 0.08 % and take the same time (1024 rows
    // over 4024 keys, 8 heads on one KV head: 133.7 us, every tile 133.0 us, two runs of one side differ by 0.9 us).
    floatx4_t o[FT], sum[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) o[f] = sum[f] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    float M = -INFINITY, den = 0.f;

    const int tiles = (last - t0) / kTile + 1;
    for (int t = 0; t < tiles; ++t) {
        const int buf = t & 1, key0 = t0 + t * kTile;
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");    // tile t is in LDS, every wave has read tile t - 1
        if (t + 1 < tiles) { request(key0 + kTile, buf ^ 1); look_up(key0 + 2 * kTile); }
        if (key0 > wave_last) continue;                                  // nothing for this wave's rows (it keeps loading its share)
        const char *kt = reinterpret_cast<const char *>(kv[buf][0]), *vt = reinterpret_cast<const char *>(kv[buf][1]);
        floatx4_t s[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {                               // four independent accumulators per k-step
            u32x4_t kf[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int key = j * 16 + col;
                kf[j] = *reinterpret_cast<const u32x4_t *>(kt + (key * PC + ((ks * 4 + g4) ^ (key & (PC - 1)))) * 16);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) s[j] = mfma_16x16x32(kf[j], qh[ks], s[j]);
#pragma unroll
            for (int j = 0; j < 4; ++j) s[j] = mfma_16x16x32(kf[j], ql[ks], s[j]);
        }
        float p[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) p[j] = s[j >> 2][j & 3];
        if (key0 + kTile - 1 > wave_first) {                             // the diagonal (and whatever lies past the item's last key, which is past pos too)
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (key0 + (j >> 2) * 16 + g4 * 4 + (j & 3) > pos) p[j] = -INFINITY;
        }
        float mt = p[0];
#pragma unroll
        for (int j = 1; j < 16; ++j) mt = fmaxf(mt, p[j]);
        mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
        mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
        const float Mn = fmaxf(M, mt);
#pragma unroll
        for (int f = 0; f < FT; ++f) { sum[f] += o[f]; o[f] = floatx4_t{0.f, 0.f, 0.f, 0.f}; }      // the products of the tile before are long done
        if (__any(Mn > M)) {                                             // some row of the wave has a new maximum
            const float corr = M == Mn ? 1.f : __builtin_amdgcn_exp2f(M - Mn);      // exp2(-inf) = 0 on the row's first keys
            M = Mn;
            den *= corr;
#pragma unroll
            for (int f = 0; f < FT; ++f) sum[f] *= corr;
        }
        const float m0_ = M == -INFINITY ? 0.f : M;                      // a row that has seen no key yet: all its scores are -inf, p = 0
#pragma unroll
        for (int j = 0; j < 16; ++j) p[j] = __builtin_amdgcn_exp2f(p[j] - m0_);
        den += (((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]))) +
               (((p[8] + p[9]) + (p[10] + p[11])) + ((p[12] + p[13]) + (p[14] + p[15])));
#pragma unroll
        for (int u = 0; u < 2; ++u) {                                    // 32 keys: the 16-key tiles 2 u and 2 u + 1
            u32x4_t ph, pm, pl;
            split3_bf16(p + u * 8, ph, pm, pl);
            const int ka = u * 32 + g4 * 4 + (col >> 2), kb = ka + 16;   // keys whose pieces this lane addresses
#pragma unroll
            for (int f = 0; f < FT; ++f) {
                const int piece = f * 2 + ((col & 3) >> 1), half = (col & 1) * 8;
                const uint2 va = lds_read_tr(vt + (ka * PC + (piece ^ (ka & (PC - 1)))) * 16 + half);
                const uint2 vb = lds_read_tr(vt + (kb * PC + (piece ^ (kb & (PC - 1)))) * 16 + half);
                const u32x4_t vf = {va.x, va.y, vb.x, vb.y};
                o[f] = mfma_16x16x32(vf, ph, o[f]);
                o[f] = mfma_16x16x32(vf, pm, o[f]);
                o[f] = mfma_16x16x32(vf, pl, o[f]);
            }
        }
    }
    den += __shfl_xor(den, 16, 64);
    den += __shfl_xor(den, 32, 64);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < FT; ++f) o[f] += sum[f];

    // A row's products with the keys it does not see (and the zero terms of p) are products with zero: not a number where
    // such a V is infinite or not a number itself.  Rows that met one are summed again, one key after the other and only
    // those of some weight, so that a position never depends on a later one.
    bool bad = false;
#pragma unroll
    for (int f = 0; f < FT; ++f) bad |= o[f][0] != o[f][0] || o[f][1] != o[f][1] || o[f][2] != o[f][2] || o[f][3] != o[f][3];
    if (__any(bad && live)) {
        const float scale = rsqrtf((float)D) * 1.44269504f, top = M == -INFINITY ? 0.f : M;
        const float *qp = qkv + (int64_t)(row0 + min(pi, n - 1)) * ldq + head * D;
        const int end = min(wave_last, last);
        den = 0.f;
#pragma unroll
        for (int f = 0; f < FT; ++f) o[f] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int key = t0; key <= end; ++key) {
            const int64_t at = pt[key >> lgP] * page_bytes + (int64_t)(key & (P - 1)) * (D * 2);
            const uint16_t *kr = reinterpret_cast<const uint16_t *>(pool[0] + at), *vr = reinterpret_cast<const uint16_t *>(pool[1] + at);
            float dot = 0.f;
#pragma unroll 1
            for (int e = 0; e < D; ++e) dot = fmaf(qp[e] * scale, bf16_to_f32(kr[e]), dot);
            const float w = key <= pos ? __builtin_amdgcn_exp2f(dot - top) : 0.f;
            den += w;
            if (w != 0.f) {
#pragma unroll
                for (int f = 0; f < FT; ++f)
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[f][j] = fmaf(w, bf16_to_f32(vr[f * 16 + g4 * 4 + j]), o[f][j]);
            }
        }
    }
    if (!live || pos < t0) return;                                       // the row takes no part in this chunk (no barrier follows)
    if (DIRECT) {
        const float inv = 1.0f / den;
        const int KSo = a.hq * D / 32;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            uint16_t hh[4], ll[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) split_bf16(o[f][j] * inv, hh[j], ll[j]);
            const int64_t off = packed_elem_offset(row0 + pi, head * D + f * 16 + g4 * 4, KSo);
            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.ohi) + off) = make_uint2((uint32_t)hh[0] | ((uint32_t)hh[1] << 16), (uint32_t)hh[2] | ((uint32_t)hh[3] << 16));
            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.olo) + off) = make_uint2((uint32_t)ll[0] | ((uint32_t)ll[1] << 16), (uint32_t)ll[2] | ((uint32_t)ll[3] << 16));
        }
    } else {
        const int64_t ci = a.chunk_start[row0 + pi] + t0 / C;
        float *acc = a.part_acc + (ci * a.hq + head) * D + g4 * 4;
#pragma unroll
        for (int f = 0; f < FT; ++f) *reinterpret_cast<float4 *>(acc + f * 16) = make_float4(o[f][0], o[f][1], o[f][2], o[f][3]);
        if (g4 == 0) *reinterpret_cast<float2 *>(a.part_ml + (ci * a.hq + head) * 2) = make_float2(M, den);
    }
}

template <int D, bool DIRECT>
hipError_t launch_prefill_d(const AttnArgs &a, hipStream_t s)
{
    const int lgP = __builtin_ctz(a.kv.P);
    const uint16_t *kb = a.kv.pool + a.kv.base(a.layer, 0), *vb = a.kv.pool + a.kv.base(a.layer, 1);
    switch (a.hq / a.kv.hkv) {
    case 1: attn_prefill_kernel<D, 1, DIRECT><<<a.n_items, 256, 0, s>>>(a.chunk_meta, kb, vb, a.qkv, a.page_table, (uint32_t)a.kv.hkv, a.ldq, lgP, a.chunk_tokens, a.max_pages, a); break;
    case 2: attn_prefill_kernel<D, 2, DIRECT><<<a.n_items, 256, 0, s>>>(a.chunk_meta, kb, vb, a.qkv, a.page_table, (uint32_t)a.kv.hkv, a.ldq, lgP, a.chunk_tokens, a.max_pages, a); break;
    case 4: attn_prefill_kernel<D, 4, DIRECT><<<a.n_items, 256, 0, s>>>(a.chunk_meta, kb, vb, a.qkv, a.page_table, (uint32_t)a.kv.hkv, a.ldq, lgP, a.chunk_tokens, a.max_pages, a); break;
    case 8: attn_prefill_kernel<D, 8, DIRECT><<<a.n_items, 256, 0, s>>>(a.chunk_meta, kb, vb, a.qkv, a.page_table, (uint32_t)a.kv.hkv, a.ldq, lgP, a.chunk_tokens, a.max_pages, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

int attn_prefill_block(int G) { return kRows / G; }

// a.chunk_meta holds block records (first row, rows, slot, first position | first key of the chunk), a.n_items = records x KV heads
hipError_t launch_attn_prefill(const AttnArgs &a, bool direct, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    if (a.chunk_tokens <= 0 || a.chunk_tokens % kTile) return hipErrorInvalidValue;
    if (a.kv.d == 128) return direct ? launch_prefill_d<128, true>(a, s) : launch_prefill_d<128, false>(a, s);
    if (a.kv.d == 64) return direct ? launch_prefill_d<64, true>(a, s) : launch_prefill_d<64, false>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace pat
