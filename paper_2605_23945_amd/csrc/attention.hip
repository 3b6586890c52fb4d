// Split-KV decode attention over the ragged, paged bf16 cache.
//
// Work item = (sequence, chunk of up to `chunk_tokens` cached positions, KV head), one workgroup
// each.  The flat item list covers the whole live batch, so one long sequence on a shard with a
// single KV head still spreads over the chip, and neighbouring items read neighbouring heads of
// the same pages.  Two kernels produce an item's partial (m, l, acc):
//   * G < 4 query heads per KV head (attn_stream_kernel): one pass, K and V rows of a round of
//     tokens in flight together and one round ahead, an online-softmax state per wave;
//   * G >= 4 (attn_gqa.hip): one pass on the matrix cores, K and V through LDS.
// A second kernel merges a sequence's partials with the online-softmax identity in a fixed
// order, so the result is run-to-run identical.
#include "attn_merge_dev.h"

namespace pat {

namespace {

constexpr int kAttnThreads = 256;

// G < 4 query heads per KV head (no matrix products), one pass: K and V rows of a round of
// tokens are requested together, one round ahead of the arithmetic, and every wave keeps an
// online-softmax state (running maximum, denominator, weighted V sum) over its own token rows,
// so nothing but the final combination of the four waves' states goes through LDS and no
// barrier separates the K stream from the V stream.
// What bounds it: HBM where the batch is long, the dependent loads of an item (record, rows) and the merge where it is short.
// What leads to the first loads comes as leading scalar arguments (in registers when a wave starts, see gemm_xs_kernel), page
// arithmetic is shifts: before, an item began with a round trip for its arguments and signed divisions per token row.  K and
// V are read once: as streamed (nontemporal) loads they arrive 6-13 % faster.  Kernel and merge, microseconds, before and now:
// one sequence of 2047 tokens on 8 heads 9.1, 7.9; two of about 2900 on 32 25.8, 20.6; 27 of about 1777 on 20 94, 80.7; 60 of
// about 1100 on 32 194, 165 (6.6 TB/s); 256 of about 620 456, 397.
// Sums: a lane adds one token of TPR per sub-round.  In chunks of more than 128 tokens (FOLD) its sums go to a second set every 128
// tokens and start again from zero, so that the rounding does not grow with the chunk.  Weighted sum of N(0, 1) values under N(0, 1)
// scores against float64, this order restated on the host, one chain and folded (in chunks of 128 tokens): 620 tokens whole
// 1.55e-7, 1.22e-7 (1.24e-7); 930 whole 1.73e-7, 1.27e-7 (1.26e-7); 2000 in chunks of 384 1.49e-7, 1.36e-7 (1.37e-7).  What it
// costs, a layer with its projections, microseconds: 60 sequences of about 1100 tokens on 32 heads 201.9, 202.0; 256 of about 620
// 438, 440; two query heads per KV head, 64 of about 2500 on 8 KV heads in chunks of 384 148.7, 149.1.  The registers of the second
// set leave three workgroups per compute unit of 128 features (held to 128 for four, 16 of about 1500 on 32 heads took 90.1, not 87.8).
constexpr int kFoldTokens = 128;
template <int D, int G, bool FOLD>
__global__ __launch_bounds__(kAttnThreads, !FOLD ? 1 : G == 2 ? 3 : D == 64 ? 4 : 1) void attn_stream_kernel(const int32_t *meta, const uint16_t *kbase, const uint16_t *vbase, const float *qkv, uint32_t hkv,
                                                                   int ldq, int lgP, int C, AttnArgs a)
{
    constexpr int LPT = D / 8;                  // lanes per token row
    constexpr int TPR = kAttnThreads / LPT;     // token rows per sub-round of the workgroup
    constexpr int UR = 4;                       // sub-rounds per round
    constexpr int RT = TPR * UR;                // tokens per round
    static_assert(RT == kFoldTokens || 2 * RT == kFoldTokens, "folds at every or every other round");
    __shared__ float red[4 * G * D];
    __shared__ float wml[4 * G * 2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ts = tid / LPT, seg = tid % LPT;
    const int P = 1 << lgP;
    const float scale = rsqrtf((float)D);
    const uint32_t page_bytes = (hkv << lgP) * (D * 2);                    // 32 bits: fewer than 2^16 heads of 128 features on pages of 128
    const uint32_t ce = blockIdx.x / hkv, h = blockIdx.x - ce * hkv;
    int4 m0 = reinterpret_cast<const int4 *>(meta)[2 * (int64_t)ce];
    int4 m1 = reinterpret_cast<const int4 *>(meta)[2 * (int64_t)ce + 1];
    asm volatile("" : "+s"(m0.x), "+s"(m0.y), "+s"(m0.z), "+s"(m1.x), "+s"(m1.y), "+s"(m1.z), "+s"(m1.w));     // one load, not two in turn
    int pg0 = m1.x, pg1 = m1.y, pg2 = m1.z, pg3 = m1.w;
    asm volatile("" : "+v"(pg0), "+v"(pg1), "+v"(pg2), "+v"(pg3));         // in vector registers a row's page is three selects, not branches
    const int b = m0.x, t0 = m0.y, cnt = m0.z;
    const bool rec_pages = C <= 4 * P;
    const int pfirst = t0 >> lgP;
    // chunks of more pages than their record holds (at most kAttnMaxChunk / 16): lane i keeps the chunk's i-th page, so that no
    // page look-up stands between a round's requests and the previous round's
    int pages = 0;
    if (!rec_pages) {
        const int32_t *pt = a.page_table + (int64_t)(a.row_slot ? a.row_slot[b] : b) * a.max_pages;
        pages = pt[min(pfirst + lane, (t0 + cnt - 1) >> lgP)];
    }
    const uint32_t head_off = ((h << lgP) * D + seg * 8) * 2;

    // K and V rows of one round: addresses first (unconditional, clamped to the chunk's last
    // token), then all 2 UR loads back to back
    auto fetch = [&](int r0, u32x4_t (&kr)[UR], u32x4_t (&vr)[UR]) {
        int tc[UR], page[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) { tc[u] = t0 + min(r0 + u * TPR + ts, cnt - 1); page[u] = (tc[u] >> lgP) - pfirst; }
        if (rec_pages) {
#pragma unroll
            for (int u = 0; u < UR; ++u) { const int lo = (page[u] & 1) ? pg1 : pg0, hi = (page[u] & 1) ? pg3 : pg2; page[u] = (page[u] & 2) ? hi : lo; }
        } else {
#pragma unroll
            for (int u = 0; u < UR; ++u) page[u] = __shfl(pages, page[u], 64);
        }
        uint64_t off[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) off[u] = (uint64_t)(uint32_t)page[u] * page_bytes + (head_off + (uint32_t)(tc[u] & (P - 1)) * (D * 2));
#pragma unroll
        for (int u = 0; u < UR; ++u) kr[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(reinterpret_cast<const char *>(kbase) + off[u]));
#pragma unroll
        for (int u = 0; u < UR; ++u) vr[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(reinterpret_cast<const char *>(vbase) + off[u]));
        __builtin_amdgcn_sched_barrier(0);
    };

    float q[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float *qp = qkv + (int64_t)b * ldq + (h * G + g) * D + seg * 8;
        const float4 q0 = *reinterpret_cast<const float4 *>(qp);
        const float4 q1 = *reinterpret_cast<const float4 *>(qp + 4);
        q[g][0] = q0.x * scale; q[g][1] = q0.y * scale; q[g][2] = q0.z * scale; q[g][3] = q0.w * scale;
        q[g][4] = q1.x * scale; q[g][5] = q1.y * scale; q[g][6] = q1.z * scale; q[g][7] = q1.w * scale;
    }
    // acc, den: of the tokens since the last fold; sum, dsum: of those before it, relative to Ms, the maximum at that fold
    float acc[G][8], den[G], M[G], sum[G][8], dsum[G], Ms[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        den[g] = dsum[g] = 0.f; M[g] = Ms[g] = -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[g][j] = sum[g][j] = 0.f;
    }
    auto fold = [&] {
        if (!FOLD) return;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (M[g] == -INFINITY) continue;                     // this wave has seen no token yet: nothing to add, nothing to scale
            const float corr = expf(Ms[g] - M[g]);               // 0 at the first fold
            dsum[g] = fmaf(dsum[g], corr, den[g]); den[g] = 0.f; Ms[g] = M[g];
#pragma unroll
            for (int j = 0; j < 8; ++j) { sum[g][j] = fmaf(sum[g][j], corr, acc[g][j]); acc[g][j] = 0.f; }
        }
    };

    auto consume = [&](int r0, const u32x4_t (&kr)[UR], const u32x4_t (&vr)[UR]) {
        float sv[UR][G];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const float k0 = bf16lo(kr[u].x), k1 = bf16hi(kr[u].x), k2 = bf16lo(kr[u].y), k3 = bf16hi(kr[u].y);
            const float k4 = bf16lo(kr[u].z), k5 = bf16hi(kr[u].z), k6 = bf16lo(kr[u].w), k7 = bf16hi(kr[u].w);
            const bool ok = r0 + u * TPR + ts < cnt;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float s = q[g][0] * k0;
                s = fmaf(q[g][1], k1, s); s = fmaf(q[g][2], k2, s); s = fmaf(q[g][3], k3, s);
                s = fmaf(q[g][4], k4, s); s = fmaf(q[g][5], k5, s); s = fmaf(q[g][6], k6, s);
                s = fmaf(q[g][7], k7, s);
#pragma unroll
                for (int o = LPT / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
                sv[u][g] = ok ? s : -INFINITY;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mr = sv[0][g];
#pragma unroll
            for (int u = 1; u < UR; ++u) mr = fmaxf(mr, sv[u][g]);
#pragma unroll
            for (int o = 32; o >= LPT; o >>= 1) mr = fmaxf(mr, __shfl_xor(mr, o, 64));
            const float Mn = fmaxf(M[g], mr);                    // the same in every lane of the wave
            if (Mn == -INFINITY) continue;                       // this wave has seen no token yet
            const float corr = expf(M[g] - Mn);                  // 0 on the wave's first tokens
            M[g] = Mn;
            den[g] *= corr;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[g][j] *= corr;
#pragma unroll
            for (int u = 0; u < UR; ++u) sv[u][g] = expf(sv[u][g] - Mn);     // exp(-inf) = 0 past the chunk
        }
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const float v0 = bf16lo(vr[u].x), v1 = bf16hi(vr[u].x), v2 = bf16lo(vr[u].y), v3 = bf16hi(vr[u].y);
            const float v4 = bf16lo(vr[u].z), v5 = bf16hi(vr[u].z), v6 = bf16lo(vr[u].w), v7 = bf16hi(vr[u].w);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (M[g] == -INFINITY) continue;                 // sv still holds -inf scores, not weights
                const float p = sv[u][g];
                den[g] += p;
                acc[g][0] = fmaf(p, v0, acc[g][0]); acc[g][1] = fmaf(p, v1, acc[g][1]);
                acc[g][2] = fmaf(p, v2, acc[g][2]); acc[g][3] = fmaf(p, v3, acc[g][3]);
                acc[g][4] = fmaf(p, v4, acc[g][4]); acc[g][5] = fmaf(p, v5, acc[g][5]);
                acc[g][6] = fmaf(p, v6, acc[g][6]); acc[g][7] = fmaf(p, v7, acc[g][7]);
            }
        }
    };

    u32x4_t kA[UR], vA[UR], kB[UR], vB[UR];
    fetch(0, kA, vA);
    for (int r0 = 0; r0 < cnt; r0 += 2 * RT) {
        const bool second = r0 + RT < cnt;
        if (second) fetch(r0 + RT, kB, vB);
        consume(r0, kA, vA);
        if (RT >= kFoldTokens) fold();
        if (second) {
            if (r0 + 2 * RT < cnt) fetch(r0 + 2 * RT, kA, vA);
            consume(r0 + RT, kB, vB);
            if (RT >= kFoldTokens) fold();
        }
        if (RT < kFoldTokens) fold();
    }

    // the wave's rows: lanes at distance LPT, 2 LPT, ... hold the same feature segment
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (FOLD) den[g] = dsum[g];
#pragma unroll
        for (int o = 32; o >= LPT; o >>= 1) den[g] += __shfl_xor(den[g], o, 64);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float v = FOLD ? sum[g][j] : acc[g][j];
#pragma unroll
            for (int o = 32; o >= LPT; o >>= 1) v += __shfl_xor(v, o, 64);
            acc[g][j] = v;
        }
    }
    if (lane < LPT) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int j = 0; j < 8; ++j) red[(wave * G + g) * D + lane * 8 + j] = acc[g][j];
    }
    if (lane == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) { wml[(wave * G + g) * 2] = M[g]; wml[(wave * G + g) * 2 + 1] = den[g]; }
    }
    __syncthreads();
    // the four waves' states in wave order; wave 0 always holds the chunk's first token
    if (a.direct) {
        // The row's only chunk (no merge: 8 sequences of the tiny configuration, two layers, step 82 -> 72 us together with
        // the plan's and the embedding's common launch): the operand of the O
        // projection, as the merge of one chunk would write it
        for (int e = tid; e < G * D / 8; e += kAttnThreads) {
            const int g = e / (D / 8), d0 = (e - g * (D / 8)) * 8;
            float mw[4], sw[4], Mc = -INFINITY;
#pragma unroll
            for (int w = 0; w < 4; ++w) { mw[w] = wml[(w * G + g) * 2]; Mc = fmaxf(Mc, mw[w]); }
#pragma unroll
            for (int w = 0; w < 4; ++w) sw[w] = mw[w] == -INFINITY ? 0.f : expf(mw[w] - Mc);
            const float inv = 1.0f / ((wml[(0 * G + g) * 2 + 1] * sw[0] + wml[(1 * G + g) * 2 + 1] * sw[1]) +
                                      (wml[(2 * G + g) * 2 + 1] * sw[2] + wml[(3 * G + g) * 2 + 1] * sw[3]));
            float o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int dd = d0 + j;
                o[j] = ((red[(0 * G + g) * D + dd] * sw[0] + red[(1 * G + g) * D + dd] * sw[1]) +
                        (red[(2 * G + g) * D + dd] * sw[2] + red[(3 * G + g) * D + dd] * sw[3])) * inv;
            }
            attn_write_operand<false>(a, b, (h * G + g) * D + d0, o);
        }
        return;
    }
    for (int e = tid; e < G * D + G; e += kAttnThreads) {
        const int g = e < G * D ? e / D : e - G * D;
        float mw[4], Mc = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) { mw[w] = wml[(w * G + g) * 2]; Mc = fmaxf(Mc, mw[w]); }
        float sw[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) sw[w] = mw[w] == -INFINITY ? 0.f : expf(mw[w] - Mc);
        if (e < G * D) {
            const int dd = e - g * D;
            a.part_acc[((int64_t)ce * a.hq + h * G + g) * D + dd] =
                (red[(0 * G + g) * D + dd] * sw[0] + red[(1 * G + g) * D + dd] * sw[1]) +
                (red[(2 * G + g) * D + dd] * sw[2] + red[(3 * G + g) * D + dd] * sw[3]);
        } else {
            float *ml = a.part_ml + ((int64_t)ce * a.hq + h * G + g) * 2;
            ml[0] = Mc;
            ml[1] = (wml[(0 * G + g) * 2 + 1] * sw[0] + wml[(1 * G + g) * 2 + 1] * sw[1]) +
                    (wml[(2 * G + g) * 2 + 1] * sw[2] + wml[(3 * G + g) * 2 + 1] * sw[3]);
        }
    }
}

// One wave per (sequence, query head): see attn_merge_row_head.
template <int D>
__global__ __launch_bounds__(64) void attn_merge_kernel(const int32_t *chunk_start, const float *part_ml, const float *part_acc, uint4 *ohi, uint4 *olo, int hq, float ml_unit, AttnArgs a)
{
    a.chunk_start = chunk_start; a.part_ml = const_cast<float *>(part_ml); a.part_acc = const_cast<float *>(part_acc); a.ohi = ohi; a.olo = olo; a.hq = hq; a.ml_unit = ml_unit;
    attn_merge_row_head<D, false>(a, blockIdx.y, blockIdx.x, threadIdx.x);
}

// Four waves per (sequence, query head), their states combined in wave order: what a merge of a long context takes is its
// rounds of dependent loads (16 chunks a round for one wave of 128 features, 64 for four).  One sequence
// of 33 chunks on 8 heads: the launch 4.86 -> 3.92 us, two of 23 on 32 heads 4.87 -> 4.78.
constexpr int kMergeWaves = 4;
template <int D>
__global__ __launch_bounds__(kMergeWaves * 64) void attn_merge_wide_kernel(const int32_t *chunk_start, const float *part_ml, const float *part_acc, uint4 *ohi, uint4 *olo, int hq, float ml_unit, AttnArgs a)
{
    a.chunk_start = chunk_start; a.part_ml = const_cast<float *>(part_ml); a.part_acc = const_cast<float *>(part_acc); a.ohi = ohi; a.olo = olo; a.hq = hq; a.ml_unit = ml_unit;
    constexpr int LPT = D / 8;
    __shared__ float st[kMergeWaves][LPT][10];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, b = blockIdx.y, head = blockIdx.x;
    const int ce0 = a.chunk_start[b], nch = a.chunk_start[b + 1] - ce0;
    float M, den, o[8];
    attn_merge_fold<D>(a, ce0, nch, head, lane, wave, kMergeWaves, M, den, o);
    if (lane < LPT) {
        st[wave][lane][8] = M; st[wave][lane][9] = den;
#pragma unroll
        for (int j = 0; j < 8; ++j) st[wave][lane][j] = o[j];
    }
    __syncthreads();
    if (threadIdx.x >= LPT) return;
    float Mc = M;
#pragma unroll
    for (int w = 1; w < kMergeWaves; ++w) Mc = fmaxf(Mc, st[w][lane][8]);
    const float s0 = M == -INFINITY ? 0.f : expf((M - Mc) * a.ml_unit);
    den *= s0;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] *= s0;
#pragma unroll
    for (int w = 1; w < kMergeWaves; ++w) {
        const float sw = st[w][lane][8] == -INFINITY ? 0.f : expf((st[w][lane][8] - Mc) * a.ml_unit);
        den += st[w][lane][9] * sw;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] += st[w][lane][j] * sw;
    }
    const float inv = 1.0f / den;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] *= inv;
    attn_write_operand<false>(a, b, head * D + lane * 8, o);
}

// Unused LDS, with which two workgroups fit a compute unit (160 KiB) and not four.  Over a long stream fewer rows read at a
// time are faster: 60 sequences of about 1100 tokens on 32 heads 165 us against 175 (chunks of 384 tokens), 256 of about 620
// 403 against 423; short ones need the four (3 sequences of about 2900: 28 against 36).
constexpr size_t kTwoPerCu = 54 * 1024;

template <int D, int G>
void launch_stream(const AttnArgs &a, int grid, size_t lds, int lgP, const uint16_t *kb, const uint16_t *vb, hipStream_t s)
{
    if (a.chunk_tokens > kFoldTokens) attn_stream_kernel<D, G, true><<<grid, kAttnThreads, lds, s>>>(a.chunk_meta, kb, vb, a.qkv, (uint32_t)a.kv.hkv, a.ldq, lgP, a.chunk_tokens, a);
    else attn_stream_kernel<D, G, false><<<grid, kAttnThreads, lds, s>>>(a.chunk_meta, kb, vb, a.qkv, (uint32_t)a.kv.hkv, a.ldq, lgP, a.chunk_tokens, a);
}

template <int D>
hipError_t launch_partial_d(const AttnArgs &a, int grid, hipStream_t s)
{
    const int G = a.hq / a.kv.hkv, lgP = __builtin_ctz(a.kv.P);
    const uint16_t *kb = a.kv.pool + a.kv.base(a.layer, 0), *vb = a.kv.pool + a.kv.base(a.layer, 1);
    const size_t lds = a.two_per_cu ? kTwoPerCu : 0;
    switch (G) {
    case 1: launch_stream<D, 1>(a, grid, lds, lgP, kb, vb, s); break;
    case 2: launch_stream<D, 2>(a, grid, lds, lgP, kb, vb, s); break;
    case 4: case 8: return launch_attn_gqa(a, s);
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_partial(const AttnArgs &a, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    if (a.chunk_tokens > kAttnMaxChunk || a.chunk_tokens <= 0) return hipErrorInvalidValue;
    const int grid = a.n_items;          // one workgroup per item: measured faster than any capped grid with a loop
    if (a.kv.d == 128) return launch_partial_d<128>(a, grid, s);
    if (a.kv.d == 64) return launch_partial_d<64>(a, grid, s);
    return hipErrorInvalidValue;
}

hipError_t launch_attn_merge(const AttnArgs &a, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    const dim3 grid(a.hq, a.B);
    if (a.kv.d != 128 && a.kv.d != 64) return hipErrorInvalidValue;
    // four waves where one would take a second round of loads and the chip has room for the others beside it
    if (a.longest_chunks > 4 * (512 / a.kv.d) && (int64_t)a.hq * a.B <= 1024) {
        if (a.kv.d == 128) attn_merge_wide_kernel<128><<<grid, kMergeWaves * 64, 0, s>>>(a.chunk_start, a.part_ml, a.part_acc, a.ohi, a.olo, a.hq, a.ml_unit, a);
        else attn_merge_wide_kernel<64><<<grid, kMergeWaves * 64, 0, s>>>(a.chunk_start, a.part_ml, a.part_acc, a.ohi, a.olo, a.hq, a.ml_unit, a);
    } else if (a.kv.d == 128) attn_merge_kernel<128><<<grid, 64, 0, s>>>(a.chunk_start, a.part_ml, a.part_acc, a.ohi, a.olo, a.hq, a.ml_unit, a);
    else attn_merge_kernel<64><<<grid, 64, 0, s>>>(a.chunk_start, a.part_ml, a.part_acc, a.ohi, a.olo, a.hq, a.ml_unit, a);
    return hipGetLastError();
}

}  // namespace pat
