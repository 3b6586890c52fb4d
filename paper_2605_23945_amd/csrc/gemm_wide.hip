// Projections of more than 32 rows, where the batch is a real dense dimension: a kernel that streams the weights past up
// to 128 rows at once and keeps both operand streams several k-steps ahead of the matrix cores.
//
// A workgroup of four waves (one per SIMD) owns RA row tiles x ALL 4 RB batch tiles of a row group x a K slice; wave w holds
// the accumulators of all RA row tiles against its own RB batch tiles.  So a batch fragment is needed by one wave only and
// goes straight from memory to its registers (a ring of XD + 1 k-steps), while the weight fragments, needed by all four
// waves, go straight from memory to LDS (`global_load_lds`, 1 KiB per instruction, a ring of WS k-steps) without
// touching a register.  One workgroup barrier per k-step; every row tile's step is one LDS read, its share of the k-step's
// requests and 2 RB matrix instructions (high and low halves), so requests, LDS reads and products interleave evenly.
//
// Sums: every XD + 1 k-steps a row tile's accumulators are added to a second set and start again from zero.  One chain over all
// of K rounds 2 K / 32 times at the size of the result; against float64 sums of the same operands that gave 5.7e-7 (2-norm,
// K = 4096), 8.1e-7 (K = 8192); in blocks it is 1.34e-7 .. 1.63e-7 over 102 pairs of shape and rows with K up to 11008.  The second
// set is why a wave takes at most two batch tiles.  The row tiles start their chains at different k-steps, and a tile's additions are spread between the
// products of the others: all tiles at once, in one k-step of the ring, they held up the matrix cores for 90 (8 x 2 tiles) to
// 180 (12 x 2) clocks per k-step.
//
// More than 128 rows are cut into NG equal groups in ONE launch: the groups of a row range are neighbours on one XCD and
// share its weight stream in L2.  That is faster than one group of up to 256 rows with one set of sums (22016 x 4096 at 256
// rows 85 us against 101, 8192 x 1024 16 against 31) but for wide projections of 129..192 rows (22016 x 4096 at 130 rows 81
// against 72) and of passes of about 1000 (1024 rows: 325 against 310; 7168 x 8192 213, now 184 by
// 16 row tiles, against 191).
//
// What bounds it: up to 128 rows the weight stream from HBM (the per-k-step requests of all workgroups in flight,
// up to 130 KB per compute unit, are what hides its latency).  Above, two things in turn.  The operands' delivery: clocks per k-step
// with all-zero operands, of products / alone without loads / in all, are 512 / 599 / 791 with 8 x 2 tiles, 768 / 899 / 1109 with
// 12 x 2, 384 / 445 / 768 with 12 x 1, so 31 to 50 % of a k-step is not products.  The one wave that a SIMD has issues everything (a
// product of 16 clocks leaves room for one other instruction: the loop has 57 others to 32 products, 8 x 2 tiles, where it had 75), and
// with one batch tile per wave LDS is the bound (4 waves read every weight: 125 bytes per clock at the products' rate).  Then the
// chip's power limit: with random operands the clock falls to 1.8 .. 2.0 GHz (all-zero ones: 2.4), and what the operands' way from L2
// and through LDS takes of the power is missing at the matrix cores.
// Staging the weights through registers into LDS, with exact waits, took the same time (8 x 2) or 10 % more (12 x 2); other
// cache policies of the weights' loads changed nothing.
// Measured against the kernel it replaced (batch
// fragments staged through registers into LDS, two k-steps ahead; same box, reduction included), microseconds:
//     rows          60            101           180           256           1024
//     22016 x 4096  52.1 -> 46.1  73.2 -> 57.4  88.4 -> 82.5  112  -> 84.6  449  -> 325
//     5120 x 6912   28.9 -> 27.5  40.6 -> 37.0  47.7 -> 42.2  59.4 -> 47.3  230  -> 128
//     1280 x 8192   21.9 -> 16.8  31.0 -> 19.6  33.5 -> 24.9  38.7 -> 28.2  147  -> 57.8
//     4096 x 1024   13.4 -> 12.9  17.8 -> 12.9  21.0 -> 13.2  24.1 -> 13.6  88.4 -> 23.9
//
// K can be split across workgroups (`plan_wide`); the slices' partial sums go to a scratch tensor and a reduction
// kernel adds them in slice order and runs the epilogue, so results never depend on timing.
#include <algorithm>
#include <type_traits>
#include <utility>
#include "gemm_dev.h"

namespace pat {

namespace {

// Depth of the two rings per tile shape: batch fragments XD k-steps ahead in registers (RA RB 4 accumulator registers
// and as many of the second sums beside them), weights WS - 1 k-steps ahead in LDS.  Loads complete in order, so a wait for a batch fragment also waits
// for the weights requested before it: XD bounds how much of the weight stream is in flight.
template <int RA, int RB> struct WideRings;
template <> struct WideRings<4, 1> { static constexpr int XD = 7, WS = 14; };
template <> struct WideRings<8, 1> { static constexpr int XD = 7, WS = 12; };
template <> struct WideRings<12, 1> { static constexpr int XD = 7, WS = 11; };
template <> struct WideRings<4, 2> { static constexpr int XD = 7, WS = 12; };
template <> struct WideRings<8, 2> { static constexpr int XD = 7, WS = 11; };
template <> struct WideRings<12, 2> { static constexpr int XD = 5, WS = 9; };
template <> struct WideRings<16, 2> { static constexpr int XD = 5, WS = 8; };
template <int RA, int RB> constexpr int wide_lds_bytes() { return WideRings<RA, RB>::WS * RA * 1024; }

// elements of a wave's row tile that are added to the second sums after j of the RA - 1 other row tiles
__host__ __device__ constexpr int wide_folded(int RA, int RB, int j) { return j * 4 * RB / (RA - 1); }
template <class F, int... I> __device__ __forceinline__ void static_for_i(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for_i(f, std::make_integer_sequence<int, N>{}); }

// MODE kPartial: the tile's sums go to a.part[kb][b][n_tiles * 16] (kb = K slice); otherwise (one slice) the epilogue runs here.
constexpr int kPartial = -1;
// The leading arguments are in registers when a wave starts (see gemm_xs_kernel): 14 words, the most that fit.  ng_gb: groups
// and rows of a group (<< 16); ks_qr: k-steps of a slice and how many slices have one more (<< 24).
template <int RA, int RB, int MODE>
__global__ __launch_bounds__(256) void gemm_wide_kernel(const uint4 *w, const uint4 *xhi, const uint4 *xlo, int KS, int B, uint32_t total, uint32_t ng_gb, uint32_t Rg, uint32_t ks_qr,
                                                        int tiles_q, int tiles_r, GemmArgs a)
{
    const uint32_t NG = ng_gb & 0xFFFFu;
    const int GB = ng_gb >> 16, ks_q = ks_qr & 0xFFFFFFu, ks_r = ks_qr >> 24;
    a.B = B;
    constexpr int XD = WideRings<RA, RB>::XD, WS = WideRings<RA, RB>::WS;
    constexpr int CW = RA / 4, CX = 2 * RB, PER = CW + CX;      // requests per wave and k-step: weights, batch fragments
    constexpr int U = XD + 1, DA = WS - 1, PF = 4;              // DA: k-steps the weights are requested ahead; PF: LDS reads in flight
    static_assert(RA % 4 == 0 && DA >= XD + 1 && (DA - 2) * PER <= 63, "the hand-counted waits fit the counter");
    extern __shared__ u32x4_t wring[];                          // [WS][RA][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroups are dealt round robin to the eight XCDs (blockIdx % 8); giving each XCD consecutive work items, slice
    // major, lets its workgroups share one K slice of the activations in their L2.
    const uint32_t id = blockIdx.x, item = (id & 7) * (total >> 3) + min(id & 7, total & 7) + (id >> 3);
    const uint32_t part = item / NG, grp = item - part * NG, kb = part / Rg, rg = part - kb * Rg;
    const int b0 = grp * GB, nb = min(GB, B - b0);              // this workgroup's batch rows b0 .. b0 + nb - 1
    // its k-steps and row tiles: the first ks_r slices (tiles_r ranges) have one more than the others
    const int ks0 = kb * ks_q + min((int)kb, ks_r), n = ks_q + ((int)kb < ks_r ? 1 : 0);
    const int rt0 = rg * tiles_q + min((int)rg, tiles_r), rt1 = rt0 + tiles_q + ((int)rg < tiles_r ? 1 : 0);
    const int bt0 = b0 >> 4, bt_last = (nb - 1) >> 4;
    const uint32_t lds0 = lds_offset(wring);

    // All requests are unconditional, from clamped (always valid) addresses, so that every wave issues the same number
    // per k-step: row tiles past the range repeat its last one and batch tiles past the live batch the last live one
    // (neither is stored), k-steps past the slice repeat its last one (never multiplied).  One wave per SIMD issues
    // everything, so what stands between its matrix instructions is kept short: bases in scalar registers, one offset per
    // operand and k-step (kw, kx) that stops at the slice's last k-step, ring slots as byte offsets.
    const char *wsrc[CW], *xsrc[CX];
#pragma unroll
    for (int i = 0; i < CW; ++i) wsrc[i] = reinterpret_cast<const char *>(w) + (uint64_t)(uint32_t)(min(rt0 + wave * CW + i, rt1 - 1) * KS + ks0) * 1024;
#pragma unroll
    for (int i = 0; i < CX; ++i)
        xsrc[i] = reinterpret_cast<const char *>(i / RB ? xlo : xhi) + (uint64_t)(uint32_t)((bt0 + min(wave * RB + i % RB, bt_last)) * KS + ks0) * 1024;
    const uint32_t lane16 = lane * 16, k_last = (uint32_t)(n - 1) * 1024, ring = lds0 + (uint32_t)(wave * CW) * 1024;
    uint32_t kw = 0, kx = 0;                                    // byte offsets of the next requests' k-steps inside the slice
    uint32_t at_req = 0, at_cur = 0;                            // ring slots (bytes): of the next request, of the current k-step
    constexpr uint32_t SLOT = RA * 1024, END = WS * SLOT;
    auto request_w = [&](int i) { load_to_lds_stream(wsrc[i], lane16 + kw, ring + at_req + i * 1024); };
    auto request_x = [&](int i) -> u32x4_t { return *reinterpret_cast<const u32x4_t *>(xsrc[i] + (lane16 + kx)); };

    floatx4_t acc[RA][RB], sum[RA][RB];
#pragma unroll
    for (int ra = 0; ra < RA; ++ra)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[ra][rb] = sum[ra][rb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t x[U][CX], wf[PF];
    // the requests of the k-steps -DA .. -1, in the order the loop would have issued them
#pragma unroll
    for (int s = -DA; s < 0; ++s) {
#pragma unroll
        for (int i = 0; i < CW; ++i) request_w(i);
        at_req += SLOT; kw = min(kw + 1024, k_last);
        if (s + XD >= 0) {
#pragma unroll
            for (int i = 0; i < CX; ++i) x[s + XD][i] = request_x(i);
            kx = min(kx + 1024, k_last);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // W(0), W(1): at least (DA - 2) CW younger requests are outstanding or done
    asm volatile("s_waitcnt vmcnt(%c0)\n\ts_barrier" ::"i"((DA - 2) * CW) : "memory");
#pragma unroll
    for (int p = 0; p < PF - 1; ++p) wf[p] = wring[p * 64 + lane];

    // One k-step.  The wait covers this wave's part of W(t + 1) (its requests are followed by those of DA - 2 whole
    // k-steps); after the barrier all parts are in LDS and every wave is done with the slot of W(t - 1), which takes W(t + DA).
    // Rows r with r % U == u start a new chain in this k-step; their sums so far were added to `sum` since their last products.
    auto step = [&](auto uu) {
        constexpr int u = decltype(uu)::value;
        const u32x4_t (&xc)[CX] = x[u];
        u32x4_t (&xn)[CX] = x[(u + XD) % U];
        asm volatile("s_waitcnt vmcnt(%c0)\n\ts_barrier" ::"i"((DA - 2) * PER) : "memory");
        const uint32_t at_nxt = at_cur + SLOT == END ? 0 : at_cur + SLOT;
        const char *cur = reinterpret_cast<const char *>(wring) + (at_cur + lane16), *nxt = reinterpret_cast<const char *>(wring) + (at_nxt + lane16);
#pragma unroll
        for (int r = 0; r < RA; ++r) {
#pragma unroll
            for (int v = (r * PER) / RA; v < ((r + 1) * PER) / RA; ++v) { if (v < CW) request_w(v); else xn[v - CW] = request_x(v - CW); }
            wf[(r + PF - 1) % PF] = *reinterpret_cast<const u32x4_t *>(r + PF - 1 < RA ? cur + (r + PF - 1) * 1024 : nxt + (r + PF - 1 - RA) * 1024);
#pragma unroll
            for (int i = 0; i < CX; ++i) acc[r][i % RB] = mfma16(wf[r % PF], xc[i], i < RB && r % U == u ? floatx4_t{0.f, 0.f, 0.f, 0.f} : acc[r][i % RB]);
            // the chains that restart in the next occurrence of their row: a share of their elements after every row
#pragma unroll
            for (int f = 0; f < RA; ++f) {
                const bool here = r > f ? f % U == (u + 1) % U : f % U == u;            // since f's products of the k-step before
                if (r == f || !here) continue;
                const int j = r > f ? r - f - 1 : r - f - 1 + RA, lo = wide_folded(RA, RB, j), hi = wide_folded(RA, RB, j + 1);
#pragma unroll
                for (int e = lo; e < hi; ++e) sum[f][e / 4][e % 4] += acc[f][e / 4][e % 4];
            }
            __builtin_amdgcn_sched_barrier(0);                  // keeps the interleaving, and every LDS read of a k-step before the next barrier
        }
        at_req = at_cur; at_cur = at_nxt;                       // the slot just read takes W(t + 1 + DA)
        kw = min(kw + 1024, k_last); kx = min(kx + 1024, k_last);
    };
    int t = 0;
    for (; t + U <= n; t += U) static_for<U>([&](auto u) { step(u); });
    static_for<U - 1>([&](auto u) { if (t + decltype(u)::value < n) step(u); });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // no write to LDS may be in flight when the workgroup ends
    const int u_end = n % U;                                    // rows r with r % U == u_end: part of their last chain is in `sum` already

    // the epilogue's addresses are derived from a copy of the lane index that the compiler cannot see through:
    // hoisted above the loop they would occupy registers it needs
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
#pragma unroll
    for (int ra = 0; ra < RA; ++ra) {
        const int rt = rt0 + ra;
        if (rt >= rt1) continue;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            floatx4_t s = sum[ra][rb];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += u_end == ra % U && rb * 4 + e < wide_folded(RA, RB, RA - 1 - ra) ? 0.f : acc[ra][rb][e];
            const float4 v = make_float4(s[0], s[1], s[2], s[3]);
            const int bl = (wave * RB + rb) * 16 + (lane_e & 15), b = bl < nb ? b0 + bl : a.B, quad = lane_e >> 4;     // b == a.B: not stored
            if (MODE == kPartial) {
                if (b < a.B) *reinterpret_cast<float4 *>(a.part + ((int64_t)kb * a.B + b) * ((int64_t)a.n_tiles * 16) + rt * 16 + quad * 4) = v;
            } else gemm_epilogue<MODE == kPartial ? 0 : MODE>(a, rt, quad, b, v);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// The four consecutive features 4 q .. of batch row b, summed over the K slices in slice order; the slices' loads are
// issued together (a loop over a run-time count would wait for each).
template <int KB>
__device__ __forceinline__ float4 sum_slices_n(const GemmArgs &a, int b, int q)
{
    const int64_t row = (int64_t)b * a.n_tiles * 16 + q * 4, slice = (int64_t)a.B * a.n_tiles * 16;
    float4 t[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) t[kb] = *reinterpret_cast<const float4 *>(a.part + row + kb * slice);
    float4 v = t[0];
#pragma unroll
    for (int kb = 1; kb < KB; ++kb) { v.x += t[kb].x; v.y += t[kb].y; v.z += t[kb].z; v.w += t[kb].w; }
    return v;
}
__device__ __forceinline__ float4 sum_slices(const GemmArgs &a, int b, int q)
{
    switch (a.Kb) {                                             // max_slices() is at most 8
    case 1: return sum_slices_n<1>(a, b, q);
    case 2: return sum_slices_n<2>(a, b, q);
    case 3: return sum_slices_n<3>(a, b, q);
    case 4: return sum_slices_n<4>(a, b, q);
    case 5: return sum_slices_n<5>(a, b, q);
    case 6: return sum_slices_n<6>(a, b, q);
    case 7: return sum_slices_n<7>(a, b, q);
    default: return sum_slices_n<8>(a, b, q);
    }
}

// Slice sums, then the epilogue: one thread per (row tile, batch row, quad), quads fastest, then batch rows, so that a
// wave reads 64-byte runs of 16 rows and its SwiGLU results (packed operand, 4 bytes per lane) form 256-byte runs.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(float *part, int B, int Kb, int n_tiles, GemmArgs a)
{
    a.part = part; a.B = B; a.Kb = Kb; a.n_tiles = n_tiles;
    const uint32_t i = blockIdx.x * 256 + threadIdx.x, per_tile = B * 4;      // fewer than 2^32: B rows of n_tiles x 4 quads
    const int rt = i / per_tile, r = i - rt * per_tile;
    if (rt >= n_tiles) return;
    const int b = r >> 2, quad = r & 3;
    gemm_epilogue<MODE>(a, rt, quad, b, sum_slices(a, b, rt * 4 + quad));
}

// Slice sums of a residual projection, y += sums, and the RMSNorm that the next projection applies to y, written as
// its packed split-bf16 operand: one workgroup per batch row, so that the row's sum of squares is at hand without a
// kernel (and a pass over y) of its own.  What bounds it is the latency of its loads: a thread requests the slices and y of
// its KEEP x 4 features together (up to 4 x 2048 features of a row; wider rows take more rounds and re-read their y).
// One quad after another: 9.9 us for 180 rows of 8192 features in two slices, 8.7 for 256 of 4096 in four; with them together a
// step of the 70B TP = 8 shard at 180 rows is 7 us per layer faster.
constexpr int kNormThreads = 512;
template <int KB>
__global__ __launch_bounds__(kNormThreads) void gemm_reduce_norm_kernel(const float *part, float *y0, const uint16_t *gains, uint4 *hi, uint4 *lo, int n_tiles, int ldy, int64_t slice,
                                                                        int s_h, float s_eps)
{
    constexpr int KEEP = 4;
    __shared__ float wsum[kNormThreads / 64];
    const int b = blockIdx.x, quads = n_tiles * 4, KSo = n_tiles >> 1;
    float4 *y = reinterpret_cast<float4 *>(y0 + (int64_t)b * ldy);
    const float4 *p = reinterpret_cast<const float4 *>(part) + (int64_t)b * quads;
    float ss = 0.f;
    float4 keep[KEEP];
    uint2 gk[KEEP];
#pragma unroll
    for (int i = 0; i < KEEP; ++i) gk[i] = *reinterpret_cast<const uint2 *>(gains + min((int)threadIdx.x + i * kNormThreads, quads - 1) * 4);
    auto round = [&](int q0, bool kept) {
        float4 t[KEEP][KB], c[KEEP];
#pragma unroll
        for (int i = 0; i < KEEP; ++i) {
            const int q = min(q0 + i * kNormThreads, quads - 1);               // past the row: a clamped, unused load
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) t[i][kb] = p[q + kb * slice];
            c[i] = y[q];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < KEEP; ++i) {
            const int q = q0 + i * kNormThreads;
            if (q >= quads) break;
            float4 v = t[i][0];
#pragma unroll
            for (int kb = 1; kb < KB; ++kb) { v.x += t[i][kb].x; v.y += t[i][kb].y; v.z += t[i][kb].z; v.w += t[i][kb].w; }
            v.x += c[i].x; v.y += c[i].y; v.z += c[i].z; v.w += c[i].w;
            y[q] = v;
            ss += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
            if (kept) keep[i] = v;
        }
    };
    round(threadIdx.x, true);
    for (int q0 = threadIdx.x + KEEP * kNormThreads; q0 < quads; q0 += KEEP * kNormThreads) round(q0, false);
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kNormThreads / 64; ++w) tot += wsum[w];
    const float inv = 1.0f / sqrtf(tot / (float)s_h + s_eps);
    auto emit = [&](int q, float4 v, uint2 gv) {
        uint16_t h[4], l[4];
        split_bf16(v.x * inv * bf16lo(gv.x), h[0], l[0]); split_bf16(v.y * inv * bf16hi(gv.x), h[1], l[1]);
        split_bf16(v.z * inv * bf16lo(gv.y), h[2], l[2]); split_bf16(v.w * inv * bf16hi(gv.y), h[3], l[3]);
        const int64_t off = packed_elem_offset(b, q * 4, KSo);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(hi) + off) = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(lo) + off) = make_uint2((uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16));
    };
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        const int q = threadIdx.x + i * kNormThreads;
        if (q < quads) emit(q, keep[i], gk[i]);
    }
    for (int q = threadIdx.x + KEEP * kNormThreads; q < quads; q += kNormThreads) emit(q, y[q], *reinterpret_cast<const uint2 *>(gains + q * 4));
}

template <int KB>
hipError_t launch_reduce_norm_t(const GemmArgs &a, hipStream_t s)
{
    gemm_reduce_norm_kernel<KB><<<(unsigned)a.B, kNormThreads, 0, s>>>(a.part, a.y, a.ngains, a.npk_hi, a.npk_lo, a.n_tiles, a.ldy, (int64_t)a.B * a.n_tiles * 4, a.s_h, a.s_eps);
    return hipGetLastError();
}

hipError_t launch_reduce_norm(const GemmArgs &a, hipStream_t s)
{
    switch (a.Kb) {                                             // max_slices() is at most 8
    case 1: return launch_reduce_norm_t<1>(a, s);
    case 2: return launch_reduce_norm_t<2>(a, s);
    case 3: return launch_reduce_norm_t<3>(a, s);
    case 4: return launch_reduce_norm_t<4>(a, s);
    case 5: return launch_reduce_norm_t<5>(a, s);
    case 6: return launch_reduce_norm_t<6>(a, s);
    case 7: return launch_reduce_norm_t<7>(a, s);
    default: return launch_reduce_norm_t<8>(a, s);
    }
}

template <int RA, int RB, int MODE>
hipError_t launch_wide_t(const GemmArgs &a, hipStream_t s)
{
    const unsigned total = (unsigned)(a.Rg * a.Kb * a.NG);
    gemm_wide_kernel<RA, RB, MODE><<<total, 256, wide_lds_bytes<RA, RB>(), s>>>(a.w, a.xhi, a.xlo, a.KS, a.B, total, (uint32_t)a.NG | (uint32_t)a.GB << 16, (uint32_t)a.Rg,
                                                                                (uint32_t)(a.KS / a.Kb) | (uint32_t)(a.KS % a.Kb) << 24, a.n_tiles / a.Rg, a.n_tiles % a.Rg, a);
    return hipGetLastError();
}

template <int RA, int RB>
hipError_t launch_wide_modes(const GemmArgs &a, int mode, hipStream_t s)
{
    switch (mode) {
    case kPartial: return launch_wide_t<RA, RB, kPartial>(a, s);
    case kGemmStore: return launch_wide_t<RA, RB, kGemmStore>(a, s);
    case kGemmAccum: return launch_wide_t<RA, RB, kGemmAccum>(a, s);
    case kGemmQKV: return launch_wide_t<RA, RB, kGemmQKV>(a, s);
    default: return launch_wide_t<RA, RB, kGemmSwiGLU>(a, s);
    }
}

// mode: kPartial, kGemmStore, or (8, 12 and 16 row tiles) any other epilogue in the kernel
template <int RB>
hipError_t launch_wide_rb(const GemmArgs &a, int RA, int mode, hipStream_t s)
{
    if (RA == 4) return mode == kPartial ? launch_wide_t<4, RB, kPartial>(a, s) : launch_wide_t<4, RB, kGemmStore>(a, s);
    if (RA == 8) return launch_wide_modes<8, RB>(a, mode, s);
    if constexpr (RB == 2) { if (RA == 16) return launch_wide_modes<16, RB>(a, mode, s); }
    return launch_wide_modes<12, RB>(a, mode, s);
}

template <int RA, int RB, int MODE>
hipError_t wide_set_lds_limit() { return hipFuncSetAttribute((const void *)gemm_wide_kernel<RA, RB, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds_bytes<RA, RB>()); }

template <int RA, int RB>
hipError_t wide_set_lds_limit_modes()
{
    hipError_t e = wide_set_lds_limit<RA, RB, kPartial>();
    if (e == hipSuccess) e = wide_set_lds_limit<RA, RB, kGemmStore>();
    if (e == hipSuccess) e = wide_set_lds_limit<RA, RB, kGemmAccum>();
    if (e == hipSuccess) e = wide_set_lds_limit<RA, RB, kGemmQKV>();
    if (e == hipSuccess) e = wide_set_lds_limit<RA, RB, kGemmSwiGLU>();
    return e;
}

template <int RB>
hipError_t wide_set_lds_limits()
{
    hipError_t e = wide_set_lds_limit<4, RB, kPartial>();
    if (e == hipSuccess) e = wide_set_lds_limit<4, RB, kGemmStore>();
    if (e == hipSuccess) e = wide_set_lds_limit_modes<8, RB>();
    if (e == hipSuccess) e = wide_set_lds_limit_modes<12, RB>();
    return e;
}

// How many K slices a projection may be cut into: about one workgroup of 16 row tiles per compute unit and at least
// 8 k-steps per slice.  The bound on the partial sums' scratch follows from it, so it is kept apart from the choice below.
int max_slices(int n_tiles, int KS, int n_cu)
{
    const int chunks = (n_tiles + 15) / 16;
    int kb = std::max(1, std::min(8, n_cu / chunks));
    while (kb > 1 && KS / kb < 8) --kb;
    return kb;
}

}  // namespace

hipError_t gemm_wide_prepare_device()
{
    hipError_t e = wide_set_lds_limits<1>();
    if (e == hipSuccess) e = wide_set_lds_limits<2>();
    return e == hipSuccess ? wide_set_lds_limit_modes<16, 2>() : e;
}

// Row tiles per workgroup (4, 8, 12, and 16 with two batch tiles per wave), batch tiles per wave (1, 2: groups of up to 64 or
// 128 rows) and K slices, by a cost model fitted to 8039 measured launches: every cut of 17 projections (1280..32000 features,
// K 1024..11008) at 16 live batches of 33..1024 rows, the residual ones with the RMSNorm that follows (rms error 7 %; the cut it
// picks is 0.9 % off the best measured on average, within 3 % in 90 % of the 272 cases, within 10 % in 96 %).  A launch takes
// 8.7 us plus its k-steps, each the longest of the matrix products (0.067 us and 0.0183 per tile pair), the operand fetch (0.0194
// us per KiB of weights and 0.0105 per KiB of batch fragments of a workgroup) and the weight stream (0.038 us per KiB and
// workgroup with all 256 busy, less where groups share it).  Partial sums cost 0.83 us per MB; a following norm 6.8 us and 0.89 us
// per MB of results as a launch of its own, 2.2 us and 0.24 per MB of results within the reduction of the slices.  16 row
// tiles read the least per product and need one round of workgroups where 8 need two: 7168 x 8192 at 1024 rows 184 us against
// 207, 8192 x 3584 92 against 105, 8192 x 1024 35 against 41.  Few row
// tiles per workgroup and few slices suit narrow projections (1280 x 8192, 64 rows: 4 tiles 16.9 us, 8 tiles 20.3), many
// tiles wide ones (22016 x 4096, 256 rows: 12 tiles 86 us, 8 tiles 115).  A projection without scratch for partial sums takes
// the kernels of 8 tiles and more, which exist with every epilogue; part_bytes bounds the slices (B rows of partial sums each).
void plan_wide(int n_tiles, int KS, int B, int n_cu, int64_t part_bytes, bool norm, GemmPlan &p)
{
    const int kb_max = max_slices(n_tiles, KS, n_cu);
    double best = 0.0;
    for (int RB = 1; RB <= 2; ++RB) {
        const int ng = (B + 64 * RB - 1) / (64 * RB), gb = ((B + ng - 1) / ng + 15) / 16 * 16;
        if (RB == 2 && gb <= 64) continue;                                         // as with one tile per wave
        for (int RA = 4; RA <= (RB == 1 ? 12 : 16); RA += 4)
            for (int kb = 1; kb <= kb_max; ++kb) {
                const int64_t bytes = (int64_t)kb * B * n_tiles * 64;
                if (bytes > part_bytes && (kb > 1 || RA == 4)) continue;             // without scratch: one slice, kernels with every epilogue
                const int rg = (n_tiles + RA - 1) / RA, wgs = rg * kb * ng, rounds = (wgs + n_cu - 1) / n_cu;
                const double busy = std::min(1.0, (double)wgs / n_cu);
                const double step = std::max({0.067 + 0.0183 * RA * RB, 0.0074 + 0.0194 * RA + 0.084 * RB, 0.0383 * RA * busy * (ng > 1 ? 0.49 : 1.0)});
                const bool direct = kb == 1 && RA != 4;
                const double mb = 1e-6 * (double)bytes, y_mb = mb / kb;
                const double tail = norm ? (direct ? 6.8 + 0.89 * y_mb : 2.2 + 0.72 * mb + 0.24 * y_mb) : direct ? 0.0 : 0.08 + 0.83 * mb;
                const double cost = 8.7 + rounds * ((KS + kb - 1) / kb) * step + tail;
                if (best == 0.0 || cost < best) { best = cost; p.Kb = kb; p.Rg = rg; p.MT = RA; p.NB = 4 * RB; p.NG = ng; p.GB = gb; }
            }
    }
}

// Bytes of partial sums a launch may need (an upper bound over the cuts plan_wide chooses from).
int64_t gemm_wide_scratch_bytes(int n_tiles, int KS, int B, int n_cu)
{
    const int kb = max_slices(n_tiles, KS, n_cu);
    return kb > 1 ? (int64_t)kb * B * n_tiles * 64 : 0;
}

hipError_t launch_gemm_wide(const GemmArgs &a0, const GemmPlan &p, int mode, hipStream_t s)
{
    GemmArgs a = a0;
    const bool direct = p.Kb == 1 && (mode == kGemmStore || p.MT != 4);
    if (!direct && (a.part == nullptr || (int64_t)a.Kb * a.B * a.n_tiles * 64 > a.part_bytes)) return hipErrorInvalidValue;
    const int m = direct ? mode : kPartial;
    if (direct) a.ngains = nullptr;          // the epilogue's own hand-over is the small-batch one (x * gains and per-tile statistics)
    const hipError_t e = p.NB == 4 ? launch_wide_rb<1>(a, p.MT, m, s) : launch_wide_rb<2>(a, p.MT, m, s);
    if (e != hipSuccess) return e;
    if (direct) {
        if (mode == kGemmAccum && a0.ngains != nullptr) return launch_rmsnorm_pack(a.y, a0.ngains, a.B, a.s_h, a.s_eps, a.npk_hi, a.npk_lo, s);
        return hipSuccess;
    }
    if (mode == kGemmAccum && a.ngains != nullptr) {
        return launch_reduce_norm(a, s);
    }
    const unsigned blocks = (unsigned)(((int64_t)a.B * a.n_tiles * 4 + 255) / 256);
    switch (mode) {
    case kGemmStore: gemm_reduce_kernel<kGemmStore><<<blocks, 256, 0, s>>>(a.part, a.B, a.Kb, a.n_tiles, a); break;
    case kGemmAccum: gemm_reduce_kernel<kGemmAccum><<<blocks, 256, 0, s>>>(a.part, a.B, a.Kb, a.n_tiles, a); break;
    case kGemmQKV: gemm_reduce_kernel<kGemmQKV><<<blocks, 256, 0, s>>>(a.part, a.B, a.Kb, a.n_tiles, a); break;
    default: gemm_reduce_kernel<kGemmSwiGLU><<<blocks, 256, 0, s>>>(a.part, a.B, a.Kb, a.n_tiles, a); break;
    }
    return hipGetLastError();
}

}  // namespace pat
