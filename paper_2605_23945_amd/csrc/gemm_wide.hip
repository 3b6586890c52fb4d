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
// Sums: every XD + 1 k-steps the accumulators are added to a second set and start again from zero.  One chain over all of K
// rounds 2 K / 32 times at the size of the result; against float64 sums of the same operands that gave 5.7e-7 (2-norm,
// K = 4096), 8.1e-7 (K = 8192); in blocks it is 1.4e-7 .. 1.9e-7 at every K up to 11008, no more than the K slices of the
// kernel it replaces gave (1.4e-7 .. 4.0e-7).  The second set is why a wave takes at most two batch tiles: 12 x 3, 8 x 4 and
// 12 x 4 tiles have no registers for it.  The additions cost 1-3 % of a launch.
//
// More than 128 rows are cut into NG equal groups in ONE launch: the groups of a row range are neighbours on one XCD and
// share its weight stream in L2.  That is faster than one group of up to 256 rows with one set of sums (22016 x 4096 at 256
// rows 85 us against 101, 8192 x 1024 16 against 31) but for wide projections of 129..192 rows (22016 x 4096 at 130 rows 81
// against 72) and of passes of about 1000 (1024 rows: 325 against 310; 7168 x 8192 213 against 191).
//
// What bounds it: up to 128 rows the weight stream from HBM (the per-k-step requests of all workgroups in flight,
// up to 130 KB per compute unit, are what hides its latency); at 256 rows the chip's power limit (random operands run
// 25-40 % slower than all-zero ones at the same instruction stream).  Measured against the kernel it replaces (batch
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
template <int RA, int RB> constexpr int wide_lds_bytes() { return WideRings<RA, RB>::WS * RA * 1024; }

// MODE kPartial: the tile's sums go to a.part[kb][b][n_tiles * 16] (kb = K slice); otherwise (one slice) the epilogue runs here.
constexpr int kPartial = -1;
template <int RA, int RB, int MODE>
__global__ __launch_bounds__(256) void gemm_wide_kernel(GemmArgs a)
{
    constexpr int XD = WideRings<RA, RB>::XD, WS = WideRings<RA, RB>::WS;
    constexpr int CW = RA / 4, CX = 2 * RB, PER = CW + CX;      // requests per wave and k-step: weights, batch fragments
    constexpr int U = XD + 1, DA = WS - 1, PF = 4;              // DA: k-steps the weights are requested ahead; PF: LDS reads in flight
    static_assert(RA % 4 == 0 && DA >= XD + 1 && (DA - 2) * PER <= 63, "the hand-counted waits fit the counter");
    extern __shared__ u32x4_t wring[];                          // [WS][RA][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KS = a.KS;
    // Workgroups are dealt round robin to the eight XCDs (blockIdx % 8); giving each XCD consecutive work items, slice
    // major, lets its workgroups share one K slice of the activations in their L2.
    const int id = blockIdx.x, total = a.Kb * a.Rg * a.NG;
    const int item = (id & 7) * (total >> 3) + min(id & 7, total & 7) + (id >> 3);
    const int part = item / a.NG, grp = item - part * a.NG, kb = part / a.Rg, rg = part - kb * a.Rg;
    const int b0 = grp * a.GB, nb = min(a.GB, a.B - b0);        // this workgroup's batch rows b0 .. b0 + nb - 1
    const int ks0 = (int)((int64_t)kb * KS / a.Kb), n = (int)((int64_t)(kb + 1) * KS / a.Kb) - ks0;
    const int rt0 = (int)((int64_t)rg * a.n_tiles / a.Rg), rt1 = (int)((int64_t)(rg + 1) * a.n_tiles / a.Rg);
    const int bt0 = b0 >> 4, bt_last = (nb - 1) >> 4;
    const uint32_t lds0 = lds_offset(wring);

    // All requests are unconditional, from clamped (always valid) addresses, so that every wave issues the same number
    // per k-step: row tiles past the range repeat its last one and batch tiles past the live batch the last live one
    // (neither is stored), k-steps past the slice repeat its last one (never multiplied).
    const u32x4_t *wsrc[CW], *xsrc[CX];
#pragma unroll
    for (int i = 0; i < CW; ++i) wsrc[i] = reinterpret_cast<const u32x4_t *>(a.w) + ((int64_t)min(rt0 + wave * CW + i, rt1 - 1) * KS + ks0) * 64;
#pragma unroll
    for (int i = 0; i < CX; ++i)
        xsrc[i] = reinterpret_cast<const u32x4_t *>(i / RB ? a.xlo : a.xhi) + ((int64_t)(bt0 + min(wave * RB + i % RB, bt_last)) * KS + ks0) * 64;
    int s_req = 0, s_cur = 0;                                   // ring slots: of the next request, of the current k-step
    auto request_w = [&](int t, int i) { load_to_lds_stream(wsrc[i] + min(t, n - 1) * 64, lane * 16, lds0 + (s_req * RA + wave * CW + i) * 1024); };
    auto request_x = [&](int t, int i) -> u32x4_t { return *(xsrc[i] + min(t, n - 1) * 64 + lane); };

    floatx4_t acc[RA][RB], sum[RA][RB];
#pragma unroll
    for (int ra = 0; ra < RA; ++ra)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[ra][rb] = sum[ra][rb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t x[U][CX], w[PF];
    // the requests of the k-steps -DA .. -1, in the order the loop would have issued them
#pragma unroll
    for (int s = -DA; s < 0; ++s) {
#pragma unroll
        for (int i = 0; i < CW; ++i) request_w(s + DA, i);
        ++s_req;
        if (s + XD >= 0) {
#pragma unroll
            for (int i = 0; i < CX; ++i) x[s + XD][i] = request_x(s + XD, i);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // W(0), W(1): at least (DA - 2) CW younger requests are outstanding or done
    asm volatile("s_waitcnt vmcnt(%c0)\n\ts_barrier" ::"i"((DA - 2) * CW) : "memory");
#pragma unroll
    for (int p = 0; p < PF - 1; ++p) w[p] = wring[p * 64 + lane];

    // One k-step.  The wait covers this wave's part of W(t + 1) (its requests are followed by those of DA - 2 whole
    // k-steps); after the barrier all parts are in LDS and every wave is done with the slot of W(t - 1), which takes W(t + DA).
    auto step = [&](int t, const u32x4_t (&xc)[CX], u32x4_t (&xn)[CX], auto fold) {
        asm volatile("s_waitcnt vmcnt(%c0)\n\ts_barrier" ::"i"((DA - 2) * PER) : "memory");
        const int s_nxt = s_cur + 1 == WS ? 0 : s_cur + 1;
        const u32x4_t *cur = wring + s_cur * RA * 64 + lane, *nxt = wring + s_nxt * RA * 64 + lane;
#pragma unroll
        for (int r = 0; r < RA; ++r) {
#pragma unroll
            for (int v = (r * PER) / RA; v < ((r + 1) * PER) / RA; ++v) { if (v < CW) request_w(t + DA, v); else xn[v - CW] = request_x(t + XD, v - CW); }
            w[(r + PF - 1) % PF] = r + PF - 1 < RA ? cur[(r + PF - 1) * 64] : nxt[(r + PF - 1 - RA) * 64];
            if constexpr (decltype(fold)::value) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) { sum[r][rb] += acc[r][rb]; acc[r][rb] = floatx4_t{0.f, 0.f, 0.f, 0.f}; }
            }
#pragma unroll
            for (int i = 0; i < CX; ++i) acc[r][i % RB] = mfma16(w[r % PF], xc[i], acc[r][i % RB]);
            __builtin_amdgcn_sched_barrier(0);                  // keeps the interleaving, and every LDS read of a k-step before the next barrier
        }
        s_cur = s_nxt; s_req = s_req + 1 == WS ? 0 : s_req + 1;
    };
    int t = 0;
    for (; t + U <= n; t += U) {
        step(t, x[0], x[XD % U], std::true_type{});
#pragma unroll
        for (int u = 1; u < U; ++u) step(t + u, x[u], x[(u + XD) % U], std::false_type{});
    }
    if (t < n) step(t, x[0], x[XD % U], std::true_type{});
#pragma unroll
    for (int u = 1; u < U - 1; ++u)
        if (t + u < n) step(t + u, x[u], x[(u + XD) % U], std::false_type{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // no write to LDS may be in flight when the workgroup ends

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
            const floatx4_t s = sum[ra][rb] + acc[ra][rb];
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
    const int64_t ldp = (int64_t)a.n_tiles * 16;
    float4 t[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) t[kb] = *reinterpret_cast<const float4 *>(a.part + ((int64_t)kb * a.B + b) * ldp + q * 4);
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
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int per_tile = a.B * 4;
    const int rt = (int)(i / per_tile), r = (int)(i - (int64_t)rt * per_tile);
    if (rt >= a.n_tiles) return;
    const int b = r >> 2, quad = r & 3;
    gemm_epilogue<MODE>(a, rt, quad, b, sum_slices(a, b, rt * 4 + quad));
}

// Slice sums of a residual projection, y += sums, and the RMSNorm that the next projection applies to y, written as
// its packed split-bf16 operand: one workgroup per batch row, so that the row's sum of squares is at hand without a
// kernel (and a pass over y) of its own.  Up to 4 x 2048 features stay in registers; wider rows re-read their y.
// A reduction and a norm launch took 7.7 + 7.2 us at 256 rows of 4096 features, 4.7 + 5.1 us at 60.
constexpr int kNormThreads = 512;
__global__ __launch_bounds__(kNormThreads) void gemm_reduce_norm_kernel(GemmArgs a)
{
    constexpr int KEEP = 4;
    __shared__ float wsum[kNormThreads / 64];
    const int b = blockIdx.x, quads = a.n_tiles * 4, KSo = a.n_tiles >> 1;
    float *y = a.y + (int64_t)b * a.ldy;
    float4 keep[KEEP];
    float ss = 0.f;
    auto take = [&](int q) {
        float4 v = sum_slices(a, b, q);
        const float4 c = *reinterpret_cast<const float4 *>(y + q * 4);
        v.x += c.x; v.y += c.y; v.z += c.z; v.w += c.w;
        *reinterpret_cast<float4 *>(y + q * 4) = v;
        ss += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
        return v;
    };
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        const int q = threadIdx.x + i * kNormThreads;
        keep[i] = q < quads ? take(q) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int q = threadIdx.x + KEEP * kNormThreads; q < quads; q += kNormThreads) (void)take(q);
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kNormThreads / 64; ++w) tot += wsum[w];
    const float inv = 1.0f / sqrtf(tot / (float)a.s_h + a.s_eps);
    auto emit = [&](int q, float4 v) {
        const uint2 gv = *reinterpret_cast<const uint2 *>(a.ngains + q * 4);
        uint16_t h[4], l[4];
        split_bf16(v.x * inv * bf16lo(gv.x), h[0], l[0]); split_bf16(v.y * inv * bf16hi(gv.x), h[1], l[1]);
        split_bf16(v.z * inv * bf16lo(gv.y), h[2], l[2]); split_bf16(v.w * inv * bf16hi(gv.y), h[3], l[3]);
        const int64_t off = packed_elem_offset(b, q * 4, KSo);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.npk_hi) + off) = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.npk_lo) + off) = make_uint2((uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16));
    };
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        const int q = threadIdx.x + i * kNormThreads;
        if (q < quads) emit(q, keep[i]);
    }
    for (int q = threadIdx.x + KEEP * kNormThreads; q < quads; q += kNormThreads) emit(q, *reinterpret_cast<const float4 *>(y + q * 4));
}

template <int RA, int RB, int MODE>
hipError_t launch_wide_t(const GemmArgs &a, hipStream_t s)
{
    gemm_wide_kernel<RA, RB, MODE><<<(unsigned)(a.Rg * a.Kb * a.NG), 256, wide_lds_bytes<RA, RB>(), s>>>(a);
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

// mode: kPartial, kGemmStore, or (8 and 12 row tiles) any other epilogue in the kernel
template <int RB>
hipError_t launch_wide_rb(const GemmArgs &a, int RA, int mode, hipStream_t s)
{
    if (RA == 4) return mode == kPartial ? launch_wide_t<4, RB, kPartial>(a, s) : launch_wide_t<4, RB, kGemmStore>(a, s);
    if (RA == 8) return launch_wide_modes<8, RB>(a, mode, s);
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
    const hipError_t e = wide_set_lds_limits<1>();
    return e == hipSuccess ? wide_set_lds_limits<2>() : e;
}

// Row tiles per workgroup (4, 8, 12), batch tiles per wave (1, 2: groups of up to 64 or 128 rows) and K slices, by a cost
// model fitted to 6910 measured launches: every cut of 17 projections (1280..32000 features, K 1024..11008) at 16 live
// batches of 33..1024 rows, the residual ones with the RMSNorm that follows (rms error 7 %; the cut it picks is within 3 % of
// the best measured in 91 % of the 272 cases, within 10 % in 97 %, 0.8 % off on average).  A launch takes 9.1 us plus its
// k-steps, each the longest of the matrix products (0.0215 us per tile pair), the operand fetch (0.0194 us per KiB of weights
// and 0.0104 per KiB of batch fragments of a workgroup) and the weight stream (0.037 us per KiB and workgroup with all 256
// busy, less where groups share it).  Partial sums cost 0.88 us per MB; a following norm 7.4 us and 0.87 us per MB of
// results as a launch of its own, 2.4 us and 0.15 per MB of results within the reduction of the slices.  Few row
// tiles per workgroup and few slices suit narrow projections (1280 x 8192, 64 rows: 4 tiles 16.9 us, 8 tiles 20.3), many
// tiles wide ones (22016 x 4096, 256 rows: 12 tiles 86 us, 8 tiles 115).  A projection without scratch for partial sums takes
// the 8- or 12-tile kernels, which exist with every epilogue; part_bytes bounds the slices (B rows of partial sums each).
void plan_wide(int n_tiles, int KS, int B, int n_cu, int64_t part_bytes, bool norm, GemmPlan &p)
{
    const int kb_max = max_slices(n_tiles, KS, n_cu);
    double best = 0.0;
    for (int RB = 1; RB <= 2; ++RB) {
        const int ng = (B + 64 * RB - 1) / (64 * RB), gb = ((B + ng - 1) / ng + 15) / 16 * 16;
        if (RB == 2 && gb <= 64) continue;                                         // as with one tile per wave
        for (int RA = 4; RA <= 12; RA += 4)
            for (int kb = 1; kb <= kb_max; ++kb) {
                const int64_t bytes = (int64_t)kb * B * n_tiles * 64;
                if (bytes > part_bytes && (kb > 1 || RA == 4)) continue;             // without scratch: one slice, kernels with every epilogue
                const int rg = (n_tiles + RA - 1) / RA, wgs = rg * kb * ng, rounds = (wgs + n_cu - 1) / n_cu;
                const double busy = std::min(1.0, (double)wgs / n_cu);
                const double step = std::max({0.0215 * RA * RB, 0.0065 + 0.0194 * RA + 0.0832 * RB, 0.037 * RA * busy * (ng > 1 ? 0.3 : 1.0)});
                const bool direct = kb == 1 && RA != 4;
                const double mb = 1e-6 * (double)bytes, y_mb = mb / kb;
                const double tail = norm ? (direct ? 7.4 + 0.87 * y_mb : 2.4 + 0.8 * mb + 0.15 * y_mb) : direct ? 0.0 : 0.6 + 0.88 * mb;
                const double cost = 9.1 + rounds * ((KS + kb - 1) / kb) * step + tail;
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
        gemm_reduce_norm_kernel<<<(unsigned)a.B, kNormThreads, 0, s>>>(a);
        return hipGetLastError();
    }
    const unsigned blocks = (unsigned)(((int64_t)a.B * a.n_tiles * 4 + 255) / 256);
    switch (mode) {
    case kGemmStore: gemm_reduce_kernel<kGemmStore><<<blocks, 256, 0, s>>>(a); break;
    case kGemmAccum: gemm_reduce_kernel<kGemmAccum><<<blocks, 256, 0, s>>>(a); break;
    case kGemmQKV: gemm_reduce_kernel<kGemmQKV><<<blocks, 256, 0, s>>>(a); break;
    default: gemm_reduce_kernel<kGemmSwiGLU><<<blocks, 256, 0, s>>>(a); break;
    }
    return hipGetLastError();
}

}  // namespace pat
