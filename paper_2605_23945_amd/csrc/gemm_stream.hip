// Weight-streaming skinny GEMM  Y[B, N] = X[B, K] W^T  for the sharded
// projections of the decode step (QKV, O, gate/up, down, vocabulary head).
//
// The step is bound by reading W once from HBM.  W is kept in a streaming layout
// (see pat_dev.h): the 16 rows x K strip of a row tile is one contiguous run,
// every wave load is a full 1 KiB line-aligned block of 16-byte vectors, and each
// vector is directly the A operand of v_mfma_f32_16x16x32_bf16.  The live batch
// (padded to 16) is the MFMA's N dimension, so B <= 16 costs the same bytes as
// B = 1.  Activations are fp32 split into two bf16 terms (hi + lo), giving
// fp32-class products on the bf16 matrix cores; accumulation is fp32.
//
// gemm_xs_kernel (live batch <= 32) is activation-stationary: each wave keeps its K slice of the activations in
// registers and streams row tiles past it (wave-level split-K, partial tiles summed through LDS in wave order).
// Larger live batches: gemm_wide.hip.
#include <algorithm>
#include <cstdlib>
#include <mutex>
#include "gemm_dev.h"

namespace pat {

namespace {

// ---- live batch <= 32: activation-stationary streaming ------------------------------
// A workgroup owns a group of row tiles over the whole of K.  Each of its waves (8 or 16) owns a
// contiguous K range and walks it in passes of UK k-steps: for a pass it loads its
// split-bf16 activation fragments into registers once and streams every row tile of the
// group past them, so activations are fetched once per workgroup instead of once per row
// tile, nearly every load in flight is a 1 KiB block of the HBM weight stream, and the
// waves run free of barriers while they stream.  A wave accumulates its partial tiles in
// its own LDS slots; after the last pass one barrier lets wave i sum tile i's partials in
// wave order.  No cross-workgroup reduction, no atomics: a fixed summation order.

// One pass of a wave: U k-steps [kw0, kw0 + U) against row tiles [tb0, tb0 + nt).  The wave's
// activation fragments of the pass are loaded once and stay in registers.  All loads are
// unconditional 16-byte vectors at constant offsets from one base.  Batch rows past the live batch
// re-read the last live row: their output columns are never stored, and a matrix-core output
// column depends on its own activation column only.
template <int NB, int U, int WAVES>
__device__ __forceinline__ void xs_pass(const GemmArgs &a, int lane, int wave, int kw0, int tb0, int nt, bool first,
                                        float4 *red)
{
    const int KS = a.KS;
    uint4 xh[U][NB], xl[U][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int rsel = min(lane & 15, a.B - 1 - nb * 16);
        const uint4 *ph = a.xhi + (nb * KS + kw0) * 64 + (lane >> 4) * 16 + rsel;
        const uint4 *pl = a.xlo + (nb * KS + kw0) * 64 + (lane >> 4) * 16 + rsel;
#pragma unroll
        for (int u = 0; u < U; ++u) { xh[u][nb] = ph[u * 64]; xl[u][nb] = pl[u * 64]; }
    }
    for (int i = 0; i < nt; ++i) {
        const uint4 *wp = a.w + ((int64_t)(tb0 + i) * KS + kw0) * 64 + lane;
        u32x4_t w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = ld16_stream(wp + u * 64);
        // keep all U loads in flight: without this the scheduler interleaves load / wait / multiply
        // through one register quad and the wave has a single KiB outstanding
        __builtin_amdgcn_sched_barrier(0);
        floatx4_t acc_h[NB], acc_l[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) { acc_h[nb] = floatx4_t{0.f, 0.f, 0.f, 0.f}; acc_l[nb] = floatx4_t{0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                acc_h[nb] = mfma16(w[u], xh[u][nb], acc_h[nb]);
                acc_l[nb] = mfma16(w[u], xl[u][nb], acc_l[nb]);
            }
        }
        // every accumulator is read here, in the block of the matrix instructions and before any branch (see mfma_sum_pinned)
        float4 v[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) v[nb] = mfma_sum_pinned(acc_h[nb], acc_l[nb]);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float4 *slot = &red[((i * WAVES + wave) * NB + nb) * 64 + lane];    // this wave's own slot
            if (!first) { const float4 o = *slot; v[nb].x += o.x; v[nb].y += o.y; v[nb].z += o.z; v[nb].w += o.w; }
            *slot = v[nb];
        }
    }
}

// The same for a live batch of at most 8 rows, whose high and low terms share one operand: columns 0 .. 7 hold the rows'
// high terms, columns 8 .. 15 their low terms, and a tile's sum is column c plus column c ^ 8: bit by bit the sums of
// xs_pass.  Half the matrix instructions, and half the activation loads: a 1 KiB load instruction costs a compute unit
// about 14 ns wherever its data is, and with two per k-step the activations took 2/3 of the loads of a workgroup with one row
// tile (7B down projection, 4096 x 11008: 1032 loads, 14 of the launch's 19 us).  7B shard, 2 rows: step 3.78 -> 3.64 ms;
// its TP = 4 shard, 1 row: 1.57 -> 1.53 ms.  The registers this frees are better left free: a second tile's weights in
// flight gave nothing (1.53 ms), passes of 11 k-steps lost 1 %.
template <int U, int WAVES>
__device__ __forceinline__ void xs_pass8(const GemmArgs &a, int lane, int wave, int kw0, int tb0, int nt, bool first, float4 *red)
{
    const int KS = a.KS;
    u32x4_t x[U];
    const uint4 *px = ((lane & 8) ? a.xlo : a.xhi) + kw0 * 64 + (lane >> 4) * 16 + min(lane & 7, a.B - 1);
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = ld16(px + u * 64);
    auto fetch = [&](u32x4_t (&w)[U], int i) {
        const uint4 *wp = a.w + ((int64_t)(tb0 + i) * KS + kw0) * 64 + lane;
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = ld16_stream(wp + u * 64);
        __builtin_amdgcn_sched_barrier(0);                  // all U loads in flight, ahead of the matrix instructions
    };
    auto tile = [&](const u32x4_t (&w)[U], int i) {
        floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) acc = mfma16(w[u], x[u], acc);
        float4 v = mfma_halves_pinned(acc);
        float4 *slot = &red[(i * WAVES + wave) * 64 + lane];
        if (!first) { const float4 o = *slot; v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w; }
        *slot = v;
    };
    for (int i = 0; i < nt; ++i) {
        u32x4_t w[U];
        fetch(w, i);
        tile(w, i);
    }
}

// one pass of either kind
template <int NB, int U, int WAVES, bool HL>
__device__ __forceinline__ void xs_run(const GemmArgs &a, int lane, int wave, int kw0, int tb0, int nt, bool first, float4 *red)
{
    if constexpr (HL) xs_pass8<U, WAVES>(a, lane, wave, kw0, tb0, nt, first, red);
    else xs_pass<NB, U, WAVES>(a, lane, wave, kw0, tb0, nt, first, red);
}

// The arguments that only the epilogue reads, as values that the compiler cannot see through at the place of the call: what
// is derived from them (a null test, a layer's address) is derived there and not ahead of the stream, which would wait for
// their fetch.  Whole groups of neighbours, also where a mode needs a part: the compiler fetches a group with one load, and
// would put something else into the registers of an unused neighbour, after a wait for the load.
template <class T> __device__ __forceinline__ void opaque(T &v) { asm volatile("" : "+s"(v)); }
template <class T>
__device__ __forceinline__ void opaque(T *&p)                   // stays a pointer to global memory for the compiler
{
    uint64_t v = (uint64_t)p;
    asm volatile("" : "+s"(v));
    p = (T *)(__attribute__((address_space(1))) T *)v;
}
template <class... T> __device__ __forceinline__ void opaque_all(T &...v) { (opaque(v), ...); }
template <int MODE>
__device__ __forceinline__ GemmArgs epilogue_args(GemmArgs a)
{
    opaque_all(a.y, a.ldy, a.n_valid);
    if (MODE == kGemmQKV) opaque_all(a.kv.pool, a.kv.n_pages, a.kv.hkv, a.kv.P, a.kv.d, a.layer, a.hq, a.max_pages, a.KS_out, a.kv_len, a.page_table, a.row_slot, a.rope_cs);
    if (MODE == kGemmSwiGLU) opaque_all(a.yhi, a.ylo, a.KS_out);
    if (MODE == kGemmAccum) opaque_all(a.ngains, a.npk_hi, a.npk_lo, a.nstats, a.n_tiles);
    else opaque_all(a.sstats, a.s_parts, a.s_h, a.s_eps, a.n_tiles);
    return a;
}

// What the first loads depend on comes as leading scalar arguments, which the compiler's kernel-argument preload has in
// registers when a wave starts; the rest of the arguments is fetched beside the stream.  The workgroup's row tiles follow
// from a quotient and a remainder that the host divides.  Before, a launch began with a round trip to memory for its
// arguments and two 64-bit divisions (150 scalar instructions each): eight steps of the 7B TP = 4 shard, one row, 11.95 ->
// 11.13 ms, four of the TP = 1 shard, two rows, 14.51 -> 13.92 ms, 32 of the tiny configuration 2.29 -> 2.03 ms.
template <int NB, int UK, int TB, int kXsWaves, bool HL, int MODE>
__global__ __launch_bounds__(kXsWaves * 64) void gemm_xs_kernel(const uint4 *w, const uint4 *xhi, const uint4 *xlo, int KS, int B, int tiles_q, int tiles_r, GemmArgs a)
{
    a.w = w; a.xhi = xhi; a.xlo = xlo; a.KS = KS; a.B = B;
    extern __shared__ float4 red[];   // [TB][kXsWaves][NB][64]
    constexpr int R = 16 * NB, PQ = R / 4;          // batch rows of the tiles, 16-byte pieces per part of the row statistics
    __shared__ __align__(16) float s_part[kXsWaves][R];
    // the wave index as a scalar: what derives from it (k share, slots, tile) stays in scalar registers
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = blockIdx.x;
    // the wave's contiguous share of the k-steps (shares differ by at most one step)
    const int kown0 = (int)((unsigned)(wave * KS) / kXsWaves), kown1 = (int)((unsigned)((wave + 1) * KS) / kXsWaves);
    // the workgroup's row tiles: the first tiles_r workgroups own one more than the others
    const int rt0 = rg * tiles_q + min(rg, tiles_r), rt1 = rt0 + tiles_q + (rg < tiles_r ? 1 : 0);

    // Folded RMSNorm (a.sstats set): the operand rows are x * gains, the results are multiplied by 1 / rms of their
    // batch row.  The rows' sums of squares come as per-part sums sstats[part][R]; the workgroup adds them once, in
    // a fixed order: thread t takes the 16-byte pieces t, t + threads, ... (four rows of one part) in increasing
    // order, a wave folds its pieces per row group with a shuffle butterfly, and the wave sums meet in LDS at the
    // barrier the first tile group has anyway.
    float inv[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) inv[nb] = 1.f;

    for (int tb0 = rt0; tb0 < rt1; tb0 += TB) {
        const int nt = min(TB, rt1 - tb0);
        // passes of 8 k-steps and one exact remainder pass cover the share: no block of W is read twice
        for (int k = kown0; k < kown1;) {
            const int rem = kown1 - k;
            const bool first = k == kown0;
            if (rem >= 8) { xs_run<NB, 8, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); k += 8; continue; }
            switch (rem) {
            case 7: xs_run<NB, 7, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            case 6: xs_run<NB, 6, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            case 5: xs_run<NB, 5, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            case 4: xs_run<NB, 4, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            case 3: xs_run<NB, 3, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            case 2: xs_run<NB, 2, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            default: xs_run<NB, 1, kXsWaves, HL>(a, lane, wave, k, tb0, nt, first, red); break;
            }
            k = kown1;
        }
        // The epilogue's own reads (see EpiPre) travel while the workgroup meets at the barrier.  What the epilogue
        // derives from the lane index is computed from this copy, which the compiler cannot see through: hoisted
        // above the stream those values would occupy registers the stream needs (spills inside the loop).
        int lane_e = lane, KS_e = KS;
        asm volatile("" : "+v"(lane_e), "+s"(KS_e));
        const GemmArgs e = epilogue_args<MODE>(a);
        const bool scale = MODE != kGemmAccum && e.sstats != nullptr;     // the residual projections are never the consumer of a norm
        EpiPre pre[NB];
        if (wave < nt) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) pre[nb] = epilogue_prefetch<MODE>(e, tb0 + wave, lane_e >> 4, nb * 16 + (lane_e & 15));
        }
        if (scale && tb0 == rt0) {
            // read after the stream, like the epilogue's other operands: nothing of it occupies registers during the stream
            float4 ssq = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int i = (wave << 6) + lane_e; i < e.s_parts * PQ; i += kXsWaves * 64) {
                const float4 t = reinterpret_cast<const float4 *>(e.sstats)[i];
                ssq.x += t.x; ssq.y += t.y; ssq.z += t.z; ssq.w += t.w;
            }
#pragma unroll
            for (int off = PQ; off < 64; off <<= 1) {
                ssq.x += __shfl_xor(ssq.x, off, 64); ssq.y += __shfl_xor(ssq.y, off, 64);
                ssq.z += __shfl_xor(ssq.z, off, 64); ssq.w += __shfl_xor(ssq.w, off, 64);
            }
            if (lane_e < PQ) *reinterpret_cast<float4 *>(&s_part[wave][lane_e * 4]) = ssq;
        }
        __syncthreads();
        if (scale && tb0 == rt0) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int row = min(nb * 16 + (lane & 15), a.B - 1);
                float tot = 0.f;
#pragma unroll
                for (int w = 0; w < kXsWaves; ++w) tot += s_part[w][row];
                inv[nb] = 1.0f / sqrtf(tot / (float)e.s_h + e.s_eps);
            }
        }
        if (wave < nt) {
            // D tile layout: lane l holds rows (l/16)*4 .. +3 of column l%16 = 4 consecutive
            // output features of one batch row.  Waves with an empty share left no partial.
            const int rt = tb0 + wave;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (KS_e >= kXsWaves) {                                    // every wave owns k-steps
                    v = red[(wave * kXsWaves * NB + nb) * 64 + lane];
#pragma unroll
                    for (int ww = 1; ww < kXsWaves; ++ww) {
                        const float4 t = red[((wave * kXsWaves + ww) * NB + nb) * 64 + lane];
                        v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
                    }
                } else {
                    for (int ww = 0; ww < kXsWaves; ++ww) {
                        if ((ww + 1) * KS_e / kXsWaves == ww * KS_e / kXsWaves) continue;   // empty share: no partial
                        const float4 t = red[((wave * kXsWaves + ww) * NB + nb) * 64 + lane];
                        v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
                    }
                }
                if (scale) { v.x *= inv[nb]; v.y *= inv[nb]; v.z *= inv[nb]; v.w *= inv[nb]; }
                gemm_epilogue<MODE>(e, rt, lane_e >> 4, nb * 16 + (lane_e & 15), v, pre[nb]);
            }
        }
        if (tb0 + TB < rt1) __syncthreads();
    }
}

// Matrices into the streaming layout, any number of them up to kPackJobs in one launch (a layer's; the workgroups of a
// matrix are consecutive).  A wave takes kPackSteps consecutive k-steps of a row tile: every lane loads 16 bytes of its
// row per k-step, all of them together, so that a row is read in runs of 256 bytes, and writes 1 KiB blocks.  A launch per
// matrix and one k-step per wave took 57 us per layer of the 7B TP = 4 shard cut from unsharded matrices (101 MB, six
// launches, 3.5 TB/s read and written), without the gaps between them; now 41 us, 4.9 TB/s, bound by memory.
constexpr int kPackSteps = 4;
__global__ __launch_bounds__(256) void pack_weight_kernel(PackJobs jobs)
{
    int q = 0;
    while (q + 1 < jobs.n && (int)blockIdx.x >= jobs.job[q + 1].block0) ++q;
    const PackJob &j = jobs.job[q];
    const int lane = threadIdx.x & 63, KS = j.KS, groups = (KS + kPackSteps - 1) / kPackSteps;
    const int64_t i = (int64_t)((int)blockIdx.x - j.block0) * 4 + (threadIdx.x >> 6);
    const int tile = (int)(i / groups), ks0 = (int)(i - (int64_t)tile * groups) * kPackSteps;
    if (tile >= j.n_tiles) return;
    const int row = tile * 16 + (lane & 15);
    const uint16_t *src = j.w;
    int srow = row;
    if (j.w2 != nullptr) { src = (row & 1) ? j.w2 : j.w; srow = row >> 1; }
    if (row < j.rope_rows) {                     // rotary partners (j, j + d/2) become stored neighbours
        const int head = row / j.d, p = row - head * j.d;
        srow = head * j.d + ((p & 1) ? (p >> 1) + (j.d >> 1) : (p >> 1));
    }
    const uint16_t *line = src + (int64_t)min(srow, j.n - 1) * j.ld + (lane >> 4) * 8;        // ld: elements between source rows
    uint4 v[kPackSteps];
#pragma unroll
    for (int u = 0; u < kPackSteps; ++u) v[u] = *reinterpret_cast<const uint4 *>(line + min(ks0 + u, KS - 1) * 32);
    uint4 *to = j.packed + ((int64_t)tile * KS + ks0) * 64 + lane;
#pragma unroll
    for (int u = 0; u < kPackSteps; ++u)
        if (ks0 + u < KS) to[u * 64] = srow < j.n ? v[u] : make_uint4(0, 0, 0, 0);
}

// one thread per (row, 8 consecutive k)
__global__ void pack_act_kernel(const float *x, int b, int k, int KS, uint4 *hi, uint4 *lo)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int groups = k >> 3;
    if (i >= (int64_t)b * groups) return;
    const int row = (int)(i / groups), k0 = (int)(i % groups) * 8;
    const float4 p = *reinterpret_cast<const float4 *>(x + (int64_t)row * k + k0);
    const float4 q = *reinterpret_cast<const float4 *>(x + (int64_t)row * k + k0 + 4);
    const float v[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
    uint16_t h[8], l[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) split_bf16(v[j], h[j], l[j]);
    const int64_t vi = packed_elem_offset(row, k0, KS) >> 3;
    hi[vi] = make_uint4(h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16, h[4] | (uint32_t)h[5] << 16,
                        h[6] | (uint32_t)h[7] << 16);
    lo[vi] = make_uint4(l[0] | (uint32_t)l[1] << 16, l[2] | (uint32_t)l[3] << 16, l[4] | (uint32_t)l[5] << 16,
                        l[6] | (uint32_t)l[7] << 16);
}

// RMSNorm of four rows per workgroup, written as packed split-bf16 activations.  In the packed operand the 16-byte
// pieces of neighbouring rows are neighbours, so the lanes of a wave take 16 pieces of each of the four rows (rows
// fastest): 512-byte reads of every row and 64-byte runs of the output.  One row per workgroup scattered its output in
// 16-byte pieces and was bound by those writes (1024 rows of 8192 features: 30 us).  Up to kKeep x 1024 features of a row
// stay in registers between the sum of squares and the scaling; wider rows are read again.
constexpr int kPackRows = 4, kPackThreads = 512, kPackLanes = kPackThreads / kPackRows;      // lanes per row
__global__ __launch_bounds__(kPackThreads) void rmsnorm_pack_kernel(const float *x, const uint16_t *g, int b, int h, int KS,
                                                                    float eps, uint4 *hi, uint4 *lo)
{
    constexpr int kKeep = 8;
    __shared__ float part[kPackThreads / 64][kPackRows];
    const int r = threadIdx.x & (kPackRows - 1), c0 = threadIdx.x / kPackRows;
    const int row = blockIdx.x * kPackRows + r;
    const float *xr = x + (int64_t)min(row, b - 1) * h;
    float4 xp[kKeep], xq[kKeep];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int k0 = min((c0 + i * kPackLanes) * 8, h - 8);                 // past the row: a clamped, unused load
        xp[i] = *reinterpret_cast<const float4 *>(xr + k0);
        xq[i] = *reinterpret_cast<const float4 *>(xr + k0 + 4);
    }
    float ss = 0.f;
    auto square = [&](float4 p, float4 q) { ss += p.x * p.x + p.y * p.y + p.z * p.z + p.w * p.w + q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w; };
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if ((c0 + i * kPackLanes) * 8 < h) square(xp[i], xq[i]);
    for (int k0 = (c0 + kKeep * kPackLanes) * 8; k0 < h; k0 += kPackLanes * 8)
        square(*reinterpret_cast<const float4 *>(xr + k0), *reinterpret_cast<const float4 *>(xr + k0 + 4));
#pragma unroll
    for (int o = 32; o >= kPackRows; o >>= 1) ss += __shfl_xor(ss, o, 64);
    if ((threadIdx.x & 63) < kPackRows) part[threadIdx.x >> 6][r] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kPackThreads / 64; ++w) tot += part[w][r];
    const float inv = 1.0f / sqrtf(tot / (float)h + eps);
    if (row >= b) return;
    auto emit = [&](int k0, float4 p, float4 q) {
        const uint4 gv = *reinterpret_cast<const uint4 *>(g + k0);
        const float v[8] = {p.x * inv * bf16lo(gv.x), p.y * inv * bf16hi(gv.x), p.z * inv * bf16lo(gv.y),
                            p.w * inv * bf16hi(gv.y), q.x * inv * bf16lo(gv.z), q.y * inv * bf16hi(gv.z),
                            q.z * inv * bf16lo(gv.w), q.w * inv * bf16hi(gv.w)};
        uint16_t hh[8], ll[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) split_bf16(v[j], hh[j], ll[j]);
        const int64_t vi = packed_elem_offset(row, k0, KS) >> 3;
        hi[vi] = make_uint4(hh[0] | (uint32_t)hh[1] << 16, hh[2] | (uint32_t)hh[3] << 16, hh[4] | (uint32_t)hh[5] << 16,
                            hh[6] | (uint32_t)hh[7] << 16);
        lo[vi] = make_uint4(ll[0] | (uint32_t)ll[1] << 16, ll[2] | (uint32_t)ll[3] << 16, ll[4] | (uint32_t)ll[5] << 16,
                            ll[6] | (uint32_t)ll[7] << 16);
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int k0 = (c0 + i * kPackLanes) * 8;
        if (k0 < h) emit(k0, xp[i], xq[i]);
    }
    for (int k0 = (c0 + kKeep * kPackLanes) * 8; k0 < h; k0 += kPackLanes * 8)
        emit(k0, *reinterpret_cast<const float4 *>(xr + k0), *reinterpret_cast<const float4 *>(xr + k0 + 4));
}

// the kernels' dynamic LDS exceeds the default limit: raised per device by gemm_prepare_device()
template <int NB, int UK, int TB, int kXsWaves, bool HL>
hipError_t xs_set_lds_limit()
{
    constexpr size_t lds = (size_t)TB * kXsWaves * NB * 64 * sizeof(float4);
    hipError_t e = hipFuncSetAttribute((const void *)gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmStore>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmAccum>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmSwiGLU>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmQKV>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    return e;
}

template <int NB, int UK, int TB, int kXsWaves, bool HL>
hipError_t launch_xs(const GemmArgs &a, int mode, hipStream_t s)
{
    const unsigned grid = (unsigned)a.Rg;
    const int tq = a.n_tiles / a.Rg, tr = a.n_tiles % a.Rg;
    constexpr size_t lds = (size_t)TB * kXsWaves * NB * 64 * sizeof(float4);
    switch (mode) {
    case kGemmStore: gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmStore><<<grid, kXsWaves * 64, lds, s>>>(a.w, a.xhi, a.xlo, a.KS, a.B, tq, tr, a); break;
    case kGemmAccum: gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmAccum><<<grid, kXsWaves * 64, lds, s>>>(a.w, a.xhi, a.xlo, a.KS, a.B, tq, tr, a); break;
    case kGemmQKV: gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmQKV><<<grid, kXsWaves * 64, lds, s>>>(a.w, a.xhi, a.xlo, a.KS, a.B, tq, tr, a); break;
    default: gemm_xs_kernel<NB, UK, TB, kXsWaves, HL, kGemmSwiGLU><<<grid, kXsWaves * 64, lds, s>>>(a.w, a.xhi, a.xlo, a.KS, a.B, tq, tr, a); break;
    }
    return hipGetLastError();
}

}  // namespace

// Once per device and process (the attribute belongs to the device's copy of the kernel); a bit per device id.
hipError_t gemm_prepare_device()
{
    static std::mutex mu;
    static uint64_t done = 0;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (dev >= 0 && dev < 64 && (done >> dev & 1)) return hipSuccess;
    e = xs_set_lds_limit<1, 8, 8, 16, true>();
    if (e == hipSuccess) e = xs_set_lds_limit<1, 8, 8, 16, false>();
    if (e == hipSuccess) e = xs_set_lds_limit<2, 8, 8, 8, false>();
    if (e == hipSuccess) e = gemm_wide_prepare_device();
    if (e == hipSuccess) e = attn_gqa_prepare_device();
    if (e == hipSuccess && dev >= 0 && dev < 64) done |= 1ull << dev;
    return e;
}

static int g_target_wgs = 256;   // one resident workgroup per compute unit
void gemm_set_compute_units(int n) { if (n > 0) g_target_wgs = n; }

GemmPlan gemm_plan(int n_tiles, int KS, int B, int64_t part_bytes, bool norm)
{
    GemmPlan p{1, 1, 1, 16, kAlgoXs, 1, B};
    if (B <= 32) {
        p.Kb = 1;                                              // a workgroup walks all of K itself
        p.Rg = n_tiles < g_target_wgs ? n_tiles : g_target_wgs;
        p.NB = B <= 16 ? 1 : 2; p.MT = B <= 16 ? 16 : 8;
    } else {
        p.algo = kAlgoWide;
        plan_wide(n_tiles, KS, B, g_target_wgs, part_bytes, norm, p);
    }
    return p;
}

int64_t gemm_scratch_bytes(int n_tiles, int KS, int B) { return B <= 32 ? 0 : gemm_wide_scratch_bytes(n_tiles, KS, B, g_target_wgs); }

hipError_t launch_gemm(const GemmArgs &a0, int mode, hipStream_t s)
{
    if (a0.B <= 0 || a0.n_tiles <= 0) return hipSuccess;
    if (a0.KS < 1) return hipErrorInvalidValue;
    GemmArgs a = a0;
    const GemmPlan p = gemm_plan(a.n_tiles, a.KS, a.B, a.part ? a.part_bytes : 0, mode == kGemmAccum && a.ngains != nullptr);
    a.Kb = p.Kb; a.Rg = p.Rg; a.NG = p.NG; a.GB = p.GB;
    if (a.sstats != nullptr && a.B > 32) return hipErrorInvalidValue;      // the consumer side of a folded RMSNorm: small-batch kernels only
    if (a.ngains != nullptr && (a.n_valid % 32 != 0 || !a.npk_hi || !a.npk_lo || (a.B <= 32 && !a.nstats))) return hipErrorInvalidValue;
    { const hipError_t e = gemm_prepare_device(); if (e != hipSuccess) return e; }
    // measured on MI355X: 16 waves x 8 resident k-steps is best for one batch tile, 8 x 8 for two; up to 8 rows both halves of
    // the split share the tile (xs_pass8)
    if (a.B <= 8) return launch_xs<1, 8, 8, 16, true>(a, mode, s);
    if (a.B <= 16) return launch_xs<1, 8, 8, 16, false>(a, mode, s);
    if (a.B <= 32) return launch_xs<2, 8, 8, 8, false>(a, mode, s);
    return launch_gemm_wide(a, p, mode, s);
}

PackJob pack_job(const uint16_t *w, const uint16_t *w2, int n, int k, int64_t ld, uint4 *packed, int rope_rows, int d)
{
    PackJob j{};
    j.w = w; j.w2 = w2; j.packed = packed; j.n = n; j.ld = ld; j.KS = k / 32; j.rope_rows = rope_rows; j.d = d;
    j.n_tiles = ((w2 ? 2 * n : n) + 15) / 16;
    return j;
}

hipError_t launch_pack_weights(const PackJob *jobs, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n > kPackJobs) return hipErrorInvalidValue;
    PackJobs p{};
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        p.job[i] = jobs[i];
        p.job[i].block0 = (int)blocks;
        blocks += ((int64_t)jobs[i].n_tiles * ((jobs[i].KS + kPackSteps - 1) / kPackSteps) + 3) / 4;
        if (blocks > INT32_MAX) return hipErrorInvalidValue;
    }
    p.n = n;
    if (blocks == 0) return hipSuccess;
    pack_weight_kernel<<<(unsigned)blocks, 256, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_pack_weight(const uint16_t *w, const uint16_t *w2, int n, int k, int64_t ld, uint4 *packed, hipStream_t s)
{
    const PackJob j = pack_job(w, w2, n, k, ld, packed, 0, 1);
    return launch_pack_weights(&j, 1, s);
}

hipError_t launch_pack_act(const float *x, int b, int k, uint4 *hi, uint4 *lo, hipStream_t s)
{
    if (b <= 0) return hipSuccess;
    const int64_t n = (int64_t)b * (k / 8);
    pack_act_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(x, b, k, k / 32, hi, lo);
    return hipGetLastError();
}

hipError_t launch_rmsnorm_pack(const float *x, const uint16_t *g, int b, int h, float eps, uint4 *hi, uint4 *lo,
                               hipStream_t s)
{
    if (b <= 0) return hipSuccess;
    rmsnorm_pack_kernel<<<(unsigned)((b + kPackRows - 1) / kPackRows), kPackThreads, 0, s>>>(x, g, b, h, h / 32, eps, hi, lo);
    return hipGetLastError();
}

}  // namespace pat
