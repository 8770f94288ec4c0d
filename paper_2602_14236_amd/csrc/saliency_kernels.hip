// Saliency map (Canny edges + LAB colour variance) and patch pooling for gfx950.
//
// Spatial Filtering via Saliency-Guided Quantization (saliency map S, Eq. 7) and
// Implementation Details (Canny edge detection combined with adaptive thresholding on the
// local colour variance in LAB).  Everything here is integer arithmetic, so scores are exact.
//
//   k_prep   one pass over the RGB frame, 32x32 tiles with a 4-pixel halo staged in LDS (colour
//            tables held in LDS too):
//            gray -> 5x5 binomial blur -> Sobel -> non-maximum suppression
//            -> weak/strong class, and RGB -> 8-bit LAB -> 5x5 variance sum V, plus the frame
//            sum of V (one 64-bit atomic per block).
//            8-connected hysteresis is a lock-free union-find over weak/strong pixels.  A
//            pixel's key is its index with bit 31 set for weak pixels; links always point to
//            the smaller key, so a walk along links meets a strong key iff the component has one.
//            k_prep joins the components of its own tile in LDS (label equivalence, no
//            global traffic) and writes each pixel's link to a strong pixel of its tile's part
//            or, without one, to that part's root.
//   k_union  carries "has a strong pixel" across tile borders with global atomics (border pixels only).
//   k_pool   per patch: E = edge pixel whose component is strong, C = V above the frame mean and
//            above a floor; q = sum(E + C); score = floor(q * 2^15 / |P|) / 65536.  In the
//            chained step it also reduces the flow field to the patch's motion (Eq. 5).
//   k_pool_tail  one block per frame: the gate (Eq. 6) and the ranking of the frame's tokens; the
//            last of them to finish writes the frame-table rows in video order.
//
// Every kernel takes the frame as a grid dimension (per-frame pointers in a by-value struct): one
// small frame cannot fill 256 compute units.
//
// All stencils replicate the border; non-maximum suppression treats out-of-image neighbours
// as magnitude 0.

#include "sali_internal.h"
#include "saliency_body.h"
#include "tier_body.h"

namespace sali {

// gray only, blockIdx.y = frame of the batch: what the flow needs of a frame with a single, large level (elsewhere the
// kernels that read gray values convert them).  Sixteen pixels per thread (48 bytes in, 16 out) where
// the caller's image is 16-byte aligned, else pixel by pixel.
__global__ __launch_bounds__(256) void k_gray(int n, PrepBatch f) {
    const uint8_t* __restrict__ rgb = f.frame[blockIdx.y].rgb;
    uint8_t* __restrict__ y8 = f.frame[blockIdx.y].y8;
    const int i0 = (blockIdx.x * 256 + threadIdx.x) * 16;
    if (i0 >= n) return;
    if (i0 + 16 <= n && (reinterpret_cast<uintptr_t>(rgb) & 15u) == 0) {
        const uint4* src = reinterpret_cast<const uint4*>(rgb + (size_t)i0 * 3);
        const uint4 a = src[0], b = src[1], c = src[2];
        const uint32_t in[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
        uint32_t out[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            out[q] = gray_of_quad(in + 3 * q);
        }
        *reinterpret_cast<uint4*>(y8 + i0) = make_uint4(out[0], out[1], out[2], out[3]);   // lane scratch: 256-byte aligned
        return;
    }
    for (int i = i0; i < n && i < i0 + 16; ++i) {
        const uint8_t* px = rgb + (size_t)i * 3;
        y8[i] = (uint8_t)gray_of(px[0], px[1], px[2]);
    }
}

template <bool kGated, int NT>
__global__ __launch_bounds__(NT) void k_prep(const uint32_t* __restrict__ lut_words, int h, int w, int lo2, int hi2, GateParams gp,
                                             PrepBatch f) {
    // blockIdx.z = frame of the batch
    __shared__ PrepShared sh;
    prep_tile<kGated, NT>(sh, f, (int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, h, w, gp, lut_words, lo2, hi2);
}

// hysteresis, cross-tile part; blockIdx.y = frame of the batch.  A thread per border pixel: with a thread per
// image pixel, nearly all of them idle, and walks to the root also between strong components sixteen 640x360
// frames took 44 us in the pipeline, one frame alone 16.8; then 23.5 and 10.4 (chains of trips past the L2), and 9.2 alone since the
// frame's skip flag is asked for with an item's first loads instead of ahead of them.
// kGated: the pre-pass ran ahead of the flow and could not ask the reuse rule; it is evaluated here, from the motions.
template <bool kGated>
__global__ __launch_bounds__(256) void k_union(int h, int w, int n_items, GateParams gp, PrepBatch f) {
    if constexpr (kGated) {
        __shared__ int s_cnt[4];
        if (frame_redundant<256>(f.frame, (int)blockIdx.y, gp, s_cnt)) return;
    }
    const PrepFrame& frame = f.frame[blockIdx.y];
    together(frame.skip, frame.cls, frame.parent);
    union_item(frame, h, w, (int)(blockIdx.x * 256 + threadIdx.x), n_items,
               [&] { return !kGated && *frame.skip != 0u; });       // redundant frame, says the pre-pass
}

// Gate (Eq. 6), tier assignment and compaction indices of frame `b` of a launch of `n_frames`, by
// one block of 256 threads, after every patch score and patch motion of the frame has been written:
// n_static = #{dP_i < tau_t}, R = n_static / 576, redundant iff R > theta_R; a frame without
// predecessor (no flow) is never redundant.  The last such block of the launch (arrival counter,
// nobody waits) writes the frame-table rows and advances the pool cursors in video order.
// Bound by the trips of a single chain: arguments, scores and motions, ranking, hand-over, rows.  The hand-over records are written and
// read past the caches that the compute dies do not share and a block counts itself in when its own has arrived, so it needs no
// device-scope fence (two of them, an L2 written back and one given up).
__device__ __forceinline__ void pool_tail(TierShared& sh, int* s_cnt, const PoolBatch& f, int b, int n_frames,
                                          float tau_t, float theta_r, const TierLaunch& tl, uint32_t* batch_done) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // gate: n_static = #{dP_i < tau_t}, R = n_static / 576, redundant iff R > theta_R; a frame
    // without predecessor (no flow) is never redundant
    const PoolFrame& frame = f.frame[b];
    const float* const scores_of = frame.scores;
    const float* const dp = frame.dp;
    const bool have_flow = frame.flow != nullptr;
    together(scores_of, dp, frame.flow, frame.gate, frame.tcounts);
    // the scores are asked for now, with the patch motions: one memory round trip instead of two on the
    // critical path of the batch (a redundant frame does not use them)
    const TierScores scores = tier_load_scores(scores_of);
    CursorRegs cr = {};                 // of the block that turns out to be the last: nobody else moves them
    if (threadIdx.x == 0) cr = cursor_load(tl.cur);
    // a tiled frame's patches are those of all its tiles (entries b0 .. b0 + tiles - 1 of the launch): the
    // block of every tile counts them all and so reaches the frame's one decision on its own
    const int tiles = tl.tiles;
    int n = 0;
    if (have_flow && tiles == 1) {
        n = count_static<kTierThreads>(dp, tau_t);
    } else if (have_flow) {
        const int b0 = b - b % tiles;
        for (int j = 0; j < tiles; ++j) n += count_static<kTierThreads>(f.frame[b0 + j].dp, tau_t);
    }
    for (int off = 32; off > 0; off >>= 1) n += __shfl_down(n, off);
    if (lane == 0) s_cnt[wave] = n;
    __syncthreads();
    const int n_static = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    const float r = (float)n_static / (float)(kTokens * tiles);
    const bool redundant = have_flow && r > theta_r;
    TierCounts tc = {};
    tc.state = 1;
    if (!redundant)
        tc = tier_rank(sh, scores, tl.tp, tl.tier + (size_t)b * kTokens, tl.slot + (size_t)b * kTokens,
                       tl.order + (size_t)b * kTokens);
    __syncthreads();
    if (threadIdx.x == 0) {
        sali_gate gt;
        gt.n_static = n_static;
        gt.r_frame = have_flow ? r : 0.0f;
        gt.redundant = redundant ? 1 : 0;
        gt.reserved = 0;
        *frame.gate = gt;
        bool last = n_frames == 1;              // hands nothing over
        if (!last) {
            int32_t* out = reinterpret_cast<int32_t*>(frame.tcounts);
            __hip_atomic_store(out + 0, tc.state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                __hip_atomic_store(out + 1 + t, tc.cnt[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int j = 0; j < 3; ++j)
                __hip_atomic_store(out + 5 + j, tc.q[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the record has arrived
            last = __hip_atomic_fetch_add(batch_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)n_frames - 1u;
            if (last) __hip_atomic_store(batch_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_cnt[0] = last ? 1 : 0;
    }
    __syncthreads();
    if (s_cnt[0] == 0) return;
    if (tl.tp.mode != 2) {
        // every hand-over record by a thread of its own (one round trip), then the rows by one thread with
        // the cursors in registers; the loop is kept rolled: sixteen copies of the commit step are more
        // code than this one wave should have to fetch
        TierCounts* all = reinterpret_cast<TierCounts*>(&sh);
        static_assert(sizeof(TierCounts) * kMaxBatch <= sizeof(TierShared), "records fit the ranking's memory");
        if (n_frames == 1) {
            if (threadIdx.x == 0) all[0] = tc;
        } else if ((int)threadIdx.x < n_frames) {
            const int32_t* in = reinterpret_cast<const int32_t*>(f.frame[threadIdx.x].tcounts);
            TierCounts rec = {};
            rec.state = __hip_atomic_load(in + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int t = 0; t < 4; ++t) rec.cnt[t] = __hip_atomic_load(in + 1 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            all[threadIdx.x] = rec;
        }
        __syncthreads();
        if (threadIdx.x != 0) return;
#pragma unroll 1
        for (int i = 0; i < n_frames; ++i)
            tier_commit_one(all[i], tl.frame_id + i, tl.rows, cr, tl.cap16, tl.cap8, tl.cap4, tl.cur, tl.budget,
                            tl.tiles);
        cursor_store(tl.cur, cr);
        return;
    }
    // Adaptive thresholds: the ranking above gave each frame's quantiles; its tiers depend on the
    // thresholds the frame before it left, so this block assigns them frame by frame (576 compares and
    // the compaction indices per frame, the whole block) and thread 0 commits and moves the thresholds.
    if (threadIdx.x < 3) sh.tau[threadIdx.x] = tl.cur->adapt_tau[threadIdx.x];
    __syncthreads();
    for (int i = 0; i < n_frames; ++i) {
        // the frame's hand-over record, the same words for every thread; a frame by itself is the block's own
        TierCounts tci = {};
        int q[3];
        if (n_frames == 1) {
            tci.state = tc.state;
#pragma unroll
            for (int j = 0; j < 3; ++j) q[j] = tc.q[j];
        } else {
            const int32_t* in = reinterpret_cast<const int32_t*>(f.frame[i].tcounts);
            tci.state = __hip_atomic_load(in + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int j = 0; j < 3; ++j) q[j] = __hip_atomic_load(in + 5 + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const bool ranked = tci.state == 3;
        if (ranked)
            tci = tier_assign_adaptive(sh, tier_load_scores(f.frame[i].scores), tl.tier + (size_t)i * kTokens,
                                       tl.slot + (size_t)i * kTokens, tl.order + (size_t)i * kTokens);
        __syncthreads();
        if (threadIdx.x == 0) {
            const bool stored = tier_commit_one(tci, tl.frame_id + i, tl.rows, cr, tl.cap16, tl.cap8, tl.cap4, tl.cur,
                                                tl.budget, tl.tiles);
            if (ranked && stored) tier_adapt_update(sh, q, tl.tp.adapt_q8);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        cursor_store(tl.cur, cr);
#pragma unroll
        for (int j = 0; j < 3; ++j) tl.cur->adapt_tau[j] = sh.tau[j];
    }
}

// Eq. 5 motion (kMotion) or Eq. 7 score (!kMotion) of each patch.  kWaves = 1: one wave per patch, four
// patches per block of 256 threads (small patches); kWaves = 4: the whole block works on one patch (large
// frames).  The chained step launches the motion variant after the flow and the score variant after the
// saliency pre-pass; a frame that the reuse rule finds redundant gets no scores (Algorithm 1).
// The gate and the tiers (pool_tail) are a further, small launch.  Doing them in the last block of a
// frame to finish (arrival counter) saves that launch but needs a device-scope fence per block, and
// such a fence writes back and invalidates the issuing XCD's L2: with 144 blocks per frame it made the
// K/V kernels running next to it 7 % slower (5 400 -> 5 700 frames/s without), and at 1920x1080 (576
// blocks per frame) it cost the pooling kernel itself 110 us per four-frame launch against 33 us of work.
// Bound by trips to memory, then (large frames) by the adds on each patch's many pixels: see PatchPixels and patch_sum.  Sixteen 640x360
// frames 27.8 -> 15.2 us in the pipeline, motions of four 1920x1080 frames 12.8 -> 11.9.
// kGated: as in k_union.
template <int kWaves, bool kMotion, bool kGated>
__global__ __launch_bounds__(kTierThreads) void k_pool(uint8_t* __restrict__ salmap, int h, int w, GateParams gp, PoolBatch f) {
    static_assert(kTierThreads == 256, "four waves, one patch each");
    static_assert(kWaves == 1 || kWaves == 4, "");
    const int b = blockIdx.y;                               // frame of the batch
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int token = kWaves == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
    const int p_first = kWaves == 1 ? lane : (int)threadIdx.x;
    constexpr int kStride = 64 * kWaves;
    if constexpr (!kMotion) {
        __shared__ uint32_t s_pq[kTierThreads / 64];
        const PoolFrame& frame = f.frame[b];
        if constexpr (kGated) {
            __shared__ int s_cnt[kTierThreads / 64];
            if (frame_redundant<kTierThreads>(f.frame, b, gp, s_cnt)) return;
        }
        auto stop = [&] { return !kGated && *frame.skip != 0u; };       // redundant frame, says the pre-pass
        if constexpr (kWaves == 1) {
            score_by_wave(frame, token, h, w, salmap, stop);
        } else {
            const PatchBox box = patch_box(token, h, w);
            uint32_t q = patch_sum<kStride>(frame, box, p_first, h, w, salmap, stop);
            if (q == kNoSum) return;
            for (int off = 32; off > 0; off >>= 1) q += __shfl_down(q, off);
            if (lane == 0) s_pq[wave] = q;
            __syncthreads();
            if (threadIdx.x == 0) store_score(frame, token, s_pq[0] + s_pq[1] + s_pq[2] + s_pq[3], box.area);
        }
    } else {
        __shared__ float s_pm[kTierThreads / 64];
        const float2* __restrict__ flow = f.frame[b].flow;
        float* dp_out = f.frame[b].dp_out;
        together(flow, dp_out);
        if (flow == nullptr) {                              // no predecessor: no motion
            if (lane == 0 && (kWaves == 1 || wave == 0))
                __hip_atomic_store(dp_out + token, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        const PatchBox box = patch_box(token, h, w);
        const PatchPixels pixel(box, w);
        float mag = 0.0f;
        constexpr int kUnroll = 4;                          // four pixels per pass, their loads issued together
        for (int p0 = p_first; p0 < box.area; p0 += kStride * kUnroll) {
            float2 d[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) d[u] = ld_at(flow, pixel(min(p0 + u * kStride, box.area - 1)));
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (p0 + u * kStride < box.area) mag += d[u].x * d[u].x + d[u].y * d[u].y;
        }
        for (int off = 32; off > 0; off >>= 1) mag += __shfl_down(mag, off);
        if constexpr (kWaves == 4) {
            if (lane == 0) s_pm[wave] = mag;
            __syncthreads();
            mag = (s_pm[0] + s_pm[1]) + (s_pm[2] + s_pm[3]);
        }
        if (lane == 0 && (kWaves == 1 || wave == 0))
            __hip_atomic_store(dp_out + token, sqrtf(mag / (float)box.area), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// the tail as a launch of its own: one block per frame.  A kernel per tier mode and with or without a budget: a few blocks run this code
// once, after kernels that left nothing of it in the instruction caches.  Of one kernel for all (scratch for the budget's call, scalar
// registers spilled) with fences at the hand-over one frame by thresholds took 4.1 us and takes 2.8; by counts four took 14.5 and take 13.2,
// sixteen 19.0 and 16.2.
template <int kMode, bool kBudget>
__global__ __launch_bounds__(kTierThreads) void k_pool_tail(uint32_t* batch_done, float tau_t, float theta_r, TierLaunch tl,
                                                            PoolBatch f) {
    __shared__ TierShared sh;
    __shared__ int s_cnt[kTierThreads / 64];
    tl.tp.mode = kMode;
    if constexpr (!kBudget) tl.budget = 0;
    pool_tail(sh, s_cnt, f, (int)blockIdx.x, (int)gridDim.x, tau_t, theta_r, tl, batch_done);
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_gray(const PrepBatch& f, int n, int h, int w, hipStream_t s) {
    const int px = h * w;
    hipLaunchKernelGGL(k_gray, dim3((px + 4095) / 4096, n), dim3(256), 0, s, px, f);
    return hipGetLastError();
}

hipError_t launch_prep(const PrepBatch& f, int n, int h, int w, GateParams gp, const void* d_lut,
                       int lo2, int hi2, hipStream_t s) {
    dim3 grid((w + kTile - 1) / kTile, (h + kTile - 1) / kTile, n);
    const uint32_t* lut = static_cast<const uint32_t*>(d_lut);
    bool gated = false;
    for (int i = 0; i < n; ++i) gated = gated || f.frame[i].dp != nullptr;
    // Batches (the chained step, behind its flow) on 256 threads: next to K/V kernels small blocks find room, 640x360 clips are
    // 0.5 to 1 % slower with 512.  The stand-alone call on 512, or on 1024 if every tile has a compute unit to itself: a stage of
    // 300 to 400 strips is one pass instead of two, the whole call at 640x360 37.7 -> 32.6 us (512 threads 33.2), at
    // 1920x1080 96.3 -> 92.9 (1024 threads 95.4).
    if (gated) hipLaunchKernelGGL((k_prep<true, kPrepThreads>), grid, dim3(kPrepThreads), 0, s, lut, h, w, lo2, hi2, gp, f);
    else if ((long long)grid.x * grid.y * n <= 256) hipLaunchKernelGGL((k_prep<false, 1024>), grid, dim3(1024), 0, s, lut, h, w, lo2, hi2, gp, f);
    else hipLaunchKernelGGL((k_prep<false, 512>), grid, dim3(512), 0, s, lut, h, w, lo2, hi2, gp, f);
    return hipGetLastError();
}

hipError_t launch_union(const PrepBatch& f, int n, int h, int w, const GateParams* gate_or_null, hipStream_t s) {
    const int items = border_items(h, w);
    if (items == 0) return hipSuccess;              // a single tile
    const dim3 grid((items + 255) / 256, n);
    if (gate_or_null != nullptr) hipLaunchKernelGGL(k_union<true>, grid, dim3(256), 0, s, h, w, items, *gate_or_null, f);
    else hipLaunchKernelGGL(k_union<false>, grid, dim3(256), 0, s, h, w, items, GateParams{}, f);
    return hipGetLastError();
}

namespace {
// patches of up to 1024 pixels: one wave each
template <bool kMotion, bool kGated>
hipError_t launch_patches(const PoolBatch& f, int n, int h, int w, uint8_t* d_salmap, const GateParams& gp, hipStream_t s) {
    if ((long long)h * w <= 1024ll * kTokens)
        hipLaunchKernelGGL((k_pool<1, kMotion, kGated>), dim3(kTokens / 4, n), dim3(kTierThreads), 0, s, d_salmap, h, w, gp, f);
    else
        hipLaunchKernelGGL((k_pool<4, kMotion, kGated>), dim3(kTokens, n), dim3(kTierThreads), 0, s, d_salmap, h, w, gp, f);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_motion(const PoolBatch& f, int n, int h, int w, hipStream_t s) {
    return launch_patches<true, false>(f, n, h, w, nullptr, GateParams{}, s);
}

hipError_t launch_scores(const PoolBatch& f, int n, int h, int w, uint8_t* d_salmap_or_null, const GateParams* gate_or_null,
                         hipStream_t s) {
    return gate_or_null != nullptr ? launch_patches<false, true>(f, n, h, w, d_salmap_or_null, *gate_or_null, s)
                                   : launch_patches<false, false>(f, n, h, w, d_salmap_or_null, GateParams{}, s);
}

hipError_t launch_tail(const PoolBatch& f, int n, const TierLaunch& tier, GateParams gp, uint32_t* d_done_counter,
                       hipEvent_t done_or_null, hipStream_t s) {
    const bool budget = tier.budget > 0;
    auto* const kernel = tier.tp.mode == 0 ? (budget ? k_pool_tail<0, true> : k_pool_tail<0, false>)
                         : tier.tp.mode == 1 ? (budget ? k_pool_tail<1, true> : k_pool_tail<1, false>)
                                             : (budget ? k_pool_tail<2, true> : k_pool_tail<2, false>);
    launch_recording(done_or_null, kernel, dim3(n), dim3(kTierThreads), s, d_done_counter, gp.tau_t, gp.theta_r, tier, f);
    return hipGetLastError();
}

}  // namespace sali
