// Internal declarations shared by the host API and the kernel files of libsali.
// gfx950 only; wave size 64.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "arith.h"
#include "sali.h"

namespace sali {

constexpr int kGrid = 24;
constexpr int kTokens = kGrid * kGrid;      // 576 visual tokens per frame
constexpr int kHeadDim = 128;
constexpr int kGroup = 32;                  // quantisation group along head_dim
constexpr int kGroupsPerRow = kHeadDim / kGroup;
constexpr int kMaxLevels = 6;
constexpr int kMaxIters = 8;
constexpr int kAttnMaxQPerKv = 8;           // query heads that may share one K/V head
constexpr int kAttnSlotsPerHead = 4096;     // partial-result slots of the scratch per K/V head (shared out over its queries)
constexpr int kAttnSets = 2;                // at most so many blocks share a K/V head's rows with different queries
constexpr int kAttnPartialStride = 160;     // floats per partial: max, sum, 128 values; 640 B = five whole 128-byte lines
constexpr int kMaxBatch = SALI_MAX_BATCH;   // frames analysed by one set of launches (blockIdx.z / .y)
constexpr int kMaxTiles = 8;                // images per video frame (a frame's tiles are analysed in one batch)

// flow constants (polynomial expansion 7x7 sigma 1.5; aggregation window 11x11 sigma 2.5;
// prior-centred ridge term lambda = kLamAbs + kLamRel * trace(G) / 2)
constexpr int kPolyN = 3;
constexpr float kPolySigma = 1.5f;
constexpr int kWinR = 5;
constexpr float kWinSigma = 2.5f;
constexpr float kLamAbs = 1e-4f;
constexpr float kLamRel = 1e-2f;

// colour tables, in this order: sRGB decoding [256] and companding [4096], 16-bit each, then the L byte [4096]
// of every argument of the companding
constexpr int kColourLutBytes = (256 + 4096) * 2 + 4096;

constexpr uint32_t kVMin = 10000u;          // floor of the colour-variance mask

// Device-resident bookkeeping (lives in the caller's table buffer).
// Memory-budget mode: the frames still held form a queue (oldest first) and each pool is a ring.
// The rows of the held frames of a pool are the cyclic window tail .. head (head = the pool's cursor);
// `wrapped` says that the window passes the end of the pool, in which case the rows before the wrap
// end at `end` (the cursor's value when a frame did not fit behind it and went to row 0).
struct RingState {
    int32_t oldest;             // oldest stored frame still held, -1 = none
    int32_t live_tokens;        // kept tokens of the held frames
    int32_t tail[3], end[3], live_rows[3], wrapped[3];
};

struct Cursors {
    int32_t c16, c8, c4;        // next free row of each pool
    int32_t last_src;           // frame id of the last stored frame, -1 = none
    uint32_t status;            // sticky SALI_FAULT_* bits
    uint32_t pad[3];
    RingState ring;             // used with a memory budget only
    int32_t last_src_tile[kMaxTiles];   // tiled frames: last stored entry of each tile, -1 = none
    int32_t adapt_tau[3];       // adaptive thresholds in force (tier_mode 2), units of 2^-16
    uint32_t pad2[3];
};

// The six pool arrays.  Layout of each: frame-major.  A stored frame with first row `base` and
// `n` rows in a pool owns rows [base * n_planes, (base + n) * n_planes) of the flat array, and inside
// that run plane p (layer, K|V, head) owns rows [p * n, (p + 1) * n): everything one frame writes
// to a pool is one contiguous range, whatever the capacity (with one big [plane][cap] array per
// pool a frame touched n_planes ranges megabytes apart, which cost the pack kernel 8-16 % of its
// bandwidth).
struct Pools {
    uint16_t* p16;              // fp16 bit patterns
    int8_t* c8;
    float* s8;
    uint8_t* c4;
    float* s4;
    uint16_t* z4;
    int32_t cap16, cap8, cap4;
    int32_t n_planes;
};

// first flat row of plane `plane` of a frame whose run starts at `base` and has `n` rows per plane
__host__ __device__ inline size_t pool_row0(const Pools& p, int base, int n, size_t plane) {
    return (size_t)base * (size_t)p.n_planes + plane * (size_t)n;
}

struct TierParams {
    int32_t mode;               // 0: Eq. 8 thresholds, 1: top-k counts, 2: adaptive thresholds (k = target counts)
    float tau_high, tau_med, tau_low;
    int32_t k16, k8, k4;
    int32_t adapt_q8;           // mode 2: step of the threshold update in 1/256
};

// everything the tier / compaction step needs when it is fused into another kernel; in a batched
// launch frame i of the batch has id frame_id + i and its tables follow at i * kTokens
struct TierLaunch {
    TierParams tp;
    int32_t frame_id;
    sali_frame_row* rows;
    uint8_t* tier;
    uint16_t* slot;
    uint16_t* order;
    Cursors* cur;
    int32_t cap16, cap8, cap4;
    int32_t budget;             // most tokens the cache may hold, 0 = no budget
    int32_t tiles;              // images per video frame (entries per frame), >= 1
};

struct LevelGeom {
    int32_t h[kMaxLevels];
    int32_t w[kMaxLevels];
    int64_t off[kMaxLevels];    // pixel offset of the level inside a concatenated per-level array
    int32_t tiles_x[kMaxLevels];
    int32_t tile_start[kMaxLevels + 1];   // first block index of each level in a fused launch
    int32_t levels;
};

// Per-frame operands of the batched image kernels: entry i belongs to frame i of the batch.  A frame's pointers lie side by
// side, so that a block finds its own in one or two cache lines of the kernel's arguments.
struct PrepFrame {
    const uint8_t* rgb;
    uint8_t* y8;
    uint8_t* cls;
    uint32_t* var;
    uint32_t* parent;
    unsigned long long* msum_acc;      // frame sum of the colour variance, accumulated
    unsigned long long* msum_clear;    // the accumulator of the lane's next use, cleared
    const float* dp;                   // the frame's per-patch motions, for the reuse rule; NULL: never redundant
    uint32_t* skip;                    // the pre-pass leaves the rule's answer here (1: redundant, no saliency)
};
struct PrepBatch {
    PrepFrame frame[kMaxBatch];
};

// The reuse rule (Eq. 6, R_frame > theta_R) as the kernels that come after the flow evaluate it for
// themselves: tiles = images per video frame (their patches count together).
struct GateParams {
    float tau_t, theta_r;
    int32_t tiles;
};

// A polynomial expansion is stored as 20 bytes per pixel and level: Ab = {A_xx, A_xy, A_yy, b_x} and
// by = b_y (a float4 for A plus a float2 for b would be 24, a fifth of it padding, and the flow
// updates re-read both frames' expansions once per update: at 1920x1080 that is most of the image
// side's HBM traffic).
struct ExpandFrame {
    const uint8_t* rgb;
    float4* A;
    float* b;
};
struct ExpandBatch {
    ExpandFrame frame[kMaxBatch];
};

struct PyrFrame {                                 // per-level path (more than three levels, larger frames)
    const uint8_t* rgb;
    uint8_t* y8;
    float* pyr;                                   // all levels of the frame's pyramid, LevelGeom offsets
    float4* A;
    float* b;
};
struct PyrBatch {
    PyrFrame frame[kMaxBatch];
};

struct FlowFrame {                                // expansions at level 0; the launcher adds the level offset
    const float4* A1;
    const float4* A2;
    const float* b1;
    const float* b2;
    const float2* d_in;
    float2* d_out;
};
struct FlowBatch {
    FlowFrame frame[kMaxBatch];
};

struct PoolFrame {
    const uint8_t* cls;
    const uint32_t* parent;
    const uint32_t* var;
    const unsigned long long* msum;
    float* scores;
    const float2* flow;                           // NULL: no predecessor (never redundant)
    float* dp_out;                                // per-patch motion, written by the motion launch
    const float* dp;                              // the same for the reuse rule; NULL: never redundant
    const uint32_t* skip;                         // what the pre-pass found (1: redundant, no scores)
    sali_gate* gate;
    struct TierCounts* tcounts;                   // hand-over from the frame's ranking to the row writer
};
struct PoolBatch {
    PoolFrame frame[kMaxBatch];
};

// Work of the spatial filter that rides on launches of the temporal filter: extra blocks of theirs.
struct NoRide {};
struct PrepRide {                                 // the pre-pass, on the launch that makes the expansions or a flow update
    int32_t blocks, h, w, tiles_x, tiles_y, lo2, hi2;
    const uint32_t* lut;
    PrepBatch f;
};
struct UnionRide {                                // hysteresis across tiles, on a flow update after it
    int32_t blocks, h, w, n_items, blocks_per_frame;
    PrepBatch f;
};
struct ScoreRide {                                // patch scores, on an update after that
    int32_t blocks, h, w, blocks_per_frame;
    PoolBatch f;
};
// a piece of the spatial filter that a flow launch is asked to carry
enum class FlowRider { none, prepass, hysteresis, scores };
struct FlowRiders {
    const PrepRide* prep;
    const PoolBatch* pool;
    int n, h, w;                                  // frames, their size
};

struct KvBatch {
    void* kv[kMaxBatch];
};

struct FlowWeights {
    float poly_g[2 * kPolyN + 1];    // normalised Gaussian of the expansion
    float win_g[2 * kWinR + 1];      // normalised Gaussian of the aggregation window
    float inv_m2;                    // 1 / m2
    float inv_den;                   // 1 / (m4 - m2^2)
    float inv_2m2sq;                 // 1 / (2 m2^2)
    float m2;
};

// XCD-aware block order.  The hardware deals the workgroups of a launch round-robin to the 8 XCDs
// in linear-id order (x fastest), and every XCD has an L2 of its own: with the plain order
// neighbouring tiles land on different XCDs and every L2 ends up holding every frame.  This maps
// the hardware id to a logical (x, y, z) such that each XCD works through one contiguous run of the
// (z, y, x) order: tiles that share halos share an L2, and an L2 holds an eighth of the data.  Large frames are cut into eight
// runs each instead (gz = 0) and so go one after the other.  More tiles then have neighbours elsewhere and the halos are fetched again (a flow
// update of three 1920x1080 frames by itself reads 359 MB, not 330, of three 960x540 92, not 82), but the expansion that two flows share is still
// in the last-level cache, and that counts for more: the analysis of four 1920x1080 frames 790 -> 773 us, of eight 960x540 421 -> 416, of four
// 883x1327 with two levels 416 -> 401.  Smaller frames: 15 x 320x180 4 % slower, 15 x 640x360 (240 tiles) the same.
// The grid comes as arguments: the leading ones are in registers when a block starts, the launch's own record is not.
struct BlockId {
    int x, y, z;
};
constexpr int kTilesOwnRuns = 480;
inline int frames_sharing_runs(int tiles_x, int tiles_y, int n) { return tiles_x * tiles_y >= kTilesOwnRuns ? 0 : n; }
#ifdef __HIPCC__
__device__ __forceinline__ BlockId xcd_block_id(int linear, int gx, int gy, int gz) {
    constexpr uint32_t kXcds = 8;
    const uint32_t plane = (uint32_t)(gx * gy), total = plane * (uint32_t)gz;
    const uint32_t q = total / kXcds, r = total % kXcds;
    const uint32_t xcd = (uint32_t)linear % kXcds, slot = (uint32_t)linear / kXcds;
    const uint32_t logical = xcd * q + (xcd < r ? xcd : r) + slot;      // XCDs 0..r-1 hold q + 1 blocks
    const uint32_t z = gz == 1 ? 0u : logical / plane, rem = logical - z * plane;
    const uint32_t y = rem / (uint32_t)gx;
    return {(int)(rem - y * (uint32_t)gx), (int)y, (int)z};
}
__device__ __forceinline__ BlockId xcd_block_id(int gx, int gy, int gz) {
    const int in_frame = (int)blockIdx.x + gx * (int)blockIdx.y;
    if (gz > 0) return xcd_block_id(in_frame + gx * gy * (int)blockIdx.z, gx, gy, gz);
    const BlockId b = xcd_block_id(in_frame, gx, gy, 1);
    return {b.x, b.y, (int)blockIdx.z};
}

// What a block needs of its kernel's arguments is asked for at once: an empty use of all of it, ahead of the work.  Left to the
// compiler the pieces are loaded where they are needed first, one trip of the scalar cache behind the other (a miss each:
// arguments come from memory), and five or six such trips were 1.5 us of a launch of 5 to 12.
__device__ __forceinline__ void together() {}
template <typename T, typename... Rest>
__device__ __forceinline__ void together(const T& first, const Rest&... rest) {
    asm volatile("" : : "s"(first));
    together(rest...);
}
#endif

#ifdef __HIPCC__
// Element i of an array whose base is uniform over the wave: base + 32-bit byte offset (an image level
// has fewer than 2^28 pixels, so i * 16 fits), which the hardware adds itself; with 64-bit indices a
// quarter of the gather's vector instructions were address arithmetic.
template <typename V>
__device__ __forceinline__ V ld_at(const V* __restrict__ base, uint32_t i) {
    return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(V));
}
__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Y8 of one pixel, and of four pixels in three words (bytes RGBR GBRG BRGB)
__device__ __forceinline__ uint32_t gray_of(uint32_t r, uint32_t g, uint32_t b) {
    return (77u * r + 150u * g + 29u * b + 128u) >> 8;
}
__device__ __forceinline__ uint32_t gray_of_quad(const uint32_t* w) {
    const uint32_t g0 = gray_of(w[0] & 0xFF, (w[0] >> 8) & 0xFF, (w[0] >> 16) & 0xFF);
    const uint32_t g1 = gray_of(w[0] >> 24, w[1] & 0xFF, (w[1] >> 8) & 0xFF);
    const uint32_t g2 = gray_of((w[1] >> 16) & 0xFF, w[1] >> 24, w[2] & 0xFF);
    const uint32_t g3 = gray_of((w[2] >> 8) & 0xFF, (w[2] >> 16) & 0xFF, w[2] >> 24);
    return g0 | (g1 << 8) | (g2 << 16) | (g3 << 24);
}
// the four pixels from column x of an image row of w pixels, coordinates clamped: twelve bytes at any address, as one load
// where they lie inside the row
__device__ __forceinline__ void load_rgb_quad(const uint8_t* __restrict__ row, int x, int w, uint32_t (&v)[3]) {
    if (x >= 0 && x + 3 < w) {
        __builtin_memcpy(v, row + 3 * x, 12);
    } else {
        uint32_t c[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) c[i] = row[3 * clampi(x + i / 3, 0, w - 1) + i % 3];
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = c[4 * i] | (c[4 * i + 1] << 8) | (c[4 * i + 2] << 16) | (c[4 * i + 3] << 24);
    }
}
#endif

// A launch that records `done` (may be NULL) when it has run.  The event rides on the launch's own completion signal:
// recorded by a call of its own it is a packet of its own on the stream, and the next kernel starts 5 us later.
template <typename... Params, typename... Args>
inline void launch_recording(hipEvent_t done, void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t s, Args... args) {
    if (done != nullptr) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, nullptr, done, 0, static_cast<Params>(args)...);
    else hipLaunchKernelGGL(kernel, grid, block, 0, s, static_cast<Params>(args)...);
}

// ---- launchers (each returns hipGetLastError()) ---------------------------------------------
// kv_kernels.hip
hipError_t launch_tier(const float* d_scores, const sali_gate* d_gate_or_null, TierParams tp, int frame_id,
                       sali_frame_row* d_rows, uint8_t* d_tier, uint16_t* d_slot, uint16_t* d_order,
                       Cursors* d_cur, Pools pools, int budget, int tiles, hipStream_t s);
// frame i of a batched launch has id first_frame_id + i; f.kv[i] is its dense fp16 K/V (source of
// the pack, destination of the unpack)
hipError_t launch_pack(const KvBatch& f, int n, const sali_frame_row* d_rows, int first_frame_id,
                       const uint16_t* d_order_base, Pools pools, Cursors* d_cur, int n_planes, hipStream_t s);
hipError_t launch_unpack(const sali_frame_row* d_rows, int first_frame_id, const uint16_t* d_order_base, Pools pools,
                         const KvBatch& out, int n, uint8_t* d_valid_or_null, Cursors* d_cur, int n_planes,
                         hipStream_t s);

struct RowsPerFrame {
    int n16, n8, n4;
};
// results of an attention call, and the arrival counters of its blocks (arrival_counter of kAttnSets per K/V head; zero between calls)
inline size_t arrival_words(int n_heads) { return (size_t)n_heads * kAttnSets * kAttnPartials; }
struct AttnOut {
    float* out;
    float* lse;                 // may be NULL
    uint32_t* arrived;
};
// attn_kernels.hip: single-query attention of one layer over frames [frame_lo, frame_hi) for
// n_heads * q_per_kv queries (q_per_kv in {1, 2, 4, 8}: streaming kernel; 9 .. 64: matrix-core kernel); d_partial holds
// n_heads * kAttnSlotsPerHead * kAttnPartialStride floats; tiles = cache entries per video frame (an entry's pointer
// entries lie that far apart); kept = how many rows a stored frame is
// expected to keep (it shapes the launch, any frame is read whole); the events (may be NULL) bracket
// the main kernel
hipError_t launch_attend(const sali_frame_row* d_rows, const Pools& pools, int layer, int n_heads, int q_per_kv,
                         const void* d_q, int frame_lo, int frame_hi, int tiles, RowsPerFrame kept, float softmax_scale, float* d_partial,
                         AttnOut result, hipEvent_t ev_start, hipEvent_t ev_stop, hipStream_t s);

// saliency_kernels.hip
// n = frames in the batch (1..kMaxBatch).  launch_gray: RGB -> gray only.  launch_prep: the edge / colour
// variance pre-pass; frames that the reuse rule finds redundant from
// f.dp are skipped (Algorithm 1: their saliency is not computed) and marked in f.skip, which launch_union
// and launch_scores go by.  With a gate these two evaluate the rule from f.dp themselves (behind a pre-pass that ran
// ahead of the flow).
hipError_t launch_gray(const PrepBatch& f, int n, int h, int w, hipStream_t s);
hipError_t launch_prep(const PrepBatch& f, int n, int h, int w, GateParams gp, const void* d_lut,
                       int lo2, int hi2, hipStream_t s);
hipError_t launch_union(const PrepBatch& f, int n, int h, int w, const GateParams* gate_or_null, hipStream_t s);
// launch_motion: Eq. 5, per-patch motion of every frame of the batch from its flow (0 without flow).
// launch_scores: Eq. 7 scores (none for redundant frames); d_salmap_or_null applies to frame 0 (stand-alone call).
// launch_tail: evaluates the gate and assigns tiers for the n frames in order, and records done_or_null.
hipError_t launch_motion(const PoolBatch& f, int n, int h, int w, hipStream_t s);
hipError_t launch_scores(const PoolBatch& f, int n, int h, int w, uint8_t* d_salmap_or_null, const GateParams* gate_or_null,
                         hipStream_t s);
hipError_t launch_tail(const PoolBatch& f, int n, const TierLaunch& tier, GateParams gp, uint32_t* d_done_counter,
                       hipEvent_t done_or_null, hipStream_t s);

// flow_kernels.hip
// gray image and all pyramid levels (g.levels >= 2) from f.rgb
hipError_t launch_pyramid(const PyrBatch& f, int n, const LevelGeom& g, hipStream_t s);
// the launches that complete the expansions; ride_or_null rides on them, done_or_null is recorded then
hipError_t launch_polyexp(const PyrBatch& f, int n, LevelGeom g, FlowWeights fw, const PrepRide* ride_or_null, hipEvent_t done_or_null,
                          hipStream_t s);
hipError_t launch_expand(const ExpandBatch& f, int n, LevelGeom g, FlowWeights fw, const PrepRide* ride_or_null, hipEvent_t done_or_null,
                         hipStream_t s);
// one launch of at most `wanted` (>= 1) updates of a level, as many as suit its size; *done = how many it makes
hipError_t launch_flow_updates(const FlowBatch& f, int n, int64_t level_off, int h, int w, int ch, int cw,
                               int prior_mode, int wanted, int* done, const FlowWeights& fw, FlowRider rider, const FlowRiders* riders,
                               hipStream_t s);
// has the launch for `wanted` updates of an h x w level of n frames room for that piece?
bool flow_launch_carries(FlowRider rider, const FlowRiders& riders, int n, int h, int w, int wanted);
hipError_t launch_patch_gate(const float2* d_flow, int h, int w, float tau_t, float theta_r, float* d_dp,
                             sali_gate* d_gate, float* d_flow_uv_or_null, hipStream_t s);

}  // namespace sali
