// Single-query attention that reads the mixed-precision pools directly (gfx950).
//
// Just-In-Time Dequantization (entries are dequantised while attention is computed) and
// Implementation Details (the dequantisation is fused with the attention computation).  For one
// layer and every head h: s_j = softmax_scale * <q_h, K^_j>, out_h = softmax(s) V^, over the logical
// token sequence of a frame range.  "Fused" is taken literally: the dequantised values
// K^ = code * scale (INT8), code * scale + zero (INT4) never exist as an fp16 tensor, they are
// folded into the dot products in fp32 (FP16-tier rows are used as stored).  A redundant frame's
// entry is a pointer (Algorithm 1), so its source frame's tokens count once more; pruned tokens are
// not in the cache.
//
// One query per head makes Q K^T and P V matrix-vector products: 2 flops per byte read, so the
// kernel is bound by HBM and written as a stream, not for MFMA; the arithmetic is arranged so that
// the vector ALU stays below the memory time (about 5 operations per INT8 element pair instead of
// 12 when every value is first rounded to fp16: the group scale is applied once per row to the dot
// product and to the softmax weight, the INT4 zero-point through sum(q) and a separate accumulator).
// The compressed rows are read once, in pool order (attention does not care about token order),
// with the lane mapping of the pack / unpack kernels: a row is handled by 16 adjacent lanes holding
// 8 consecutive head-dim values each, a 32-value quantisation group is one lane quad, the dot
// product is reduced over the 16 lanes with four DPP moves.  Every lane group keeps an
// online-softmax state (running max, sum and 8 output values per lane); a block merges its 16 lane
// groups through LDS and writes one partial (max, sum, 128 values); a second small kernel merges
// the partials of a head.  The three tiers of a frame are walked by three instances of one loop
// specialised on the row format.  With grouped-query attention the kQ query heads that share a K/V
// head are handled by the same block, so every compressed row is still read once.

#include "sali_internal.h"

namespace sali {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int kComputeUnits = 256;
constexpr int kResidentBlocks = kComputeUnits * 8;      // compute units x blocks of the main kernel that fit on one
constexpr int kPartialStride = kAttnPartialStride;   // max, sum, 128 values, padded to whole 128-byte lines

union Row16B {
    u32x4 u;
    _Float16 h[8];
    half2_t h2[4];
};

template <int kCtrl>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kCtrl, 0xF, 0xF, true));
}

// sum over the 16 lanes of a row: lane ^ 1, lane ^ 2 inside the quad, then mirror inside 8 and
// inside 16 lanes (every lane ends with the full sum)
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp_move<0xB1>(v);       // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);       // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);      // row_half_mirror
    v += dpp_move<0x140>(v);      // row_mirror
    return v;
}

// the lane's piece of the query: 8 values as fp32 and as packed halves, and their sum
struct QueryPiece {
    float f[8];
    half2_t h2[4];
    float sum;
};

// raw piece of one pool row for one lane (16 / 8 / 4 bytes by tier) plus its group's scale and zero
template <int kTier>
struct RawRow;
template <>
struct RawRow<SALI_TIER_FP16> {
    u32x4 u;
};
template <>
struct RawRow<SALI_TIER_INT8> {
    u32x2 u;
    float scale;
};
template <>
struct RawRow<SALI_TIER_INT4> {
    uint32_t u;
    float scale, zero;
};

// frow = row index in the flat pool array of that tier (pool_row0 of the frame and plane + the row
// inside the frame's run)
__device__ __forceinline__ void load_row(const Pools& pools, size_t frow, int l, RawRow<SALI_TIER_FP16>& r) {
    r.u = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(pools.p16) + (frow * 16 + l));
}
__device__ __forceinline__ void load_row(const Pools& pools, size_t frow, int l, RawRow<SALI_TIER_INT8>& r) {
    r.u = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(pools.c8 + frow * kHeadDim) + l);
    r.scale = pools.s8[frow * kGroupsPerRow + (l >> 2)];
}
__device__ __forceinline__ void load_row(const Pools& pools, size_t frow, int l, RawRow<SALI_TIER_INT4>& r) {
    r.u = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(pools.c4 + frow * (kHeadDim / 2)) + l);
    r.scale = pools.s4[frow * kGroupsPerRow + (l >> 2)];
    r.zero = (float)__builtin_bit_cast(_Float16, pools.z4[frow * kGroupsPerRow + (l >> 2)]);
}

// The lane's 8 stored values of a row as fp32: the halves of an FP16 row, the raw codes of an
// INT8 / INT4 row (scale and zero-point are applied once per row, see finish_dot / weight_of).
__device__ __forceinline__ void row_values(const RawRow<SALI_TIER_FP16>& r, float x[8]) {
    Row16B v;
    v.u = r.u;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (float)v.h[e];
}
__device__ __forceinline__ void row_values(const RawRow<SALI_TIER_INT8>& r, float x[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t word = e < 4 ? r.u.x : r.u.y;
        x[e] = (float)(int)(int8_t)((word >> (8 * (e & 3))) & 0xFF);
    }
}
__device__ __forceinline__ void row_values(const RawRow<SALI_TIER_INT4>& r, float x[8]) {
    // nibbles to bytes first (even elements in one word, odd ones in the other): a byte converts to fp32
    // in one instruction; the empty asm keeps the compiler from folding the bytes back into nibbles
    uint32_t ev = r.u & 0x0F0F0F0Fu, od = (r.u >> 4) & 0x0F0F0F0Fu;
    asm volatile("" : "+v"(ev), "+v"(od));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = (float)((ev >> (8 * i)) & 0xFFu);
        x[2 * i + 1] = (float)((od >> (8 * i)) & 0xFFu);
    }
}

// <q, K^_row> of the lane from the sum over its raw values: K^ = code * scale (+ zero)
__device__ __forceinline__ float finish_dot(const RawRow<SALI_TIER_FP16>&, float d, const QueryPiece&) { return d; }
__device__ __forceinline__ float finish_dot(const RawRow<SALI_TIER_INT8>& r, float d, const QueryPiece&) {
    return d * r.scale;
}
__device__ __forceinline__ float finish_dot(const RawRow<SALI_TIER_INT4>& r, float d, const QueryPiece& q) {
    return d * r.scale + q.sum * r.zero;
}

// p * V^_row = (p * scale) * code + p * zero: weight on the raw values, and the constant part
__device__ __forceinline__ float weight_of(const RawRow<SALI_TIER_FP16>&, float p) { return p; }
__device__ __forceinline__ float weight_of(const RawRow<SALI_TIER_INT8>& r, float p) { return p * r.scale; }
__device__ __forceinline__ float weight_of(const RawRow<SALI_TIER_INT4>& r, float p) { return p * r.scale; }
__device__ __forceinline__ float offset_of(const RawRow<SALI_TIER_FP16>&, float) { return 0.0f; }
__device__ __forceinline__ float offset_of(const RawRow<SALI_TIER_INT8>&, float) { return 0.0f; }
__device__ __forceinline__ float offset_of(const RawRow<SALI_TIER_INT4>& r, float p) { return p * r.zero; }

// online-softmax state of a lane group for one query (max and sum are equal in its 16 lanes); the
// INT4 zero-points are summed apart (zacc, the same for the lane's 8 values) and folded in at the end
struct SoftmaxState {
    float mx, lsum, zacc;
    float acc[8];
};

// The rows of one tier of one stored frame that fall to this block: groups of 16 * kRowsPerStep rows split,
// split + n_splits, ...; lane group g takes rows jb + g, jb + 16 + g, ... (kRowsPerStep of them in flight, K
// and V each).  `base` = first pool row of the frame in this tier, `count` = its rows.  kQ queries share
// every row that is read.  Returns the split that the next tier's first group falls to, so that the groups
// of a frame's tiers go round all splits.
template <int kTier, int kQ, int kRowsPerStep>
__device__ __forceinline__ int attend_tier(const Pools& pools, size_t plane_k, size_t plane_v, int base, int count,
                                           int split, int n_splits, int g, int l, const QueryPiece (&q)[kQ],
                                           float softmax_scale, float mult, SoftmaxState (&st)[kQ]) {
    constexpr int kGroupRows = 16 * kRowsPerStep;
    if (count == 0) return split;
    const size_t row0_k = pool_row0(pools, base, count, plane_k), row0_v = pool_row0(pools, base, count, plane_v);
    for (int jb = split * kGroupRows; jb < count; jb += n_splits * kGroupRows) {
        RawRow<kTier> rk[kRowsPerStep], rv[kRowsPerStep];
        bool valid[kRowsPerStep];
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) {
            const int j = jb + r * 16 + g;
            valid[r] = j < count;
            rk[r] = {};
            rv[r] = {};
            if (valid[r]) {
                load_row(pools, row0_k + (size_t)j, l, rk[r]);
                load_row(pools, row0_v + (size_t)j, l, rv[r]);
            }
        }
        float s[kQ][kRowsPerStep];
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) {
            float x[8];
            row_values(rk[r], x);
#pragma unroll
            for (int iq = 0; iq < kQ; ++iq) {
                float d = 0.0f;
                if constexpr (kTier == SALI_TIER_FP16) {
                    Row16B v;
                    v.u = rk[r].u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) d = __builtin_amdgcn_fdot2(q[iq].h2[e], v.h2[e], d, false);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) d += q[iq].f[e] * x[e];
                }
                d = row16_sum(finish_dot(rk[r], d, q[iq]));
                s[iq][r] = valid[r] ? softmax_scale * d : -INFINITY;
            }
        }
        float p[kQ][kRowsPerStep];
#pragma unroll
        for (int iq = 0; iq < kQ; ++iq) {
            float bm = -INFINITY;
#pragma unroll
            for (int r = 0; r < kRowsPerStep; ++r) bm = fmaxf(bm, s[iq][r]);
            const float new_mx = fmaxf(st[iq].mx, bm);
            // nothing seen yet for this lane group: keep the state (every weight below is exp(-inf) = 0,
            // and the reference maximum must stay finite for that)
            const float ref = new_mx == -INFINITY ? 0.0f : new_mx;
            const float corr = __expf(st[iq].mx - ref);     // first rows: exp(-inf) = 0
            st[iq].lsum *= corr;
            st[iq].zacc *= corr;
#pragma unroll
            for (int e = 0; e < 8; ++e) st[iq].acc[e] *= corr;
#pragma unroll
            for (int r = 0; r < kRowsPerStep; ++r) {
                p[iq][r] = mult * __expf(s[iq][r] - ref);   // absent row: exp(-inf) = 0
                st[iq].lsum += p[iq][r];
            }
            st[iq].mx = new_mx;
        }
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) {
            float x[8];
            row_values(rv[r], x);
#pragma unroll
            for (int iq = 0; iq < kQ; ++iq) {
                const float wgt = weight_of(rv[r], p[iq][r]);
                st[iq].zacc += offset_of(rv[r], p[iq][r]);
#pragma unroll
                for (int e = 0; e < 8; ++e) st[iq].acc[e] += wgt * x[e];
            }
        }
    }
    const int next = split - (count + kGroupRows - 1) / kGroupRows % n_splits;
    return next < 0 ? next + n_splits : next;
}

}  // namespace

// grid (n_chunks * n_splits, n_heads).  Block (c, s) of K/V head h takes the frames
// [frame_lo + c * frames_per_chunk, ...) and of each source frame every n_splits-th group of rows, for kQ of the query heads that share the K/V head (gridDim.z such sets:
// q_per_kv = kQ * gridDim.z), and writes one partial per query head.
template <int kQ, int kRowsPerStep>
__global__ __launch_bounds__(256) void k_attn_partial(const sali_frame_row* __restrict__ rows, Pools pools, int layer,
                                                      int n_heads, const _Float16* __restrict__ q, int frame_lo,
                                                      int frame_hi, int tiles, int frames_per_chunk, int n_splits,
                                                      float softmax_scale, float* __restrict__ partial) {
    __shared__ float s_m[16], s_l[16];
    __shared__ float s_acc[16][kHeadDim];

    const int h = blockIdx.y;
    const int q_first = (h * (int)gridDim.z + (int)blockIdx.z) * kQ;      // first query head of this block
    const int chunk = blockIdx.x / n_splits, split = blockIdx.x % n_splits;
    const int g = threadIdx.x >> 4, l = threadIdx.x & 15;
    const size_t plane_k = ((size_t)layer * 2 + 0) * n_heads + h;
    const size_t plane_v = ((size_t)layer * 2 + 1) * n_heads + h;

    QueryPiece qp[kQ];
    SoftmaxState st[kQ];
#pragma unroll
    for (int iq = 0; iq < kQ; ++iq) {
        Row16B qv;
        qv.u = reinterpret_cast<const u32x4*>(q)[(q_first + iq) * 16 + l];
        qp[iq].sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            qp[iq].f[e] = (float)qv.h[e];
            qp[iq].sum += qp[iq].f[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) qp[iq].h2[e] = qv.h2[e];
        st[iq].mx = -INFINITY;
        st[iq].lsum = 0.0f;
        st[iq].zacc = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) st[iq].acc[e] = 0.0f;
    }

    const int f0 = frame_lo + chunk * frames_per_chunk;
    const int f1 = min(frame_hi, f0 + frames_per_chunk);
    for (int f = f0; f < f1; ++f) {
        // Which stored frame does frame f bring in, and how many times?  A stored frame counts for
        // itself and for the redundant frames behind it (up to the next stored frame or the end of
        // the range); redundant frames at the head of the range, whose source lies before it, are
        // counted at the first of them.  With `tiles` entries per video frame all of this goes by the entries
        // of the same tile, which lie `tiles` apart.  Every thread takes the same decision from the same
        // (uniform) table reads.
        const sali_frame_row r = rows[f];
        bool leader = r.stored != 0;
        if (!leader && r.src >= 0 && r.src < frame_lo) {
            leader = true;
            for (int t = f - tiles; leader && t >= frame_lo; t -= tiles)
                leader = rows[t].src != r.src;                     // an earlier frame of the run counts them
        }
        if (!leader) continue;
        const int src = r.src;
        int n_uses = 1;
        for (int t = f + tiles; t < frame_hi && rows[t].stored == 0; t += tiles)
            if (rows[t].src == src) ++n_uses;
        const float mult = (float)n_uses;
        const sali_frame_row row = rows[src];
        int at = split;
        at = attend_tier<SALI_TIER_FP16, kQ, kRowsPerStep>(pools, plane_k, plane_v, row.base16, row.n16, at, n_splits, g, l, qp,
                                                           softmax_scale, mult, st);
        at = attend_tier<SALI_TIER_INT8, kQ, kRowsPerStep>(pools, plane_k, plane_v, row.base8, row.n8, at, n_splits, g, l, qp,
                                                           softmax_scale, mult, st);
        attend_tier<SALI_TIER_INT4, kQ, kRowsPerStep>(pools, plane_k, plane_v, row.base4, row.n4, at, n_splits, g, l, qp,
                                                      softmax_scale, mult, st);
    }

    // merge the 16 lane groups, one query head after the other
#pragma unroll
    for (int iq = 0; iq < kQ; ++iq) {
        if (iq > 0) __syncthreads();
        if (l == 0) {
            s_m[g] = st[iq].mx;
            s_l[g] = st[iq].lsum;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s_acc[g][8 * l + e] = st[iq].acc[e] + st[iq].zacc;
        __syncthreads();
        float* mine = partial + ((size_t)(q_first + iq) * kAttnPartials + blockIdx.x) * kPartialStride;
        if (threadIdx.x < kHeadDim) {
            float big = -INFINITY;
#pragma unroll
            for (int k = 0; k < 16; ++k) big = fmaxf(big, s_m[k]);
            float lt = 0.0f, at = 0.0f;
            if (big != -INFINITY) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const float w = __expf(s_m[k] - big);
                    lt += w * s_l[k];
                    at += w * s_acc[k][threadIdx.x];
                }
            }
            if (threadIdx.x == 0) {
                mine[0] = big;
                mine[1] = lt;
            }
            mine[2 + threadIdx.x] = at;
        }
    }
}

// grid (query heads), 64 * kWaves threads: merge of a head's partials (n_partials <= kAttnPartials; 0 for an
// empty frame range: zeros and -inf).  A kernel of its own: the kernel boundary is the only
// device-wide ordering this needs, and a device-scope fence in each of the ~2000 blocks of the
// main kernel (last-block hand-over) measured 4.5x slower, because on this chip such a fence writes
// back and invalidates the L2 of the issuing XCD under the stream that the other blocks are reading.
// All it costs is its trips to memory, so it makes one: every wave reads all maxima itself (a lane each)
// while its partials (number wave, wave + kWaves, ...; lane i holds values 2 i, 2 i + 1) are already under
// way, and the waves meet once.  Two halves of a 256-thread block that read maxima first and then took
// alternate partials: 5.2 us for 60 partials x 32 heads, 10.1 for 216 x 4; this: 4.0 and 7.1.
template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void k_attn_merge(const float* __restrict__ partial, int n_partials, int slots,
                                                            float* __restrict__ out, float* __restrict__ lse) {
    constexpr int kPerLane = kAttnPartials / 64, kFlight = kWaves == 4 ? 8 : 4;
    __shared__ float2 s_part[kWaves][64];
    const int h = blockIdx.x, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const float* p = partial + (size_t)h * slots * kPartialStride;      // `slots` partials are reserved per query head
    float m[kPerLane], l[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        const int k = 64 * j + lane;
        float2 ml = make_float2(-INFINITY, 0.0f);
        if (k < n_partials) ml = *reinterpret_cast<const float2*>(p + (size_t)k * kPartialStride);
        m[j] = ml.x;
        l[j] = ml.y;
    }
    float2 v[kFlight];
    auto request = [&](int k) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int ku = k + u * kWaves;
            if (ku < n_partials) v[u] = *reinterpret_cast<const float2*>(p + (size_t)ku * kPartialStride + 2 + 2 * lane);
        }
    };
    if (wave < n_partials) request(wave);
    float big = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
    for (int off = 32; off > 0; off >>= 1) big = fmaxf(big, __shfl_xor(big, off));
    float lt = 0.0f;
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        m[j] = big != -INFINITY ? expf(m[j] - big) : 0.0f;      // the partial's weight
        lt += m[j] * l[j];
    }
    float2 at = make_float2(0.0f, 0.0f);
    for (int k = wave; k < n_partials; k += kFlight * kWaves) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int ku = k + u * kWaves;
            if (ku < n_partials) {
                const float mine = ku < 64 ? m[0] : (ku < 128 ? m[1] : (ku < 192 ? m[2] : m[3]));
                const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), ku & 63));
                at.x += w * v[u].x;
                at.y += w * v[u].y;
            }
        }
        if (k + kFlight * kWaves < n_partials) request(k + kFlight * kWaves);
    }
    s_part[wave][lane] = at;
    __syncthreads();
    if (wave != 0) return;
    for (int off = 32; off > 0; off >>= 1) lt += __shfl_xor(lt, off);
#pragma unroll
    for (int k = 1; k < kWaves; ++k) {
        at.x += s_part[k][lane].x;
        at.y += s_part[k][lane].y;
    }
    float* dst = out + (size_t)h * kHeadDim + 2 * lane;       // the caller's: aligned for float only
    dst[0] = lt > 0.0f ? at.x / lt : 0.0f;
    dst[1] = lt > 0.0f ? at.y / lt : 0.0f;
    if (lse != nullptr && lane == 0) lse[h] = lt > 0.0f ? big + logf(lt) : -INFINITY;
}

// four waves where that is at most eight partials a wave, all under way at once; else sixteen
static void launch_merge(const float* d_partial, int n_partials, int slots, int n_q_heads, float* d_out, float* d_lse_or_null,
                         hipStream_t s) {
    if (n_partials > 32)
        hipLaunchKernelGGL(k_attn_merge<16>, dim3(n_q_heads), dim3(1024), 0, s, d_partial, n_partials, slots, d_out, d_lse_or_null);
    else
        hipLaunchKernelGGL(k_attn_merge<4>, dim3(n_q_heads), dim3(256), 0, s, d_partial, n_partials, slots, d_out, d_lse_or_null);
}

// ---------------------------------------------------------------------------------------------
// Many queries per K/V head (9 to 64: the tokens of a prompt attending to the cached video, or
// large query groups): Q K^T and P V are real matrix products, so they run on the matrix cores
// (v_mfma_f32_32x32x16_f16) and every compressed row is read once per 32 queries.
//
// One block = one K/V head x one tile of 32 queries x one share of the frame range; its eight waves take
// the share's tiles of 32 cached rows in turn and meet once, at the end.  Per tile:
//   S^T = K^ Q^T : A operand = K^ tile (lane = row n, registers = head-dim values), B operand = the
//        queries (lane = query m); the result has lane = query, registers = rows, so the softmax
//        over rows is a reduction over the lane's 16 registers and one exchange between the two
//        lane halves, and P in that layout IS the B operand of the second product (the rows of the
//        tile are contracted in the order the registers hold them);
//   out^T = V^^T P^T : A operand = V^^T (lane = head-dim value d, registers = two runs of 4
//        consecutive rows), read from the wave's LDS tile with the transposing 8-byte LDS read.
// The head-dim index of the contraction is permuted (lane half hh of a row holds values
// [64 hh, 64 hh + 64), k-step t takes 8 of them from each half) so that a lane reads one contiguous
// piece of its row; Q uses the same permutation.  Here the dequantised values DO exist as fp16
// (K^ = fp16(code * scale), fp16(code * scale + zero), the values dequantise-on-read produces) because
// the matrix cores take fp16 operands; the softmax weights are rounded to fp16 for the second product
// as well.  Both stay inside the tolerance of the floating-point results (largest error printed by
// the tests).  Accumulation, softmax state and partials are fp32; partials have the layout of the
// single-query kernel and are merged by the same k_attn_merge.
//
// What bounds it: the trip to memory of a tile (waves wait for 47 % of their time), then the vector
// instructions of a tile (610, conversions and softmax).  Hence: a tile's K^ and V^ rows are asked for a
// whole tile ahead, across tiers and frames; the launch is one block of eight waves per compute unit, forced
// to one by its LDS, so that all start at once; and a block writes one partial instead of one per wave.
// 32 heads x 32 queries over 20 frames (173 / 200 / 203 rows, 118 MB): 34.5 us + 4.6 us of merge.  The same
// tiles as 512 independent blocks of four waves that should just have fitted twice per compute unit, a
// tier's loads one tile ahead and a partial per wave, took 69.6 us + 8.0 us of merge: such blocks do not
// pack perfectly, the last of them ran alone in a second round (mean wave lifetime 26 us).
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

namespace {

constexpr int kPfRows = 32;                       // cached rows per tile
constexpr int kPfWaves = 8;                       // waves of a block
constexpr int kPfKStride = kHeadDim + 8;          // halves per LDS row: lane = row reads of 16 bytes, eight lanes cover all banks
constexpr int kPfVStride = kHeadDim + 16;         // transposing reads: four rows of 64 bytes, eight banks apart
constexpr int kPfTileHalves = kPfRows * (kPfKStride + kPfVStride);
constexpr int kPfGroup = 64;                      // frames looked up at a time
constexpr int kPfOutStride = 33;                  // floats per head-dim value of a wave's result in LDS
static_assert(kHeadDim * kPfOutStride * 4 <= kPfTileHalves * 2, "a wave's result fits its tiles");

union Half8 {
    u32x4 u;
    half4_t h4[2];
    half8_t h8;
    _Float16 h[8];
};

// what a block takes from one stored frame: its tiles i0 .. of the tiers in pool order (FP16, INT8, INT4)
struct PfFrame {
    int start;                  // number of the frame's first tile in the block's sequence
    int i0;                     // its index among the frame's tiles
    int base[3], n[3];
    float mult;                 // how often the frame counts (itself and the pointer entries behind it)
};

__device__ __forceinline__ int pf_tiles(int rows) { return (rows + kPfRows - 1) / kPfRows; }

// A tile of 32 pool rows as it comes from memory, a lane's share: 16-byte pieces of codes, consecutive
// lanes reading consecutive memory (a lane-per-row pattern, which the matrix-core operands would suggest,
// was measured at 1.6 TB/s), and the scales / zero-points of their groups.  Rows past the end of
// the run repeat its last row (their softmax weight is zero).
struct PfRaw {
    u32x4 c[8];                 // FP16: 8 x 8 values.  INT8: 4 x 16 codes, scales in c[4].  INT4: 2 x 32 codes,
};                              // scales in c[2].xy, zero-points in c[2].zw

struct PfRows {                 // the rows of one tier of one frame and plane
    const char* codes;
    const float* scale;
    const uint16_t* zero;
};

__device__ __forceinline__ void pf_load_tile(int tier, const PfRows& src, int jb, int count, int lane, PfRaw& r) {
    const int last = count - 1;
    if (tier == SALI_TIER_FP16) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t row = (uint32_t)min(jb + 4 * u + (lane >> 4), last);
            r.c[u] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4*>(src.codes + (row * (uint32_t)(kHeadDim * 2) + (uint32_t)(lane & 15) * 16u)));
        }
    } else if (tier == SALI_TIER_INT8) {
        float sc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t row = (uint32_t)min(jb + 8 * u + (lane >> 3), last);
            r.c[u] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4*>(src.codes + (row * (uint32_t)kHeadDim + (uint32_t)(lane & 7) * 16u)));
            sc[u] = src.scale[row * (uint32_t)kGroupsPerRow + (uint32_t)((lane & 7) >> 1)];
        }
        r.c[4] = (u32x4){__builtin_bit_cast(uint32_t, sc[0]), __builtin_bit_cast(uint32_t, sc[1]),
                         __builtin_bit_cast(uint32_t, sc[2]), __builtin_bit_cast(uint32_t, sc[3])};
    } else {
        float sc[2];
        uint32_t zp[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t row = (uint32_t)min(jb + 16 * u + (lane >> 2), last);
            r.c[u] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4*>(src.codes + (row * (uint32_t)(kHeadDim / 2) + (uint32_t)(lane & 3) * 16u)));
            sc[u] = src.scale[row * (uint32_t)kGroupsPerRow + (uint32_t)(lane & 3)];
            zp[u] = src.zero[row * (uint32_t)kGroupsPerRow + (uint32_t)(lane & 3)];
        }
        r.c[2] = (u32x4){__builtin_bit_cast(uint32_t, sc[0]), __builtin_bit_cast(uint32_t, sc[1]), zp[0], zp[1]};
    }
}

// dequantise the lane's pieces and put them where they belong in the LDS tile [32 rows][kStride halves]
template <int kStride>
__device__ __forceinline__ void pf_store_tile(int tier, const PfRaw& r, int lane, _Float16* tile) {
    if (tier == SALI_TIER_FP16) {
        u32x4* dst = reinterpret_cast<u32x4*>(tile + (lane >> 4) * kStride + 8 * (lane & 15));
#pragma unroll
        for (int u = 0; u < 8; ++u) dst[u * (4 * kStride / 8)] = r.c[u];
    } else if (tier == SALI_TIER_INT8) {
        u32x4* dst = reinterpret_cast<u32x4*>(tile + (lane >> 3) * kStride + 16 * (lane & 7));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t sbits = r.c[4][u];           // (a copy: bit_cast of a vector element reads element 0)
            const float sc = __builtin_bit_cast(float, sbits);
            Half8 o[2];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t word = r.c[u][w];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    o[w >> 1].h[4 * (w & 1) + i] = (_Float16)((float)(int)(int8_t)((word >> (8 * i)) & 0xFF) * sc);
            }
            dst[u * (8 * kStride / 8)] = o[0].u;
            dst[u * (8 * kStride / 8) + 1] = o[1].u;
        }
    } else {
        u32x4* dst = reinterpret_cast<u32x4*>(tile + (lane >> 2) * kStride + 32 * (lane & 3));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t sbits = r.c[2][u], zbits = r.c[2][2 + u];
            const float sc = __builtin_bit_cast(float, sbits);
            const float zp = (float)__builtin_bit_cast(_Float16, (uint16_t)zbits);
#pragma unroll
            for (int w = 0; w < 4; ++w) {                           // 8 values = one word of codes
                const uint32_t word = r.c[u][w];
                // nibbles to bytes first (even elements in one word, odd ones in another): a byte converts to
                // fp32 in one instruction, a nibble needs a shift and a mask each
                uint32_t ev = word & 0x0F0F0F0Fu, od = (word >> 4) & 0x0F0F0F0Fu;
                asm volatile("" : "+v"(ev), "+v"(od));  // (keeps the compiler from folding the bytes back into nibbles)
                Half8 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    o.h[2 * i] = (_Float16)__builtin_fmaf((float)((ev >> (8 * i)) & 0xFFu), sc, zp);
                    o.h[2 * i + 1] = (_Float16)__builtin_fmaf((float)((od >> (8 * i)) & 0xFFu), sc, zp);
                }
                dst[u * (16 * kStride / 8) + w] = o.u;
            }
        }
    }
}

// LDS operations of one wave execute in order, so the wave's private tiles need no barrier, only
// that the compiler keeps the order
__device__ __forceinline__ void pf_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Four rows x 16 columns of halves, transposed: the 16 lanes of a group give the addresses of the four rows'
// 8-byte pieces (lane i: row i / 4, columns 4 (i % 4) ..), lane i receives column i of the four rows.
__device__ __forceinline__ half4_t pf_read_transposed(const _Float16* p) {
    typedef __attribute__((address_space(3))) short4_t lds_short4;
    const short4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p));
    return __builtin_bit_cast(half4_t, v);
}

// ONE wave: the frames g0 .. g0 + 63 (below f_end) that bring tiles into the block's share, as a list in
// `list`; returns its length and, in n_tiles, the tiles.  The share of block `part` of `parts` is the
// stretch [part * n, (part + 1) * n) of the range's n frames in units of 1 / parts frame, a frame's part of
// it the same fraction of its tiles: every tile belongs to exactly one block, and with frames of like size
// the blocks get equal work.
// A stored frame counts for itself and for the redundant frames behind it (up to the next stored frame or
// the end of the range); redundant frames at the head of the range, whose source lies before it, are
// counted at the first of them.  With `tiles` entries per video frame: the entries of the same tile, `tiles` apart.
__device__ __forceinline__ int pf_list_frames(const sali_frame_row* __restrict__ rows, int frame_lo, int frame_hi, int tiles, int g0,
                                              int f_end, int part, int parts, int lane, int* s_src, PfFrame* list,
                                              int* n_tiles) {
    const int f = g0 + lane, g_end = min(f_end, g0 + kPfGroup);
    const bool valid = f < g_end;
    sali_frame_row row = {};
    row.src = -1;
    if (valid) row = rows[f];
    const bool stored = valid && row.stored != 0;
    s_src[lane] = row.src;
    pf_lds_order();
    const unsigned long long stored_mask = __ballot(stored);
    bool leader = stored;
    const int src = row.src;
    if (valid && !stored && src >= 0 && src < frame_lo) {
        leader = true;
        for (int t = f - tiles; leader && t >= frame_lo; t -= tiles)
            leader = rows[t].src != src;                     // an earlier frame of the run counts them
    }
    int n_uses = 1;
    if (leader) {
        unsigned long long behind = lane + tiles > 63 ? 0ull : stored_mask >> (lane + tiles);
        if (tiles > 1) {
            unsigned long long same = 0ull;                  // every tiles-th bit
            for (int b = 0; b < 64; b += tiles) same |= 1ull << b;
            behind &= same;
        }
        const int run_end = behind != 0ull ? f + tiles + __builtin_ctzll(behind) : g_end;
        int t = f + tiles;
        for (; t < run_end; t += tiles)
            if (s_src[t - g0] == src) ++n_uses;
        if (behind == 0ull)
            for (; t < frame_hi && rows[t].stored == 0; t += tiles)
                if (rows[t].src == src) ++n_uses;
        if (!stored) row = rows[src];
    }
    int i0 = 0, cnt = 0;
    if (leader) {
        const long long n = frame_hi - frame_lo, at = (long long)(f - frame_lo) * parts;
        const long long lo = max(0ll, part * n - at), hi = min((long long)parts, (part + 1) * n - at);
        const int t = pf_tiles(row.n16) + pf_tiles(row.n8) + pf_tiles(row.n4);
        if (hi > lo) {
            i0 = (int)(t * lo / parts);
            cnt = (int)(t * hi / parts) - i0;
        }
    }
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    const unsigned long long use = __ballot(cnt > 0);
    if (cnt > 0) {
        PfFrame e;
        e.start = incl - cnt;
        e.i0 = i0;
        e.base[0] = row.base16;
        e.base[1] = row.base8;
        e.base[2] = row.base4;
        e.n[0] = row.n16;
        e.n[1] = row.n8;
        e.n[2] = row.n4;
        e.mult = (float)n_uses;
        list[__popcll(use & (lane == 0 ? 0ull : (~0ull >> (64 - lane))))] = e;
    }
    *n_tiles = __shfl(incl, 63);
    return (int)__popcll(use);
}

}  // namespace

// grid (parts of the frame range, n_heads, ceil(q_per_kv / 32)), 512 threads.  kLongRange: a stored frame of the
// range may count more than 2^15 times, which takes more than 2^15 frames
template <bool kLongRange>
__global__ __launch_bounds__(64 * kPfWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_prefill(
    const sali_frame_row* __restrict__ rows, Pools pools, int layer, int n_heads, const _Float16* __restrict__ q,
    int q_per_kv, int frame_lo, int frame_hi, int tiles, float softmax_scale, float* __restrict__ partial) {
    __shared__ __align__(16) _Float16 s_tiles[kPfWaves][kPfTileHalves];     // a K^ and a V^ tile per wave; the results at the end
    __shared__ PfFrame s_list[kPfGroup];
    __shared__ int s_src[kPfGroup];
    __shared__ int s_n[2];
    __shared__ float s_m[kPfWaves][32], s_l[kPfWaves][32];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int m = lane & 31, hh = lane >> 5;
    const int h = blockIdx.y, part = blockIdx.x, parts = gridDim.x;
    const int qi = (int)blockIdx.z * 32 + m;                 // this lane's query among the q_per_kv of the K/V head
    const size_t plane_k = ((size_t)layer * 2 + 0) * n_heads + h;
    const size_t plane_v = ((size_t)layer * 2 + 1) * n_heads + h;
    _Float16* s_k = s_tiles[wave];
    _Float16* s_v = s_k + kPfRows * kPfKStride;

    // the queries stay in registers, as the B operand wants them (zeros past q_per_kv)
    half8_t qb[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        Half8 v;
        v.u = (u32x4){0u, 0u, 0u, 0u};
        if (qi < q_per_kv) v.u = reinterpret_cast<const u32x4*>(q + ((size_t)h * q_per_kv + qi) * kHeadDim + 64 * hh)[t];
        qb[t] = v.h8;
    }
    const float scale2 = softmax_scale * 1.44269504088896340736f;      // scores in units of log 2 from here on
    float mx = -INFINITY, lsum = 0.0f;
    float16_t acc[4];           // acc[dt][r] = out[m][32 dt + 8 (r / 4) + 4 hh + r % 4], not yet normalised
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.0f;

    const long long n_range = frame_hi - frame_lo;
    const int f_begin = frame_lo + (int)(part * n_range / parts);
    const int f_end = frame_lo + (int)(((part + 1) * n_range + parts - 1) / parts);
    for (int g0 = f_begin; g0 < f_end; g0 += kPfGroup) {
        if (g0 != f_begin) __syncthreads();                 // every wave is through with the list
        if (wave == 0) {
            int n_tiles;
            const int len = pf_list_frames(rows, frame_lo, frame_hi, tiles, g0, f_end, part, parts, lane, s_src, s_list, &n_tiles);
            if (lane == 0) {
                s_n[0] = len;
                s_n[1] = n_tiles;
            }
        }
        __syncthreads();
        const int len = __builtin_amdgcn_readfirstlane(s_n[0]), n_tiles = __builtin_amdgcn_readfirstlane(s_n[1]);
        int e = 0;                                          // list entry of the tile in flight
        // tile `g` of the block's sequence: its tier and rows, all uniform over the wave
        int tier = 0, jb = 0, count = 0;
        float mult = 1.0f;
        PfRaw rk, rv;
        auto request = [&](int g) {
            while (e + 1 < len && g >= __builtin_amdgcn_readfirstlane(s_list[e + 1].start)) ++e;
            const PfFrame& fr = s_list[e];
            int i = __builtin_amdgcn_readfirstlane(fr.i0 + g - fr.start);
            const int n0 = __builtin_amdgcn_readfirstlane(fr.n[0]), n1 = __builtin_amdgcn_readfirstlane(fr.n[1]);
            const int t0 = pf_tiles(n0), t1 = pf_tiles(n1);
            tier = i < t0 ? SALI_TIER_FP16 : (i < t0 + t1 ? SALI_TIER_INT8 : SALI_TIER_INT4);
            i -= tier == SALI_TIER_FP16 ? 0 : (tier == SALI_TIER_INT8 ? t0 : t0 + t1);
            jb = i * kPfRows;
            count = __builtin_amdgcn_readfirstlane(fr.n[tier]);
            mult = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, fr.mult)));
            const int base = __builtin_amdgcn_readfirstlane(fr.base[tier]);
            const size_t row_k = pool_row0(pools, base, count, plane_k), row_v = pool_row0(pools, base, count, plane_v);
            const char* codes = tier == SALI_TIER_FP16 ? reinterpret_cast<const char*>(pools.p16)
                                : tier == SALI_TIER_INT8 ? reinterpret_cast<const char*>(pools.c8)
                                                         : reinterpret_cast<const char*>(pools.c4);
            const uint32_t row_bytes = tier == SALI_TIER_FP16 ? kHeadDim * 2 : (tier == SALI_TIER_INT8 ? kHeadDim : kHeadDim / 2);
            const float* scale = tier == SALI_TIER_INT8 ? pools.s8 : pools.s4;
            const PfRows k = {codes + row_k * row_bytes, scale + row_k * kGroupsPerRow, pools.z4 + row_k * kGroupsPerRow};
            const PfRows v = {codes + row_v * row_bytes, scale + row_v * kGroupsPerRow, pools.z4 + row_v * kGroupsPerRow};
            pf_load_tile(tier, k, jb, count, lane, rk);
            pf_load_tile(tier, v, jb, count, lane, rv);
        };
        if (wave < n_tiles) request(wave);
        for (int g = wave; g < n_tiles; g += kPfWaves) {
            pf_lds_order();                                 // the previous tile's reads are done
            pf_store_tile<kPfKStride>(tier, rk, lane, s_k);
            pf_store_tile<kPfVStride>(tier, rv, lane, s_v);
            pf_lds_order();
            const int left = count - jb;                    // rows of this tile that exist
            const float times = mult;
            if (g + kPfWaves < n_tiles) request(g + kPfWaves);      // in flight while this tile is worked on

            // S^T = K^ Q^T with v_mfma_f32_32x32x16_f16 (A[i][k]: lane = i + 32 (k / 8), element k % 8; B alike;
            // D[i][j]: lane = j + 32 hh, register r holds i = 8 (r / 4) + 4 hh + r % 4).  Lane (row m, half hh),
            // step t: values 64 hh + 8 t .. + 7 of the row; the queries use the same assignment
            float16_t s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const half8_t ka = *reinterpret_cast<const half8_t*>(s_k + m * kPfKStride + 64 * hh + 8 * t);
                s = __builtin_amdgcn_mfma_f32_32x32x16_f16(ka, qb[t], s, 0, 0, 0);
            }
            // s[r] = <K^ row jb + n(r), query m>, n(r) = 8 (r / 4) + 4 hh + r % 4
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] *= scale2;
            if (left < kPfRows) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r / 4) + 4 * hh + (r % 4) >= left) s[r] = -INFINITY;
            }
            float tmax = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, s[r]);
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            // a weight times its count must stay an fp16 number (at most 65 504) for the second product: what a count
            // has above 2^15 raises the reference of the weights.  Up to there the counts stay out of the reference,
            // so that rows counted once next to a frame counted often keep their place above the fp16 subnormals
            if constexpr (kLongRange) tmax += fmaxf(0.0f, __log2f(times) - 15.0f);
            const float mnew = fmaxf(mx, tmax);
            const float corr = __builtin_amdgcn_exp2f(mx - mnew);
            // the softmax weights in the order the second product wants them: step jj of two, element e of the
            // lane's eight = row 16 jj + 8 (e / 4) + 4 hh + e % 4 of the tile, which is register 8 jj + e
            float psum = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(s[r] - mnew);
            if (times != 1.0f) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] *= times;
            }
            half8_t pb[2];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                psum += s[r];
                pb[r >> 3][r & 7] = (_Float16)s[r];
            }
            psum += __shfl_xor(psum, 32);
            lsum = lsum * corr + psum;
            mx = mnew;
            // the 64 accumulators are rescaled only when some query of the wave saw a new maximum (rare after
            // the first tiles); the test is wave-uniform
            if (__builtin_amdgcn_ballot_w64(corr != 1.0f) != 0) {
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[dt][r] *= corr;
            }
            // out^T += V^^T P^T: A operand lane (value d = 32 dt + m, half hh): the same eight rows of column d
            const _Float16* tr = s_v + (4 * hh + ((lane & 15) >> 2)) * kPfVStride + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) {
                    Half8 va;
                    va.h4[0] = pf_read_transposed(tr + (16 * jj) * kPfVStride + 32 * dt);
                    va.h4[1] = pf_read_transposed(tr + (16 * jj + 8) * kPfVStride + 32 * dt);
                    acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va.h8, pb[jj], acc[dt], 0, 0, 0);
                }
        }
    }

    // the eight waves meet: each rescales to the block's maximum and leaves its 128 x 32 values in the
    // memory of its own tiles, then every thread adds up eight outputs
    if (hh == 0) {
        s_m[wave][m] = mx;
        s_l[wave][m] = lsum;
    }
    __syncthreads();
    float big = -INFINITY;
#pragma unroll
    for (int w = 0; w < kPfWaves; ++w) big = fmaxf(big, s_m[w][m]);
    const float fac = mx == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mx - big);
    float* mine = reinterpret_cast<float*>(s_tiles[wave]);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(32 * dt + 8 * (r / 4) + 4 * hh + (r % 4)) * kPfOutStride + m] = acc[dt][r] * fac;
    __syncthreads();
    for (int idx = threadIdx.x; idx < 32 * kHeadDim; idx += 64 * kPfWaves) {
        const int mm = idx / kHeadDim, d = idx % kHeadDim;
        const int qq = (int)blockIdx.z * 32 + mm;
        if (qq >= q_per_kv) continue;
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kPfWaves; ++w) sum += reinterpret_cast<const float*>(s_tiles[w])[d * kPfOutStride + mm];
        float* dst = partial + (((size_t)h * q_per_kv + qq) * parts + part) * kPartialStride;
        dst[2 + d] = sum;
        if (d == 0) {
            float top = -INFINITY, lt = 0.0f;
            for (int w = 0; w < kPfWaves; ++w) top = fmaxf(top, s_m[w][mm]);
            if (top != -INFINITY)
                for (int w = 0; w < kPfWaves; ++w) lt += s_l[w][mm] * __builtin_amdgcn_exp2f(s_m[w][mm] - top);
            dst[0] = top * 0.69314718055994530942f;
            dst[1] = lt;
        }
    }
}

hipError_t launch_attend(const sali_frame_row* d_rows, Pools pools, int layer, int n_heads, int q_per_kv,
                         const void* d_q, int frame_lo, int frame_hi, int tiles, RowsPerFrame kept, float softmax_scale, float* d_partial,
                         float* d_out, float* d_lse_or_null, hipEvent_t ev_start, hipEvent_t ev_stop, hipStream_t s) {
    const int n_range = frame_hi - frame_lo;
    int n_partials = 0;
    if (n_range > 0 && q_per_kv > kAttnMaxQPerKv) {
        // matrix-core path: one block of eight waves per compute unit, as many parts of the range as that
        // gives a K/V head, but no more than leave every wave a tile (a frame has up to kTokens / kPfRows + 3),
        // and no more partials than the scratch holds (kAttnSlotsPerHead per K/V head, shared out over its queries).
        // Where one part each would leave a third of the compute units or more idle, three parts each: two rounds
        // of a third of the work.  160 heads x 9 queries x 20 frames 168 -> 133 us a call, 129 heads 167 -> 125
        // (independent blocks of four waves: 141 and 162)
        const int pairs = n_heads * ((q_per_kv + 31) / 32);
        int parts = kComputeUnits / pairs;
        if (parts == 1 && 3 * pairs <= 2 * kComputeUnits) parts = 3;
        const long long fill = ((long long)n_range * (kTokens / kPfRows + 3) + kPfWaves - 1) / kPfWaves;
        if (parts > fill) parts = (int)fill;
        if (parts > kAttnSlotsPerHead / q_per_kv) parts = kAttnSlotsPerHead / q_per_kv;
        if (parts > kAttnPartials) parts = kAttnPartials;
        n_partials = parts < 1 ? 1 : parts;
        if (ev_start != nullptr && hipEventRecord(ev_start, s) != hipSuccess) return hipErrorUnknown;
        const dim3 grid(n_partials, n_heads, (q_per_kv + 31) / 32);
        // the general variant costs 0.7 % (32 heads x 32 queries x 20 frames 143.8 -> 144.8 us for four layers)
        if (n_range > 32768)
            hipLaunchKernelGGL(k_attn_prefill<true>, grid, dim3(64 * kPfWaves), 0, s, d_rows, pools, layer, n_heads,
                               reinterpret_cast<const _Float16*>(d_q), q_per_kv, frame_lo, frame_hi, tiles, softmax_scale, d_partial);
        else
            hipLaunchKernelGGL(k_attn_prefill<false>, grid, dim3(64 * kPfWaves), 0, s, d_rows, pools, layer, n_heads,
                               reinterpret_cast<const _Float16*>(d_q), q_per_kv, frame_lo, frame_hi, tiles, softmax_scale, d_partial);
        if (ev_stop != nullptr && hipEventRecord(ev_stop, s) != hipSuccess) return hipErrorUnknown;
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        launch_merge(d_partial, n_partials, n_partials, n_heads * q_per_kv, d_out, d_lse_or_null, s);
        return hipGetLastError();
    }
    if (n_range > 0) {
        // eight queries per K/V head run as two sets of four (two blocks read the same rows, the second
        // mostly from cache): a block with eight query states needs 256 registers per lane and was slower
        const int kq = q_per_kv == 8 ? 4 : q_per_kv, sets = q_per_kv / kq;
        // One resident round of blocks: at 8 blocks of 256 threads per compute unit the chip holds
        // kResidentBlocks; more blocks than that leave a second, nearly empty round at the end of a
        // bandwidth-bound kernel.  Blocks of a head: whole frames per block for long ranges, row
        // groups of a frame split over blocks for short ones (up to 9 groups of 64 rows per tier).
        int per_head = kResidentBlocks / n_heads;
        per_head = per_head < 1 ? 1 : (per_head > kAttnPartials ? kAttnPartials : per_head);
        const int fpc = (n_range + per_head - 1) / per_head;
        const int n_chunks = (n_range + fpc - 1) / fpc;
        // Small ranges: with groups of 64 rows fewer than two blocks per compute unit would have any (at most
        // rows / 64 + 3 groups a frame), and each would be a chain of three tiers' loads and four rows'
        // arithmetic per lane group.  Groups of 16 rows then, one row per lane group, over up to twice the splits:
        // 4 queries x 8 heads, 2 frames of 124 / 28 / 84 rows 11.3 -> 6.2 us, 1 query 6.3 -> 4.3.  No more splits
        // than a frame has groups: with eighteen for frames of 64 rows, fourteen of them empty, 40 heads x 8
        // queries x 2 frames took 17.6 us (groups of 64 rows: 12.4), and 8.0 with four.  Not fewer than four, for
        // frames stored under an earlier tier rule that kept more.
        const bool small = (long long)n_range * ((kept.n16 + kept.n8 + kept.n4) / 64 + 1) * n_heads * sets < 2 * kComputeUnits;
        const int groups = (kept.n16 + 15) / 16 + (kept.n8 + 15) / 16 + (kept.n4 + 15) / 16;
        const int most = small ? (groups < 4 ? 4 : (groups < 18 ? groups : 18)) : 9;
        int n_splits = per_head / n_chunks;
        n_splits = n_splits < 1 ? 1 : (n_splits > most ? most : n_splits);
        n_partials = n_chunks * n_splits;
        if (ev_start != nullptr && hipEventRecord(ev_start, s) != hipSuccess) return hipErrorUnknown;
        const dim3 grid(n_partials, n_heads, sets);
        const _Float16* q = reinterpret_cast<const _Float16*>(d_q);
#define SALI_ATTN_LAUNCH(KQ)                                                                                              \
    do {                                                                                                                  \
        if (small)                                                                                                        \
            hipLaunchKernelGGL((k_attn_partial<KQ, 1>), grid, dim3(256), 0, s, d_rows, pools, layer, n_heads, q, frame_lo, \
                               frame_hi, tiles, fpc, n_splits, softmax_scale, d_partial);                                        \
        else                                                                                                              \
            hipLaunchKernelGGL((k_attn_partial<KQ, 4>), grid, dim3(256), 0, s, d_rows, pools, layer, n_heads, q, frame_lo, \
                               frame_hi, tiles, fpc, n_splits, softmax_scale, d_partial);                                        \
    } while (0)
        switch (kq) {
            case 1: SALI_ATTN_LAUNCH(1); break;
            case 2: SALI_ATTN_LAUNCH(2); break;
            case 4: SALI_ATTN_LAUNCH(4); break;
            default: return hipErrorInvalidValue;
        }
#undef SALI_ATTN_LAUNCH
        if (ev_stop != nullptr && hipEventRecord(ev_stop, s) != hipSuccess) return hipErrorUnknown;
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    launch_merge(d_partial, n_partials, kAttnPartials, n_heads * q_per_kv, d_out, d_lse_or_null, s);
    return hipGetLastError();
}

}  // namespace sali
