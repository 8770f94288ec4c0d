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
// the vector ALU stays below the memory time (the group scale is applied once per row to the dot
// product and to the softmax weight, the INT4 zero-point through sum(q) and a separate accumulator; dot products
// take codes as pairs of halves).  A layer of 32 heads over 20 frames (131 MB): 25.5 us, a frame more 0.97 (6.8 TB/s), what does not
// depend on the size 6.  With the merge in a kernel of its own, 60 parts a head that did not all fit the chip at once (73 registers:
// six blocks per compute unit, not eight), launch order and one code at a time: 28.4, 9 of it fixed; 8 heads x 8 queries 41.5 -> 28.5, 4 heads
// over 12 frames 17.3 -> 9.3, one frame 12.9 -> 6.9 (kernel to kernel).
// The compressed rows are read once, in pool order (attention does not care about token order),
// with the lane mapping of the pack / unpack kernels: a row is handled by 16 adjacent lanes holding
// 8 consecutive head-dim values each, a 32-value quantisation group is one lane quad, the dot
// product is reduced over the 16 lanes with four DPP moves.  Every lane group keeps an
// online-softmax state (running max, sum and 8 output values per lane); a block merges its 16 lane
// groups through LDS and writes one partial (max, sum, 128 values); the last block of a head to finish merges
// the partials, or a launch of its own where they are many (in_launch_parts).  The three tiers of a frame are walked by three instances of one loop
// specialised on the row format.  With grouped-query attention the kQ query heads that share a K/V
// head are handled by the same block, so every compressed row is still read once.

#include <type_traits>

#include "sali_internal.h"

namespace sali {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int kComputeUnits = 256;
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

// the lane's piece of the query: 8 values as packed halves, in the pairs (2 i, 2 i + 1) and (i, i + 4) that the codes of a row come in,
// and their sum
struct QueryPiece {
    half2_t h2[4], across[4];
    float sum;
};
__device__ __forceinline__ QueryPiece query_piece(const Row16B& q) {
    QueryPiece p;
    p.sum = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) p.sum += (float)q.h[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        p.h2[e] = q.h2[e];
        p.across[e] = (half2_t){q.h[e], q.h[e + 4]};
    }
    return p;
}

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

// the rows of one tier of one frame and plane; uniform over the block, so that a lane's address is a scalar base and 32 bits
struct TierRows {
    const char* codes;
    const float* scale;
    const uint16_t* zero;
};
template <int kTier>
__device__ __forceinline__ TierRows tier_rows(const Pools& pools, int base, int count, size_t plane) {
    const size_t row0 = pool_row0(pools, base, count, plane);
    if constexpr (kTier == SALI_TIER_FP16) return {reinterpret_cast<const char*>(pools.p16 + row0 * kHeadDim), nullptr, nullptr};
    else if constexpr (kTier == SALI_TIER_INT8) return {reinterpret_cast<const char*>(pools.c8 + row0 * kHeadDim), pools.s8 + row0 * kGroupsPerRow, nullptr};
    else return {reinterpret_cast<const char*>(pools.c4 + row0 * (kHeadDim / 2)), pools.s4 + row0 * kGroupsPerRow, pools.z4 + row0 * kGroupsPerRow};
}
template <typename V>
__device__ __forceinline__ const V* at_byte(const void* base, uint32_t offset) {
    return reinterpret_cast<const V*>(static_cast<const char*>(base) + offset);
}

// the lane's piece of row j
__device__ __forceinline__ void load_row(const TierRows& t, uint32_t j, uint32_t l, RawRow<SALI_TIER_FP16>& r) {
    r.u = __builtin_nontemporal_load(at_byte<u32x4>(t.codes, j * (kHeadDim * 2) + l * 16));
}
__device__ __forceinline__ void load_row(const TierRows& t, uint32_t j, uint32_t l, RawRow<SALI_TIER_INT8>& r) {
    r.u = __builtin_nontemporal_load(at_byte<u32x2>(t.codes, j * kHeadDim + l * 8));
    r.scale = *at_byte<float>(t.scale, j * (kGroupsPerRow * 4) + (l >> 2) * 4);
}
__device__ __forceinline__ void load_row(const TierRows& t, uint32_t j, uint32_t l, RawRow<SALI_TIER_INT4>& r) {
    r.u = __builtin_nontemporal_load(at_byte<uint32_t>(t.codes, j * (kHeadDim / 2) + l * 4));
    r.scale = *at_byte<float>(t.scale, j * (kGroupsPerRow * 4) + (l >> 2) * 4);
    r.zero = (float)__builtin_bit_cast(_Float16, *at_byte<uint16_t>(t.zero, j * (kGroupsPerRow * 2) + (l >> 2) * 2));
}

// The lane's raw values of a row as pairs of halves.  Codes become halves through their place in the mantissa of 1024 (then 1024, and the
// 128 of a signed byte, are taken off: exact), two at a time.
__device__ __forceinline__ half2_t half_pair(uint32_t bits, float bias) {
    const half2_t b = {(_Float16)bias, (_Float16)bias};
    return __builtin_bit_cast(half2_t, bits) - b;
}
// INT4 codes are taken around their middle (K^ = (code - 8) * scale + (zero + 8 * scale), V^ alike): the two parts of a sum then do not
// cancel as those of positive codes and the smallest value of the group do
constexpr float kMidCode4 = 8.0f;
struct HalfPairs {
    half2_t v[4];
};
__device__ __forceinline__ HalfPairs row_pairs(const RawRow<SALI_TIER_FP16>& r) {
    Row16B v;
    v.u = r.u;
    return {{v.h2[0], v.h2[1], v.h2[2], v.h2[3]}};
}
__device__ __forceinline__ HalfPairs row_pairs(const RawRow<SALI_TIER_INT8>& r) {
    const uint32_t x = r.u.x ^ 0x80808080u, y = r.u.y ^ 0x80808080u, exponent = 0x64646464u;
    return {{half_pair(__builtin_amdgcn_perm(exponent, x, 0x04010400u), 1152.0f), half_pair(__builtin_amdgcn_perm(exponent, x, 0x04030402u), 1152.0f),
             half_pair(__builtin_amdgcn_perm(exponent, y, 0x04010400u), 1152.0f), half_pair(__builtin_amdgcn_perm(exponent, y, 0x04030402u), 1152.0f)}};
}
__device__ __forceinline__ HalfPairs row_pairs(const RawRow<SALI_TIER_INT4>& r) {
    HalfPairs p;
#pragma unroll
    for (int i = 0; i < 4; ++i) p.v[i] = half_pair((r.u >> (4 * i) & 0x000F000Fu) | 0x64006400u, 1024.0f + kMidCode4);
    return p;
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
    const HalfPairs p = row_pairs(r);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = (float)p.v[i][0];
        x[i + 4] = (float)p.v[i][1];
    }
}

// <q, raw values of the row> of the lane: products of halves, which are exact, summed in fp32; half the operations of one value at a time
template <int kTier>
__device__ __forceinline__ float raw_dot(const HalfPairs& x, const QueryPiece& q) {
    const half2_t (&w)[4] = kTier == SALI_TIER_INT4 ? q.across : q.h2;
    // two short sums rather than one long one
    return __builtin_amdgcn_fdot2(w[1], x.v[1], __builtin_amdgcn_fdot2(w[0], x.v[0], 0.0f, false), false) +
           __builtin_amdgcn_fdot2(w[3], x.v[3], __builtin_amdgcn_fdot2(w[2], x.v[2], 0.0f, false), false);
}

// <q, K^_row> of the lane from the sum over its raw values: K^ = code * scale (+ zero)
__device__ __forceinline__ float finish_dot(const RawRow<SALI_TIER_FP16>&, float d, const QueryPiece&) { return d; }
__device__ __forceinline__ float finish_dot(const RawRow<SALI_TIER_INT8>& r, float d, const QueryPiece&) {
    return d * r.scale;
}
__device__ __forceinline__ float finish_dot(const RawRow<SALI_TIER_INT4>& r, float d, const QueryPiece& q) {
    return __builtin_fmaf(d, r.scale, q.sum * __builtin_fmaf(kMidCode4, r.scale, r.zero));
}

// p * V^_row = (p * scale) * code + p * zero: weight on the raw values, and the constant part
__device__ __forceinline__ float weight_of(const RawRow<SALI_TIER_FP16>&, float p) { return p; }
__device__ __forceinline__ float weight_of(const RawRow<SALI_TIER_INT8>& r, float p) { return p * r.scale; }
__device__ __forceinline__ float weight_of(const RawRow<SALI_TIER_INT4>& r, float p) { return p * r.scale; }
__device__ __forceinline__ float offset_of(const RawRow<SALI_TIER_FP16>&, float) { return 0.0f; }
__device__ __forceinline__ float offset_of(const RawRow<SALI_TIER_INT8>&, float) { return 0.0f; }
__device__ __forceinline__ float offset_of(const RawRow<SALI_TIER_INT4>& r, float p) { return p * __builtin_fmaf(kMidCode4, r.scale, r.zero); }

// online-softmax state of a lane group for one query (max and sum are equal in its 16 lanes); the
// INT4 zero-points are summed apart (zacc, the same for the lane's 8 values) and folded in at the end
struct SoftmaxState {
    float mx, lsum, zacc;
    float acc[8];
};

// Rows j0 .. j1 - 1 of one tier of one stored frame: lane group g takes rows j0 + g, j0 + 16 + g, ... (kRowsPerStep of them in
// flight, K and V each).  `base` = first pool row of the frame in this tier, `count` = its rows.  kQ queries share
// every row that is read.
template <int kTier, int kQ, int kRowsPerStep>
__device__ __forceinline__ void attend_rows(const Pools& pools, size_t plane_k, size_t plane_v, int base, int count, int j0, int j1,
                                            int g, int l, const Row16B (&raw_q)[kQ], float softmax_scale, float mult,
                                            SoftmaxState (&st)[kQ]) {
    if (j0 >= j1) return;
    const TierRows k = tier_rows<kTier>(pools, base, count, plane_k), v = tier_rows<kTier>(pools, base, count, plane_v);
    // Rows past the end repeat the last one; they count for nothing: their scores are -inf, and FP16 values are taken out, since a weight of zero
    // does not take out an infinity (quantised ones are finite, or unspecified)
    struct Step {
        RawRow<kTier> k[kRowsPerStep], v[kRowsPerStep];
    };
    auto request = [&](int jb, Step& step) {
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) load_row(k, (uint32_t)min(jb + r * 16 + g, j1 - 1), (uint32_t)l, step.k[r]);
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) load_row(v, (uint32_t)min(jb + r * 16 + g, j1 - 1), (uint32_t)l, step.v[r]);
    };
    Step next;
    request(j0, next);
    // only now, so that the first rows need not wait for the query's trip
    QueryPiece q[kQ];
#pragma unroll
    for (int iq = 0; iq < kQ; ++iq) q[iq] = query_piece(raw_q[iq]);
    for (int jb = j0; jb < j1; jb += 16 * kRowsPerStep) {
        Step now = next;
        const RawRow<kTier> (&rk)[kRowsPerStep] = now.k;
        RawRow<kTier> (&rv)[kRowsPerStep] = now.v;
        if (jb + 16 * kRowsPerStep < j1) request(jb + 16 * kRowsPerStep, next);      // under way while this step is worked on
        bool valid[kRowsPerStep];
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) valid[r] = jb + r * 16 + g < j1;
        float s[kQ][kRowsPerStep];
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) {
            const HalfPairs x = row_pairs(rk[r]);
#pragma unroll
            for (int iq = 0; iq < kQ; ++iq) {
                float d = raw_dot<kTier>(x, q[iq]);
                d = row16_sum(finish_dot(rk[r], d, q[iq]));
                s[iq][r] = valid[r] ? softmax_scale * d : -INFINITY;
            }
        }
        float p[kQ][kRowsPerStep], corr[kQ];
#pragma unroll
        for (int iq = 0; iq < kQ; ++iq) {
            float bm = -INFINITY;
#pragma unroll
            for (int r = 0; r < kRowsPerStep; ++r) bm = fmaxf(bm, s[iq][r]);
            const float new_mx = fmaxf(st[iq].mx, bm);
            // nothing seen yet for this lane group: keep the state (every weight below is exp(-inf) = 0,
            // and the reference maximum must stay finite for that)
            const float ref = new_mx == -INFINITY ? 0.0f : new_mx;
            corr[iq] = __expf(st[iq].mx - ref);             // first rows: exp(-inf) = 0
            float sum = 0.0f;
#pragma unroll
            for (int r = 0; r < kRowsPerStep; ++r) {
                p[iq][r] = mult * __expf(s[iq][r] - ref);   // absent row: exp(-inf) = 0
                sum += p[iq][r];
            }
            st[iq].lsum = __builtin_fmaf(st[iq].lsum, corr[iq], sum);
            st[iq].mx = new_mx;
        }
        if constexpr (kTier == SALI_TIER_FP16)
            if (jb + 16 * kRowsPerStep > j1)                // the last step
#pragma unroll
                for (int r = 0; r < kRowsPerStep; ++r)
                    if (!valid[r]) rv[r] = {};
        // the step's rows are added up first, so that the long sums are rounded once a step
        float sums[kQ][8], zeros[kQ];
#pragma unroll
        for (int r = 0; r < kRowsPerStep; ++r) {
            float x[8];
            row_values(rv[r], x);
#pragma unroll
            for (int iq = 0; iq < kQ; ++iq) {
                const float wgt = weight_of(rv[r], p[iq][r]);
                zeros[iq] = (r == 0 ? 0.0f : zeros[iq]) + offset_of(rv[r], p[iq][r]);
#pragma unroll
                for (int e = 0; e < 8; ++e) sums[iq][e] = r == 0 ? wgt * x[e] : __builtin_fmaf(wgt, x[e], sums[iq][e]);
            }
        }
#pragma unroll
        for (int iq = 0; iq < kQ; ++iq) {
            st[iq].zacc = __builtin_fmaf(st[iq].zacc, corr[iq], zeros[iq]);
#pragma unroll
            for (int e = 0; e < 8; ++e) st[iq].acc[e] = __builtin_fmaf(st[iq].acc[e], corr[iq], sums[iq][e]);
        }
    }
}

// Hand-over of partials inside a launch: the block of a head that is the last to arrive merges them, nobody waits.  The partials
// are written and read past the caches that the compute dies do not share (relaxed agent-scope accesses, each coherent
// by itself) and a block counts itself in only when its own have arrived, so no fence is needed: an agent-scope fence writes back and
// invalidates the L2 of the issuing die under the stream that the other blocks are reading (with one in each of
// 2000 blocks this hand-over measured 4.5 times the time of a merge kernel).
__device__ __forceinline__ void put(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float2 get_pair(const float* p) {
    return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ bool last_to_arrive(uint32_t* arrived, int head_set, int parts, int* s_last) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // every wave: its stores have arrived
    __syncthreads();
    if (threadIdx.x == 0)
        *s_last = last_arrival(atomicInc(arrived + arrival_counter(head_set, parts), (uint32_t)parts - 1u), parts) ? 1 : 0;       // relaxed, agent scope
    __syncthreads();
    return *s_last != 0;
}

// over the 64 lanes, the result in every lane: inside the rows of 16, then row by row through scalar registers
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_sum(float v) {
    v = row16_sum(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_move<0xB1>(v));
    v = fmaxf(v, dpp_move<0x4E>(v));
    v = fmaxf(v, dpp_move<0x141>(v));
    v = fmaxf(v, dpp_move<0x140>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

// A wave's share of merging the partials of a query: partials `first`, first + kStep, ... of n (at most kAttnPartials),
// whose values it adds up weighted (lane i: values 2 i, 2 i + 1); all of it in as few trips as there are: every wave reads all
// maxima itself (a lane each) while its first kFlight partials are already under way.
struct Merged {
    float big, lt;              // largest score, sum of weights
    float2 at;
};
template <int kStep, int kFlight>
__device__ __forceinline__ Merged merge_partials(const float* p, int n, int first) {
    constexpr int kPerLane = kAttnPartials / 64;
    const int lane = threadIdx.x & 63;
    float2 ml[kPerLane], v[kFlight];
    auto request = [&](int k) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) v[u] = get_pair(p + (size_t)min(k + u * kStep, n - 1) * kPartialStride + 2 + 2 * lane);
    };
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        ml[j] = make_float2(-INFINITY, 0.0f);
        if (64 * j < n) ml[j] = get_pair(p + (size_t)min(64 * j + lane, n - 1) * kPartialStride);
    }
    request(first);
    Merged r = {-INFINITY, 0.0f, {}};
    float m[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        m[j] = 64 * j + lane < n ? ml[j].x : -INFINITY;
        r.big = fmaxf(r.big, m[j]);
    }
    r.big = wave_max(r.big);
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        if (64 * j >= n) break;
        m[j] = r.big != -INFINITY ? expf(m[j] - r.big) : 0.0f;      // the partial's weight
        r.lt += 64 * j + lane < n ? m[j] * ml[j].y : 0.0f;
    }
    // four sums side by side, added up last: shorter chains, and less rounding
    float2 sum[4] = {};
    for (int k = first; k < n; k += kFlight * kStep) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int ku = k + u * kStep;
            if (ku < n) {
                const float mine = ku < 64 ? m[0] : (ku < 128 ? m[1] : (ku < 192 ? m[2] : m[3]));
                const float w = lane_value(mine, ku & 63);
                sum[u & 3].x += w * v[u].x;
                sum[u & 3].y += w * v[u].y;
            }
        }
        if (k + kFlight * kStep < n) request(k + kFlight * kStep);
    }
    r.lt = wave_sum(r.lt);
    r.at = make_float2((sum[0].x + sum[1].x) + (sum[2].x + sum[3].x), (sum[0].y + sum[1].y) + (sum[2].y + sum[3].y));
    return r;
}
static_assert(kAttnPartials == 256, "four partials a lane");

// the merged result of query head h: lane i has values 2 i, 2 i + 1 (the caller's arrays are aligned for float only)
__device__ __forceinline__ void store_result(const AttnOut& o, int h, const Merged& r) {
    const int lane = threadIdx.x & 63;
    float* dst = o.out + (size_t)h * kHeadDim + 2 * lane;
    dst[0] = r.lt > 0.0f ? r.at.x / r.lt : 0.0f;
    dst[1] = r.lt > 0.0f ? r.at.y / r.lt : 0.0f;
    if (o.lse != nullptr && lane == 0) o.lse[h] = r.lt > 0.0f ? r.big + logf(r.lt) : -INFINITY;
}

}  // namespace

// blocks of the streaming kernel that fit a compute unit, by the registers that kQ queries take
constexpr int blocks_per_unit(int kq) { return kq == 4 ? 2 : 4; }

// Blocks: parts of the frame range x n_heads x sets, dealt so that a compute die works on one stretch of the range for all heads
// (xcd_block_id with the part as the slowest index): a frame's rows of a layer are contiguous over the heads, and each die then
// touches an eighth of the pages.  32 heads, 20 frames: 29.5 us with twelve or twenty parts in launch order, 24.8 with sixteen, which fall that
// way by themselves.  Block `part` takes the stretch [part * n, (part + 1) * n) of the range's n frames in
// units of 1 / parts frame, a frame's part of it the same fraction of its groups of 16 rows, for kQ of the query heads that share the K/V
// head (`sets` such sets: q_per_kv = kQ * sets), and writes one partial per query head; kInLaunch: the head's last block merges them.
template <int kQ, int kRowsPerStep, bool kInLaunch>
__global__ __launch_bounds__(256, blocks_per_unit(kQ)) void k_attn_partial(
    const sali_frame_row* __restrict__ rows, const _Float16* __restrict__ q, float* __restrict__ partial, int layer, int n_heads, int sets,
    int frame_lo, int frame_hi, int tiles, int parts, float softmax_scale, Pools pools, AttnOut result) {
    __shared__ float s_m[kQ][16], s_l[kQ][16];
    __shared__ __align__(16) float s_acc[kQ][16][kHeadDim];
    __shared__ int s_last;

    const BlockId blk = xcd_block_id((int)blockIdx.x, n_heads * sets, 1, parts);
    const int group = blk.x, part = blk.z;
    const int h = sets == 1 ? group : group / sets;
    const int q_first = group * kQ;                             // first query head of this block
    const long long n = frame_hi - frame_lo;
    const int f0 = frame_lo + (int)((uint32_t)part * (uint32_t)n / (uint32_t)parts);        // below 2^32: part < 256, n <= 2^24
    together(pools.p16, pools.c8, pools.s8, pools.c4, pools.s4, pools.z4, pools.n_planes, result.out, result.lse, result.arrived);
    const int g = threadIdx.x >> 4, l = threadIdx.x & 15;
    const size_t plane_k = ((size_t)layer * 2 + 0) * n_heads + h;
    const size_t plane_v = ((size_t)layer * 2 + 1) * n_heads + h;

    Row16B raw_q[kQ];
    SoftmaxState st[kQ];
#pragma unroll
    for (int iq = 0; iq < kQ; ++iq) {
        raw_q[iq].u = reinterpret_cast<const u32x4*>(q)[(q_first + iq) * 16 + l];
        st[iq].mx = -INFINITY;
        st[iq].lsum = 0.0f;
        st[iq].zacc = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) st[iq].acc[e] = 0.0f;
    }

    for (int f = f0; f < frame_hi; ++f) {
        // the block's part of the frame, in units of 1 / parts
        const long long at = (long long)(f - frame_lo) * parts, from = part * n - at, to = from + n;
        if (to <= 0) break;
        const int lo = from > 0 ? (int)(from < parts ? from : parts) : 0, hi = to < parts ? (int)to : parts;
        if (lo >= hi) continue;
        // Which stored frame does frame f bring in, and how many times?  A stored frame counts for
        // itself and for the redundant frames behind it (up to the next stored frame or the end of
        // the range); redundant frames at the head of the range, whose source lies before it, are
        // counted at the first of them.  With `tiles` entries per video frame all of this goes by the entries
        // of the same tile, which lie `tiles` apart.  Every thread takes the same decision from the same
        // (uniform) table reads; the two that nearly always decide it are asked for together.
        sali_frame_row row = rows[f];
        const bool followed = f + tiles < frame_hi;
        const int next_stored = rows[followed ? f + tiles : f].stored;
        together(row.stored, row.src, row.base16, row.n16, next_stored);
        bool leader = row.stored != 0;
        const int src = row.src;
        if (!leader) {
            if (src >= 0 && src < frame_lo) {
                leader = true;
                for (int t = f - tiles; leader && t >= frame_lo; t -= tiles)
                    leader = rows[t].src != src;                   // an earlier frame of the run counts them
            }
            if (!leader) continue;
            row = rows[src];
        }
        int n_uses = 1;
        if (followed && next_stored == 0)
            for (int t = f + tiles; t < frame_hi && rows[t].stored == 0; t += tiles)
                if (rows[t].src == src) ++n_uses;
        const float mult = (float)n_uses;
        // groups of 16 rows, tier after tier; the block's are u0 .. u1 - 1
        const int t16 = (row.n16 + 15) / 16, t8 = (row.n8 + 15) / 16, t4 = (row.n4 + 15) / 16, all = t16 + t8 + t4;
        const int u0 = (int)((uint32_t)(all * lo) / (uint32_t)parts), u1 = (int)((uint32_t)(all * hi) / (uint32_t)parts);
        auto rows_of = [&](int before, int groups, int count, int& j0, int& j1) {
            j0 = 16 * max(u0 - before, 0);
            j1 = min(16 * min(u1 - before, groups), count);
        };
        int j0, j1;
        rows_of(0, t16, row.n16, j0, j1);
        attend_rows<SALI_TIER_FP16, kQ, kRowsPerStep>(pools, plane_k, plane_v, row.base16, row.n16, j0, j1, g, l, raw_q, softmax_scale, mult, st);
        rows_of(t16, t8, row.n8, j0, j1);
        attend_rows<SALI_TIER_INT8, kQ, kRowsPerStep>(pools, plane_k, plane_v, row.base8, row.n8, j0, j1, g, l, raw_q, softmax_scale, mult, st);
        rows_of(t16 + t8, t4, row.n4, j0, j1);
        attend_rows<SALI_TIER_INT4, kQ, kRowsPerStep>(pools, plane_k, plane_v, row.base4, row.n4, j0, j1, g, l, raw_q, softmax_scale, mult, st);
    }

    // merge the 16 lane groups, all query heads together
#pragma unroll
    for (int iq = 0; iq < kQ; ++iq) {
        if (l == 0) {
            s_m[iq][g] = st[iq].mx;
            s_l[iq][g] = st[iq].lsum;
        }
#pragma unroll
        for (int e = 0; e < 8; e += 4)
            *reinterpret_cast<float4*>(&s_acc[iq][g][8 * l + e]) =
                make_float4(st[iq].acc[e] + st[iq].zacc, st[iq].acc[e + 1] + st[iq].zacc, st[iq].acc[e + 2] + st[iq].zacc,
                            st[iq].acc[e + 3] + st[iq].zacc);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (kQ * kHeadDim + 255) / 256; ++i) {
        const int idx = (int)threadIdx.x + 256 * i, iq = idx / kHeadDim, d = idx % kHeadDim, head = q_first + iq;
        if (iq >= kQ) break;                // one query: half of the block
        float big = -INFINITY;
#pragma unroll
        for (int k = 0; k < 16; ++k) big = fmaxf(big, s_m[iq][k]);
        float lts[4] = {}, ats[4] = {};
        if (big != -INFINITY) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const float w = __expf(s_m[iq][k] - big);
                lts[k & 3] += w * s_l[iq][k];
                ats[k & 3] += w * s_acc[iq][k][d];
            }
        }
        const float lt = (lts[0] + lts[1]) + (lts[2] + lts[3]), at = (ats[0] + ats[1]) + (ats[2] + ats[3]);
        if (parts > 1) {
            float* mine = partial + ((size_t)head * kAttnPartials + part) * kPartialStride;
            if (d == 0) {
                put(mine, big);
                put(mine + 1, lt);
            }
            put(mine + 2 + d, at);
        } else {
            result.out[(size_t)head * kHeadDim + d] = lt > 0.0f ? at / lt : 0.0f;
            if (result.lse != nullptr && d == 0) result.lse[head] = lt > 0.0f ? big + logf(lt) : -INFINITY;
        }
    }
    if constexpr (kInLaunch) {
        if (parts == 1 || !last_to_arrive(result.arrived, group, parts, &s_last)) return;
        // four waves: all of them on the one query, two on each of two, one on each of four
        constexpr int kWaves = 4 / kQ;
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), iq = wave / kWaves, sub = wave % kWaves;
        Merged r = merge_partials<kWaves, kQ == 4 ? 32 : 16>(partial + (size_t)(q_first + iq) * kAttnPartials * kPartialStride, parts,
                                                             min(sub, parts - 1));
        if constexpr (kWaves > 1) {
            // (with fewer partials than waves the last one is taken more than once: once too often)
            float2* s_part = reinterpret_cast<float2*>(&s_acc[0][0][0]);
            s_part[threadIdx.x] = sub < parts ? r.at : make_float2(0.0f, 0.0f);
            __syncthreads();
            if (sub != 0) return;
#pragma unroll
            for (int k = 1; k < kWaves; ++k) {
                const float2 other = s_part[threadIdx.x + 64 * k];
                r.at.x += other.x;
                r.at.y += other.y;
            }
        }
        store_result(result, q_first + iq, r);
    }
}

// The merge as a launch of its own: `parts` partials of `slots` reserved for each of n_q queries, kWaves waves a query.  All of a
// query's partials are under way at once: up to 8 with one wave, 32 with four, 128 with sixteen.
template <int kWaves>
__global__ __launch_bounds__(kWaves < 4 ? 256 : 64 * kWaves) void k_attn_merge(const float* __restrict__ partial, int parts, int slots, int n_q,
                                                                             AttnOut result) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, sub = wave % kWaves;
    const int h = kWaves < 4 ? (int)blockIdx.x * 4 + wave : (int)blockIdx.x;
    if (h >= n_q) return;
    Merged r = merge_partials<kWaves, 8>(partial + (size_t)h * slots * kPartialStride, parts, min(sub, parts - 1));
    if constexpr (kWaves > 1) {
        __shared__ float2 s_part[kWaves][64];
        s_part[sub][lane] = r.at;
        __syncthreads();
        if (sub != 0) return;
#pragma unroll
        for (int k = 1; k < kWaves; ++k) {
            if (k >= parts) break;              // with fewer partials than waves the last one is taken more than once
            r.at.x += s_part[k][lane].x;
            r.at.y += s_part[k][lane].y;
        }
    }
    store_result(result, h, r);
}

// an empty range: zeros and -inf
__global__ __launch_bounds__(256) void k_attn_empty(AttnOut result, int n_q_heads) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n_q_heads * kHeadDim) result.out[i] = 0.0f;
    if (result.lse != nullptr && i < n_q_heads) result.lse[i] = -INFINITY;
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
// single-query kernel; a launch of its own merges them.
//
// What bounds it: the trip to memory of a tile (waves wait for 47 % of their time), then the vector
// instructions of a tile (610, conversions and softmax).  Hence: a tile's K^ and V^ rows are asked for a
// whole tile ahead, across tiers and frames; the launch is one block of eight waves per compute unit, forced
// to one by its LDS, so that all start at once; and a block writes one partial instead of one per wave.
// 32 heads x 32 queries over 20 frames (173 / 200 / 203 rows, 118 MB): 32.2 us a call, of which tiles stream for 19 at 6.1 TB/s; 34.6 with
// the merge in the launch (in_launch_parts), 36.1 with 64-bit divisions in the list of frames.  The same tiles as 512 independent blocks of four waves that should just have fitted twice per compute unit, a
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
__device__ __forceinline__ int pf_list_frames(const sali_frame_row* __restrict__ rows, int frame_lo, int frame_hi, int tiles, int g0, int f_end, int part, int parts, int lane, int* s_src, PfFrame* list,
                                              int* n_tiles) {
    // entries past the share's are looked at too: which of them is stored next says how often the last ones count
    const int f = g0 + lane, g_end = min(f_end, g0 + kPfGroup), seen = min(frame_hi, g0 + kPfGroup);
    const bool valid = f < g_end;
    sali_frame_row row = {};
    row.src = -1;
    if (f < seen) row = rows[f];
    s_src[lane] = row.src;
    pf_lds_order();
    const unsigned long long stored_mask = __ballot(f < seen && row.stored != 0);
    const bool stored = valid && row.stored != 0;
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
        const int run_end = behind != 0ull ? f + tiles + __builtin_ctzll(behind) : seen;
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
        if (hi > lo) {                                      // both in 0 .. parts
            i0 = (int)((uint32_t)(t * (int)lo) / (uint32_t)parts);
            cnt = (int)((uint32_t)(t * (int)hi) / (uint32_t)parts) - i0;
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

// parts of the frame range x n_heads x ceil(q_per_kv / 32) blocks of 512 threads.  kLongRange: a stored frame of the
// range may count more than 2^15 times, which takes more than 2^15 frames
template <bool kLongRange>
__global__ __launch_bounds__(64 * kPfWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_prefill(
    const sali_frame_row* __restrict__ rows, const _Float16* __restrict__ q, float* __restrict__ partial, int layer, int n_heads, int sets,
    int q_per_kv, int frame_lo, int frame_hi, int tiles, int parts, float softmax_scale, Pools pools, AttnOut result) {
    __shared__ __align__(16) _Float16 s_tiles[kPfWaves][kPfTileHalves];     // a K^ and a V^ tile per wave; the results at the end
    __shared__ PfFrame s_list[kPfGroup];
    __shared__ int s_src[kPfGroup];
    __shared__ int s_n[2];
    __shared__ float s_m[kPfWaves][32], s_l[kPfWaves][32];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int m = lane & 31, hh = lane >> 5;
    const BlockId blk = xcd_block_id((int)blockIdx.x, n_heads * sets, 1, parts);        // as in k_attn_partial
    const int group = blk.x, part = blk.z;
    const int h = sets == 1 ? group : group / sets, set = group - h * sets;
    together(pools.p16, pools.c8, pools.s8, pools.c4, pools.s4, pools.z4, pools.n_planes, result.out, result.lse);
    const int qi = set * 32 + m;                 // this lane's query among the q_per_kv of the K/V head
    const size_t plane_k = ((size_t)layer * 2 + 0) * n_heads + h;
    const size_t plane_v = ((size_t)layer * 2 + 1) * n_heads + h;
    _Float16* s_k = s_tiles[wave];
    _Float16* s_v = s_k + kPfRows * kPfKStride;

    // the stretch's frames, the last one rounded up; products below 2^32 (part < 256, at most 2^24 frames)
    const uint32_t n_range = (uint32_t)(frame_hi - frame_lo);
    const int f_begin = frame_lo + (int)((uint32_t)part * n_range / (uint32_t)parts);
    const int f_end = frame_lo + (int)(((uint32_t)(part + 1) * n_range - 1u) / (uint32_t)parts) + 1;
    auto list_frames = [&](int g0) {
        if (wave != 0) return;
        int n_tiles;
        const int len = pf_list_frames(rows, frame_lo, frame_hi, tiles, g0, f_end, part, parts, lane, s_src, s_list, &n_tiles);
        if (lane == 0) {
            s_n[0] = len;
            s_n[1] = n_tiles;
        }
    };
    list_frames(f_begin);       // ahead of the queries: it is what every wave waits for

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

    for (int g0 = f_begin; g0 < f_end; g0 += kPfGroup) {
        if (g0 != f_begin) {
            __syncthreads();                                // every wave is through with the list
            list_frames(g0);
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
    const int queries = min(q_per_kv - set * 32, 32);
    const int q_first = h * q_per_kv + set * 32;
    float* first_partial = partial + ((size_t)q_first * parts + part) * kPartialStride;      // `parts` per query
    if (wave == 0 && hh == 0 && m < queries) {
        float lt = 0.0f;
        if (big != -INFINITY)
#pragma unroll
            for (int w = 0; w < kPfWaves; ++w) lt += s_l[w][m] * __builtin_amdgcn_exp2f(s_m[w][m] - big);
        const float natural = big * 0.69314718055994530942f;
        if (parts > 1) {
            first_partial[(size_t)m * parts * kPartialStride] = natural;
            first_partial[(size_t)m * parts * kPartialStride + 1] = lt;
        } else {
            s_l[0][m] = lt;
            if (result.lse != nullptr) result.lse[q_first + m] = lt > 0.0f ? natural + logf(lt) : -INFINITY;
        }
    }
    if (parts == 1) __syncthreads();
    constexpr int kOuts = 32 * kHeadDim / (64 * kPfWaves);
    float sum[kOuts];
#pragma unroll
    for (int i = 0; i < kOuts; ++i) {
        const int idx = (int)threadIdx.x + i * 64 * kPfWaves, mm = idx / kHeadDim, d = idx % kHeadDim;
        sum[i] = 0.0f;
#pragma unroll
        for (int w = 0; w < kPfWaves; ++w) sum[i] += reinterpret_cast<const float*>(s_tiles[w])[d * kPfOutStride + mm];
    }
#pragma unroll
    for (int i = 0; i < kOuts; ++i) {
        const int idx = (int)threadIdx.x + i * 64 * kPfWaves, mm = idx / kHeadDim, d = idx % kHeadDim;
        if (mm >= queries) continue;
        if (parts > 1) {
            first_partial[(size_t)mm * parts * kPartialStride + 2 + d] = sum[i];
        } else {
            const float lt = s_l[0][mm];
            result.out[(size_t)(q_first + mm) * kHeadDim + d] = lt > 0.0f ? sum[i] / lt : 0.0f;
        }
    }
}

// Does the last block of a head merge its parts, or a launch of its own?  In the launch one block reads them all: that saves a launch, on the GPU
// (one query a head: 4 to 16 parts 5.4 against 6.6 us a call, 128 parts 8.7 against 9.0) and on the host (32 calls of 4 queries a head and 32 parts
// 273 against 307 us, the host's time, though 9.3 against 8.4 us each on the GPU), until its compute unit is what the call waits for (two
// queries: 32 parts 7.1 either way, 74 parts 8.6 against 7.8, 256 parts 17.2 against 13.3; four: 37 parts 9.5 against 8.1, 64 parts 11.8 against
// 9.8, so only in the short calls where the host's time counts, those that take a row at a time).  32 queries behind the matrix cores gain nothing from eight parts on (32 heads x 24 frames 40.6 against 39.8) and lose by the number of
// parts: 11 parts 15.4 against 10.7, 63 parts 29.8 against 12.4.
constexpr int in_launch_parts(int kq, bool one_row) { return kq == 1 ? kAttnPartials : (kq == 2 ? 64 : (one_row ? 32 : 1)); }

// Parts where there are more heads x sets than half of the compute units: equal loads for the units, at least nearly two blocks each; a block more
// costs little.  320 sets of 4 queries x 8 frames 205.9 us with one part (a unit in four has two blocks), 132.4 with four; 160 heads x 8 frames
// 48.1 with six, 45.6 with three; 200 sets 108.9 with two, 89.1 with five.
static int balanced_parts(int pairs, int kq) {
    int best = 1;
    double least = INFINITY;
    for (int p = 1; p <= 8; ++p) {
        const double blocks = (double)p * pairs / kComputeUnits;
        const double cost = ceil(blocks) / blocks + (kq == 4 ? 0.03 : 0.06) * blocks;
        if (blocks >= 1.8 && cost < least) {
            least = cost;
            best = p;
        }
    }
    return best;
}

static void launch_merge(const float* d_partial, int parts, int slots, int n_q, const AttnOut& result, hipStream_t s) {
    if (parts <= 8) hipLaunchKernelGGL(k_attn_merge<1>, dim3((n_q + 3) / 4), dim3(256), 0, s, d_partial, parts, slots, n_q, result);
    else if (parts <= 32) hipLaunchKernelGGL(k_attn_merge<4>, dim3(n_q), dim3(256), 0, s, d_partial, parts, slots, n_q, result);
    else hipLaunchKernelGGL(k_attn_merge<16>, dim3(n_q), dim3(1024), 0, s, d_partial, parts, slots, n_q, result);
}

hipError_t launch_attend(const sali_frame_row* d_rows, const Pools& pools, int layer, int n_heads, int q_per_kv,
                         const void* d_q, int frame_lo, int frame_hi, int tiles, RowsPerFrame kept, float softmax_scale, float* d_partial,
                         AttnOut result, hipEvent_t ev_start, hipEvent_t ev_stop, hipStream_t s) {
    const int n_range = frame_hi - frame_lo;
    const _Float16* q = reinterpret_cast<const _Float16*>(d_q);
    if (n_range <= 0) {
        const int n_q_heads = n_heads * q_per_kv;
        hipLaunchKernelGGL(k_attn_empty, dim3((n_q_heads * kHeadDim + 255) / 256), dim3(256), 0, s, result, n_q_heads);
        return hipGetLastError();
    }
    if (ev_start != nullptr && hipEventRecord(ev_start, s) != hipSuccess) return hipErrorUnknown;
    int parts, slots;               // partials per query, made and reserved
    bool merged;                    // the launch leaves results
    if (q_per_kv > kAttnMaxQPerKv) {
        // matrix-core path: one block of eight waves per compute unit, as many parts of the range as that
        // gives a K/V head, but no more than leave every wave a tile (a frame has up to kTokens / kPfRows + 3),
        // and no more partials than the scratch holds (kAttnSlotsPerHead per K/V head, shared out over its queries).
        // Where one part each would leave a third of the compute units or more idle, three parts each: two rounds
        // of a third of the work.  160 heads x 9 queries x 20 frames 168 -> 133 us a call, 129 heads 167 -> 125
        // (independent blocks of four waves: 141 and 162)
        const int sets = (q_per_kv + 31) / 32, pairs = n_heads * sets;
        parts = kComputeUnits / pairs;
        if (parts == 1 && 3 * pairs <= 2 * kComputeUnits) parts = 3;
        const long long fill = ((long long)n_range * (kTokens / kPfRows + 3) + kPfWaves - 1) / kPfWaves;
        if (parts > fill) parts = (int)fill;
        if (parts > kAttnSlotsPerHead / q_per_kv) parts = kAttnSlotsPerHead / q_per_kv;
        if (parts > kAttnPartials) parts = kAttnPartials;
        if (parts < 1) parts = 1;
        slots = parts;
        merged = parts == 1;
        const dim3 grid(parts * n_heads * sets);
        // the general variant costs 0.7 % (32 heads x 32 queries x 20 frames 143.8 -> 144.8 us for four layers)
        if (n_range > 32768)
            hipLaunchKernelGGL(k_attn_prefill<true>, grid, dim3(64 * kPfWaves), 0, s, d_rows, q, d_partial, layer, n_heads, sets, q_per_kv,
                               frame_lo, frame_hi, tiles, parts, softmax_scale, pools, result);
        else
            hipLaunchKernelGGL(k_attn_prefill<false>, grid, dim3(64 * kPfWaves), 0, s, d_rows, q, d_partial, layer, n_heads, sets, q_per_kv,
                               frame_lo, frame_hi, tiles, parts, softmax_scale, pools, result);
    } else {
        // eight queries per K/V head run as two sets of four (two blocks read the same rows, the second
        // mostly from cache): a block with eight query states needs 256 registers per lane and was slower
        const int kq = q_per_kv == 8 ? 4 : q_per_kv, sets = q_per_kv / kq;
        // Whole rounds of one block per compute unit, as nearly as the parts allow (a unit with one block more than the others is
        // where the launch ends: 20 frames x 32 heads 25.6 us with 16 parts, 28.9 with 20, 26.5 with 24): two from sixteen
        // heads x sets on; one below, where more parts cost more at the merge than they bring (8 heads x 4 queries x 20 frames 19.6 us
        // with 32 parts, 21.2 with 64); no more than 128 for one head (24 frames 9.6 us, 11.8 with 256).  Shares of a block: two groups of 16 rows
        // or more; one where 64 blocks have them all (one flight of the merge: a head x 56 groups x 4 queries 8.1 us, with two a block 8.8, but
        // 148 groups 10.0 and 9.4); eight or more where heads x sets fill half the chip alone (160 heads x 14 groups 8.1 us with
        // one part, 11.2 with six).  Shares of up to two groups are taken a row per lane group at a time, others four: 4 heads x 74 groups x 4 queries
        // 9.0 and 10.9 us.
        const int pairs = n_heads * sets;
        const int groups = (kept.n16 + 15) / 16 + (kept.n8 + 15) / 16 + (kept.n4 + 15) / 16;
        const long long work = (long long)n_range * (groups < 4 ? 4 : groups);      // not fewer than four: frames stored under an earlier rule
        const long long most = work <= 64 && work * pairs <= kComputeUnits ? work : (pairs > 128 ? work / 8 : (work + 1) / 2);
        parts = pairs > 128 ? balanced_parts(pairs, kq) : kComputeUnits * (pairs >= 16 ? 2 : 1) / pairs;
        if (parts > 128) parts = 128;
        if (parts > most) parts = (int)most;
        if (parts < 1) parts = 1;
        const bool one_row = work <= 2 * parts;
        slots = kAttnPartials;
        merged = parts <= in_launch_parts(kq, one_row);
        const dim3 grid(parts * n_heads * sets);
        auto go = [&](auto queries) {
            constexpr int kQ = decltype(queries)::value;
            auto* const kernel = one_row ? (merged ? k_attn_partial<kQ, 1, true> : k_attn_partial<kQ, 1, false>)
                                         : (merged ? k_attn_partial<kQ, 4, true> : k_attn_partial<kQ, 4, false>);
            hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, d_rows, q, d_partial, layer, n_heads, sets, frame_lo, frame_hi, tiles, parts,
                               softmax_scale, pools, result);
        };
        switch (kq) {
            case 1: go(std::integral_constant<int, 1>{}); break;
            case 2: go(std::integral_constant<int, 2>{}); break;
            case 4: go(std::integral_constant<int, 4>{}); break;
            default: return hipErrorInvalidValue;
        }
    }
    if (ev_stop != nullptr && hipEventRecord(ev_stop, s) != hipSuccess) return hipErrorUnknown;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || merged) return e;
    launch_merge(d_partial, parts, slots, n_heads * q_per_kv, result, s);
    return hipGetLastError();
}

}  // namespace sali
