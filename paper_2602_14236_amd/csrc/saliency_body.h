// The spatial filter's per-block bodies: the pre-pass over a tile, the cross-tile hysteresis of a batch and the score of a
// patch.  Shared by the kernels of saliency_kernels.hip and by launches of the temporal filter that they ride on (small
// frames: the two filters need nothing from each other until the gate).  Integer arithmetic throughout, so
// nothing depends on floating-point contraction.
#pragma once

#include "hysteresis.h"
#include "sali_internal.h"

namespace sali {

constexpr int kHalo = 4;
constexpr int kReg = kTile + 2 * kHalo;        // 40: gray region
constexpr int kRegB = kTile + 4;               // 36: blur / LAB region (halo 2)
constexpr int kRegM = kTile + 2;               // 34: gradient-magnitude region (halo 1)


// #{dP_i < tau_t} over the thread's share of one image's 576 patch motions (block of NT threads); the
// loads are independent and issued together
template <int NT>
__device__ __forceinline__ int count_static(const float* dp, float tau_t) {
    constexpr int kPer = (kTokens + NT - 1) / NT;
    float v[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = (int)threadIdx.x + NT * k;
        v[k] = i < kTokens ? __hip_atomic_load(dp + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tau_t;
    }
    int n = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) n += v[k] < tau_t ? 1 : 0;
    return n;
}

// Eq. 6 and the reuse rule for frame b of a launch, evaluated by a whole block of NT threads from the
// per-patch motions that an earlier kernel left (frames[b].dp NULL: no predecessor, never redundant): the
// kernels of the spatial filter ask this first and leave at once for a redundant frame (Algorithm 1
// skips its saliency).  Same counts and the same fp32 quotient as the tail kernel that writes the gate,
// so all of them take the same decision.  s_cnt: NT / 64 ints of LDS.
template <int NT, typename Frame>
__device__ __forceinline__ bool frame_redundant(const Frame* frames, int b, const GateParams& gp, int* s_cnt) {
    const int b0 = b - b % gp.tiles;
    if (frames[b0].dp == nullptr) return false;
    int n = 0;
    for (int j = 0; j < gp.tiles; ++j) n += count_static<NT>(frames[b0 + j].dp, gp.tau_t);
    for (int off = 32; off > 0; off >>= 1) n += __shfl_down(n, off);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = n;
    __syncthreads();
    int n_static = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) n_static += s_cnt[k];
    __syncthreads();
    return (float)n_static / (float)(kTokens * gp.tiles) > gp.theta_r;
}

// A block per 32x32 tile: 256 threads in the chained step, so that blocks find room on compute units that a bandwidth
// kernel of another stream keeps busy; 512 or 1024 in the stand-alone call and where it rides on blocks of that size.
//
// Four 1920x1080 frames: 97 us (103 before the last instructions were taken out), sixteen 640x360 frames 37 (40.6), one 10.3 on 1024
// threads; bound by the vector ALU (76 % of the cycles of a busy compute unit, 288 instructions a pixel; the LDS 37 %), then by the trips of
// a block's stages (image and tables from memory, then LDS; seven blocks per compute unit).  Taken tap by tap, byte
// by byte, with clamped coordinates, the stencils were 612 instructions per pixel instead of 305, the ALU
// 90 % busy, and the kernel took 150 and 24 us.  So each
// stage takes strips of four pixels as words: byte dot products along rows, packed 16-bit arithmetic down
// columns, separable sums kept in LDS where neighbouring rows share them, gradients as 16-bit pairs whose
// squared magnitude is one dot product.  No stage clamps coordinates: a cell outside the image holds what the
// definition wants to see there (gray and colour of the clamped coordinate as loaded; blurred values copied
// from the clamped cell, gradient 0), which only blocks on the image border have to arrange.
constexpr int kPrepThreads = 256, kPrepMaxThreads = 1024;
constexpr int kQuadsY = kReg / 4;                                              // 10 quads of a gray row
constexpr int kStripsB = kRegB / 4;                                            // 9 strips of a blurred row
constexpr int kGradW = 36;                                                     // gradient row: 34 cells, whole strips
constexpr int kLutWords = kColourLutBytes / 4;
static_assert(kLutWords % 4 == 0, "tables are copied sixteen bytes at a time");
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

struct PrepShared {
    // the colour tables; from the blur's second pass on the row sums of the colour variance; in the hysteresis
    // the contacts of runs
    union {
        __attribute__((aligned(16))) uint32_t lut[kLutWords];
        uint32_t contact[2 * kTile * kTile];
        struct {
            uint4 sq[kRegB][kTile / 4];
            uint2 s[3][kRegB][kTile / 4];
        } var;
    };
    // gray image and its row sums, then the blurred image in place of the gray one; from the hysteresis on the tile's union-find
    // links (key = local index | weak bit)
    union {
        struct {
            union {
                uint32_t y[kReg][kQuadsY];
                uint32_t b[kRegB][kStripsB];
                uint8_t b8[kRegB][kRegB];
            };
            uint2 h[kReg][kStripsB];
        } gray;
        uint32_t lbl[kTile * kTile];
    };
    // LAB values; once their row sums are taken the gradients, (gx, gy) as 16-bit halves
    union {
        __attribute__((aligned(16))) uint8_t lab[3][kRegB][kRegB];
        __attribute__((aligned(16))) uint32_t grad[kRegM][kGradW];
    };
    uint32_t sum[kPrepMaxThreads / 32];
    int gate[kPrepMaxThreads / 64];
    uint32_t row[kTile];        // a tile row's edge candidates, a bit each
    uint32_t n_contacts;
};

// bytes i and i + 1 of the eight in (lo, hi) as 16-bit halves
__device__ __forceinline__ short2_t byte_pair(uint32_t lo, uint32_t hi, int i) {
    const uint32_t sel = 0x0c000c00u | (uint32_t)i | ((uint32_t)(i + 1) << 16);
    return __builtin_bit_cast(short2_t, __builtin_amdgcn_perm(hi, lo, sel));
}
__device__ __forceinline__ uint32_t dot2(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, a), __builtin_bit_cast(ushort2_t, b), c, false);
}
__device__ __forceinline__ int grad_m2(uint32_t g) {
    const short2_t v = __builtin_bit_cast(short2_t, g);
    return __builtin_amdgcn_sdot2(v, v, 0, false);
}

// Tile (bx, by) of frame bz of the batch, by a block of NT (256, 512 or 1024) threads.  kGated: frames that the reuse rule finds redundant are
// left out; without it (a launch that runs before the flow) all are done.
template <bool kGated, int NT>
__device__ __forceinline__ void prep_tile(PrepShared& sh, const PrepBatch& f, int bx, int by, int bz, int h, int w, const GateParams& gp,
                                          const uint32_t* __restrict__ lut_words, int lo2, int hi2) {
    const PrepFrame& frame = f.frame[bz];
    const uint8_t* __restrict__ rgb = frame.rgb;
    uint8_t* __restrict__ cls_out = frame.cls;
    uint32_t* __restrict__ var_out = frame.var;
    uint32_t* __restrict__ parent_out = frame.parent;
    unsigned long long* msum_acc = frame.msum_acc;
    unsigned long long* msum_clear = frame.msum_clear;
    constexpr int kPrepPx = kTile * kTile / NT;                          // pixels of the tile per thread
    constexpr int kPrepQuads = (kReg * kQuadsY + NT - 1) / NT;           // quads of the region per thread
    constexpr int kLutQuads = (kLutWords / 4 + NT - 1) / NT;
    uint32_t (&s_lbl)[kTile * kTile] = sh.lbl;

    const int tid = threadIdx.x;
    const int x0 = bx * kTile, y0 = by * kTile;
    const bool border = x0 == 0 || y0 == 0 || x0 + kTile + kHalo > w || y0 + kTile + kHalo > h;      // uniform

    if (bx == 0 && by == 0 && tid == 0 && msum_clear != nullptr) *msum_clear = 0ull;

    // stage 1a: RGB of the 40x40 region, four pixels (twelve bytes at any address) at a time, coordinates clamped.
    // These loads and those of the colour tables are issued before the reuse rule is looked at, so that its
    // memory round trip and theirs overlap: most frames are not redundant.
    uint32_t crgb[kPrepQuads][3];
#pragma unroll
    for (int k = 0; k < kPrepQuads; ++k) {
        const int p = min(tid + k * NT, kReg * kQuadsY - 1);
        const int x = x0 - kHalo + 4 * (p % kQuadsY);
        load_rgb_quad(rgb + __umul24((uint32_t)clampi(y0 - kHalo + p / kQuadsY, 0, h - 1), 3u * (uint32_t)w), x, w, crgb[k]);
    }
    u32x4 lut[kLutQuads];
#pragma unroll
    for (int k = 0; k < kLutQuads; ++k)
        lut[k] = reinterpret_cast<const u32x4*>(lut_words)[min(tid + k * NT, kLutWords / 4 - 1)];
    {
        // no saliency for a redundant frame; the frame's first block leaves the decision for the kernels
        // after this one, whose blocks are too small to count 576 patches each
        bool skip = false;
        if constexpr (kGated) skip = frame_redundant<NT>(f.frame, bz, gp, sh.gate);
        if (bx == 0 && by == 0 && tid == 0) *frame.skip = skip ? 1u : 0u;
        if (skip) return;
    }
    // colour tables -> LDS, gray of the region
#pragma unroll
    for (int k = 0; k < kLutQuads; ++k) {
        const int i = tid + k * NT;
        if (i < kLutWords / 4) reinterpret_cast<u32x4*>(sh.lut)[i] = lut[k];
    }
#pragma unroll
    for (int k = 0; k < kPrepQuads; ++k) {
        const int p = tid + k * NT;
        if (p < kReg * kQuadsY) sh.gray.y[p / kQuadsY][p % kQuadsY] = gray_of_quad(crgb[k]);
    }
    __syncthreads();

    // stage 1b: 8-bit LAB of the 36x36 region through the LDS tables
    {
        const uint16_t* s_lin = reinterpret_cast<const uint16_t*>(sh.lut);
        const uint16_t* s_fl = s_lin + 256;
        const uint8_t* s_l8 = reinterpret_cast<const uint8_t*>(s_fl + 4096);
#pragma unroll
        for (int k = 0; k < kPrepQuads; ++k) {
            const int p = tid + k * NT;
            const int ry = p / kQuadsY - 2, quad = p % kQuadsY;          // row of the region, cells 4 quad - 2 ..
            if (ry < 0 || ry >= kRegB) continue;
            // four pixels: L a byte each; a and b in 16.16, the whole part a half each, clamped and packed by pairs
            uint32_t lab[3] = {0u, 0u, 0u};
            int ab[2][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                auto byte = [&](int j) { return (crgb[k][j >> 2] >> (8 * (j & 3))) & 0xFFu; };
                const uint32_t rg = (uint32_t)s_lin[byte(3 * i)] | ((uint32_t)s_lin[byte(3 * i + 1)] << 16), lb = s_lin[byte(3 * i + 2)];
                auto row = [&](uint32_t of_r, uint32_t of_g, uint32_t of_b) {
                    return dot2(rg, of_r | (of_g << 16), __umul24(lb, of_b) + 2048u) >> 12;
                };
                const uint32_t tx = row(1777u, 1541u, 778u), ty = row(871u, 2929u, 296u), tz = row(73u, 448u, 3575u);
                const int fx = s_fl[tx], fy = s_fl[ty], fz = s_fl[tz];
                lab[0] |= (uint32_t)s_l8[ty] << (8 * i);
                ab[0][i] = __mul24(1000, fx - fy) + 2 * (4194304 + 16384);
                ab[1][i] = __mul24(400, fy - fz) + 2 * (4194304 + 16384);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const short2_t none = {0, 0}, all = {255, 255};
                auto whole = [&](int i) {
                    const short2_t v = __builtin_bit_cast(short2_t, __builtin_amdgcn_perm((uint32_t)ab[c][i + 1], (uint32_t)ab[c][i], 0x07060302u));
                    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_elementwise_max(v, none), all));
                };
                lab[1 + c] = __builtin_amdgcn_perm(whole(2), whole(0), 0x06040200u);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                uint16_t* dst = reinterpret_cast<uint16_t*>(&sh.lab[c][ry][0]) + (2 * quad - 1);
                if (quad > 0) dst[0] = (uint16_t)lab[c];
                if (quad < kQuadsY - 1) dst[1] = (uint16_t)(lab[c] >> 16);
            }
        }
    }
    // Region arrays: cell i of the gray region is image coordinate x0 - 4 + i, of the blurred and the colour
    // region x0 - 2 + i, of the gradient region x0 - 1 + i (rows alike).
    // stage 2: 5x5 binomial blur, (sum + 128) >> 8; along the rows (weights 1 4 6 4 as a byte dot product)
    for (int p = tid; p < kReg * kStripsB; p += NT) {
        const int ry = p / kStripsB, sx = p % kStripsB;
        const uint32_t w0 = sh.gray.y[ry][sx], w1 = sh.gray.y[ry][sx + 1];
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[i] = __builtin_amdgcn_udot4(i == 0 ? w0 : __builtin_amdgcn_alignbyte(w1, w0, i), 0x04060401u, (w1 >> (8 * i)) & 0xFFu, false);
        sh.gray.h[ry][sx] = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
    }
    __syncthreads();
    // ... and down the columns, two pixels per packed operation (sums stay below 2^16)
    for (int p = tid; p < kRegB * kStripsB; p += NT) {
        const int ry = p / kStripsB, sx = p % kStripsB;
        uint2 r[5];
#pragma unroll
        for (int a = 0; a < 5; ++a) r[a] = sh.gray.h[ry + a][sx];
        auto column = [&](uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e) {
            auto u = [](uint32_t v) { return __builtin_bit_cast(ushort2_t, v); };
            const ushort2_t four = {4, 4}, six = {6, 6}, half = {128, 128}, eight = {8, 8};
            const ushort2_t sum = (u(a) + u(e)) + four * (u(b) + u(d)) + six * u(c) + half;
            return __builtin_bit_cast(uint32_t, (ushort2_t)(sum >> eight));
        };
        const uint32_t lo = column(r[0].x, r[1].x, r[2].x, r[3].x, r[4].x), hi = column(r[0].y, r[1].y, r[2].y, r[3].y, r[4].y);
        sh.gray.b[ry][sx] = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
    }
    // stage 4a: colour variance, 25 * sum v^2 - (sum v)^2 over 5x5 per channel: sums over the five cells of a row
    // (the tables are done with: their memory holds these)
    for (int p = tid; p < kRegB * (kTile / 4); p += NT) {
        const int ry = p / (kTile / 4), sx = p % (kTile / 4);
        uint32_t sq[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint32_t* rowp = reinterpret_cast<const uint32_t*>(&sh.lab[c][ry][4 * sx]);
            const uint32_t w0 = rowp[0], w1 = rowp[1];
            uint32_t s1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t a4 = i == 0 ? w0 : __builtin_amdgcn_alignbyte(w1, w0, i);     // columns i .. i + 3
                const uint32_t b5 = (w1 >> (8 * i)) & 0xFFu;                                   // column i + 4
                s1[i] = __builtin_amdgcn_udot4(a4, 0x01010101u, b5, false);
                sq[i] = __builtin_amdgcn_udot4(a4, a4, sq[i], false) + b5 * b5;
            }
            sh.var.s[c][ry][sx] = make_uint2(s1[0] | (s1[1] << 16), s1[2] | (s1[3] << 16));
        }
        sh.var.sq[ry][sx] = make_uint4(sq[0], sq[1], sq[2], sq[3]);
    }
    __syncthreads();
    if (border) {
        // blurred cells outside the image: the value at the clamped coordinate
        for (int p = tid; p < kRegB * kRegB; p += NT) {
            const int ry = p / kRegB, rx = p % kRegB;
            const int cy = clampi(y0 - 2 + ry, 0, h - 1) - (y0 - 2), cx = clampi(x0 - 2 + rx, 0, w - 1) - (x0 - 2);
            if (cy != ry || cx != rx) sh.gray.b8[ry][rx] = sh.gray.b8[cy][cx];
        }
        __syncthreads();
    }

    // stage 3: Sobel gradients of the 34x34 region; cells outside the image hold 0 (that is what
    // non-maximum suppression wants to see there)
    for (int p = tid; p < kRegM * kStripsB; p += NT) {
        const int ry = p / kStripsB, sx = p % kStripsB;
        short2_t gx[2], gy[2];
        short2_t d[3][2], sm[3][2];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const uint32_t w0 = sh.gray.b[ry + a][sx], w1 = sx + 1 < kStripsB ? sh.gray.b[ry + a][sx + 1] : 0u;
            const short2_t two = {2, 2};
            const short2_t p01 = byte_pair(w0, w1, 0), p12 = byte_pair(w0, w1, 1), p23 = byte_pair(w0, w1, 2),
                           p34 = byte_pair(w0, w1, 3), p45 = byte_pair(w0, w1, 4);
            d[a][0] = p23 - p01;
            d[a][1] = p45 - p23;
            sm[a][0] = p01 + two * p12 + p23;
            sm[a][1] = p23 + two * p34 + p45;
        }
        uint32_t g[4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const short2_t two = {2, 2};
            gx[j] = d[0][j] + two * d[1][j] + d[2][j];
            gy[j] = sm[2][j] - sm[0][j];
            const uint32_t xb = __builtin_bit_cast(uint32_t, gx[j]), yb = __builtin_bit_cast(uint32_t, gy[j]);
            g[2 * j] = __builtin_amdgcn_perm(yb, xb, 0x05040100u);
            g[2 * j + 1] = __builtin_amdgcn_perm(yb, xb, 0x07060302u);
        }
        if (border) {
            const int my = y0 - 1 + ry, mx = x0 - 1 + 4 * sx;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (my < 0 || my >= h || mx + i < 0 || mx + i >= w) g[i] = 0u;
        }
        *reinterpret_cast<uint4*>(&sh.grad[ry][4 * sx]) = make_uint4(g[0], g[1], g[2], g[3]);
    }
    // stage 4b: the variance of four pixels from five rows of sums
    uint32_t local_sum = 0u;                                            // 30 431 700 a pixel at most: half a wave's stay below 2^32
    if (tid < kTile * kTile / 4) {
        const int vy = tid >> 3, sx = tid & 7;
        const int gy = y0 + vy, gx0 = x0 + 4 * sx;
        uint32_t sq[4] = {0u, 0u, 0u, 0u};
        uint32_t s1[3][2] = {{0u, 0u}, {0u, 0u}, {0u, 0u}};            // packed 16-bit sums, at most 25 * 255
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            const uint4 q = sh.var.sq[vy + a][sx];
            sq[0] += q.x;
            sq[1] += q.y;
            sq[2] += q.z;
            sq[3] += q.w;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const uint2 s = sh.var.s[c][vy + a][sx];
                s1[c][0] += s.x;
                s1[c][1] += s.y;
            }
        }
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t t = 25u * sq[i];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const uint32_t s = (s1[c][i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
                t -= __umul24(s, s);
            }
            v[i] = t;
        }
        if (gy < h) {
            uint32_t* dst = var_out + (__umul24((uint32_t)gy, (uint32_t)w) + (uint32_t)gx0);
            if (gx0 + 3 < w && (w & 3) == 0) {
                *reinterpret_cast<uint4*>(dst) = make_uint4(v[0], v[1], v[2], v[3]);
                local_sum += v[0] + v[1] + v[2] + v[3];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (gx0 + i < w) {
                        dst[i] = v[i];
                        local_sum += v[i];
                    }
            }
        }
    }
    for (int off = 16; off > 0; off >>= 1) local_sum += __shfl_down(local_sum, off);
    if ((tid & 31) == 0) sh.sum[tid >> 5] = local_sum;
    __syncthreads();
    // block sum of V -> one atomic
    if (tid == 0) {
        unsigned long long t = 0ull;
        for (int k = 0; k < NT / 32; ++k) t += sh.sum[k];
        atomicAdd(msum_acc, t);
    }

    // stage 5: non-maximum suppression + class.  kPrepPx pixels per thread (four of 256 threads, one of 1024): pixel
    // p = tid + NT q sits in tile row p / 32, so a wave always holds two complete tile rows.
    const int tx = tid % kTile;
    const int gx = x0 + tx;
    const uint32_t pixel0 = __umul24((uint32_t)(y0 + tid / kTile), (uint32_t)w) + (uint32_t)gx;      // its first pixel, in the image
    int cls[kPrepPx];
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) {
        const int ty = (tid + q * NT) / kTile;
        const int gy = y0 + ty;
        cls[q] = 0;
        if (gy < h && gx < w) {
            const uint32_t* at = &sh.grad[ty + 1][tx + 1];
            const uint32_t g = *at;
            const short2_t v = __builtin_bit_cast(short2_t, g);
            const int sgx = v.x, sgy = v.y, m2 = grad_m2(g);
            // the sector: (|gx| + |gy|)^2 against 2 gx^2 and 2 gy^2, both sides less |g|^2
            const int cross = 2 * __mul24(sgx, sgy), diff = m2 - 2 * __mul24(sgy, sgy), size = max(cross, -cross);
            int step;                         // first-listed neighbour; the second is its mirror
            if (size < diff) step = -1;
            else if (size < -diff) step = -kGradW;
            else if (cross > 0) step = -kGradW - 1;
            else step = -kGradW + 1;
            const int n1 = grad_m2(at[step]), n2 = grad_m2(at[-step]);
            if (m2 > n1 && m2 >= n2) cls[q] = m2 >= hi2 ? 2 : (m2 >= lo2 ? 1 : 0);
            cls_out[pixel0 + (uint32_t)(q * (NT / kTile)) * (uint32_t)w] = (uint8_t)cls[q];
        }
    }

    // hysteresis, tile-local part: union-find in LDS over horizontal runs.
    // A wave holds two tile rows (lanes 0-31 and 32-63), so the run a pixel lies in and the run's
    // smallest key (its leftmost strong pixel, else its leftmost pixel) follow from two ballots.
    uint32_t head_key[kPrepPx];
    bool left_is_cand[kPrepPx];
    if (tid == 0) sh.n_contacts = 0u;
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) {
        const int p = tid + q * NT;
        const int ty = p / kTile;
        const unsigned long long cand64 = __ballot(cls[q] != 0);
        const unsigned long long strong64 = __ballot(cls[q] == 2);
        const uint32_t row_c = (uint32_t)((tid & 32) ? (cand64 >> 32) : cand64);
        const uint32_t row_s = (uint32_t)((tid & 32) ? (strong64 >> 32) : strong64);
        head_key[q] = (uint32_t)p | (cls[q] == 1 ? kWeakBit : 0u);
        left_is_cand[q] = false;
        if (cls[q] != 0) {
            // candidates from this pixel to the left and to the right, itself among them; then the run's first strong pixel
            const uint32_t gaps_left = ~(row_c << (31 - tx)), gaps_right = ~(row_c >> tx);
            const int left = gaps_left == 0u ? 32 : __builtin_clz(gaps_left), right = gaps_right == 0u ? 32 : __builtin_ctz(gaps_right);
            const int start = tx + 1 - left;
            const uint32_t strong = row_s >> start;
            const int first = strong == 0u ? 32 : __builtin_ctz(strong);
            head_key[q] = (uint32_t)(ty * kTile + start) + (first < left + right - 1 ? (uint32_t)first : kWeakBit);
            left_is_cand[q] = left > 1;
        }
        s_lbl[p] = head_key[q];
        if (tx == 0) sh.row[ty] = row_c;
    }
    __syncthreads();
    // Contacts of runs of adjacent rows (S, SW, SE neighbours), each made once, by the leftmost pixel pair that
    // touches, and only where a run without a strong pixel takes part (strong runs need not be joined).
    // They are listed first and joined afterwards, a thread each: a pixel has at most two, but joining them where
    // they are found put divergent walks one after the other (5 to 7 us of a block's 16).
    {
        uint32_t other[kPrepPx][2];
        bool want[kPrepPx][2];
        unsigned long long m[kPrepPx][2];
        uint32_t total = 0u;
#pragma unroll
        for (int q = 0; q < kPrepPx; ++q) {
            const int ty = (tid + q * NT) / kTile;
            const bool inner = ty + 1 < kTile;
            const unsigned long long row_below = (unsigned long long)(inner ? sh.row[ty + 1] : 0u) << 1;
            const uint32_t near = cls[q] != 0 ? (uint32_t)(row_below >> tx) & 7u : 0u;      // SW, S, SE
            want[q][0] = (near & 3u) != 0u && !left_is_cand[q];
            want[q][1] = (near & 6u) == 4u;
            other[q][0] = s_lbl[inner ? (ty + 1) * kTile + max((near & 1u) ? tx - 1 : tx, 0) : 0];
            other[q][1] = s_lbl[inner ? (ty + 1) * kTile + min(tx + 1, kTile - 1) : 0];
        }
#pragma unroll
        for (int q = 0; q < kPrepPx; ++q)
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                want[q][side] = want[q][side] && ((head_key[q] | other[q][side]) & kWeakBit) != 0u;
                m[q][side] = __ballot(want[q][side]);
                total += (uint32_t)__popcll(m[q][side]);
            }
        uint32_t first = 0u;
        if ((tid & 63) == 0) first = atomicAdd(&sh.n_contacts, total);
        first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
#pragma unroll
        for (int q = 0; q < kPrepPx; ++q)
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                if (want[q][side]) {
                    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[q][side] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[q][side], first));
                    auto pack = [](uint32_t key) { return (key & 0x3FFu) | (key >> 21 & 0x400u); };
                    sh.contact[at] = pack(head_key[q]) | (pack(other[q][side]) << 16);
                }
                first += (uint32_t)__popcll(m[q][side]);
            }
    }
    __syncthreads();
    for (uint32_t i = tid; i < sh.n_contacts; i += NT) {
        const uint32_t c = sh.contact[i];
        auto unpack = [](uint32_t v) { return (v & 0x3FFu) | (v << 21 & kWeakBit); };
        uf_spread_strong<__HIP_MEMORY_SCOPE_WORKGROUP>(s_lbl, unpack(c & 0xFFFFu), unpack(c >> 16));
    }
    __syncthreads();
    // each pixel's global link: the global key of a strong pixel of its component or, without one, of the
    // component's smallest key in this tile (itself for pixels that are no edge candidates).  Tile-local
    // row-major order agrees with image row-major order, so "smallest" means the same in both.  The
    // walks of a thread's pixels go in step, and every pixel's link follows its walk: all walks of the tile move at
    // once, so what a walk meets has been shortened as often as itself (no root changes any more).
    uint32_t root[kPrepPx];
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) root[q] = cls[q] != 0 ? head_key[q] : (uint32_t)(tid + q * NT);
    for (;;) {
        uint32_t up[kPrepPx];
        bool moved = false;
#pragma unroll
        for (int q = 0; q < kPrepPx; ++q) up[q] = uf_load<__HIP_MEMORY_SCOPE_WORKGROUP>(s_lbl, root[q] & ~kWeakBit);
#pragma unroll
        for (int q = 0; q < kPrepPx; ++q) {
            if ((root[q] & kWeakBit) == 0u || up[q] == root[q]) continue;
            moved = true;
            root[q] = up[q];
            __hip_atomic_store(&s_lbl[tid + q * NT], up[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (!moved) break;
    }
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) {
        const int ty = (tid + q * NT) / kTile;
        if (y0 + ty >= h || gx >= w) continue;
        const uint32_t rl = root[q] & ~kWeakBit;
        const uint32_t rg = __umul24((uint32_t)y0 + rl / kTile, (uint32_t)w) + (uint32_t)x0 + rl % kTile;
        parent_out[pixel0 + (uint32_t)(q * (NT / kTile)) * (uint32_t)w] = rg | (root[q] & kWeakBit);
    }
}

// Hysteresis across tiles, item = border pixel of frame b; stop() as in patch_sum
template <typename Stop>
__device__ __forceinline__ void union_item(const PrepFrame& frame, int h, int w, int item, int n_items, Stop stop) {
    union_border(frame.cls, frame.parent, h, w, min(item, n_items - 1), item < n_items, stop);
}

// Eq. 7 for the pixels of one patch that fall to a lane, pixels p0, p0 + kStride, ...: sum of E + C
struct PatchBox {
    int ya, xa, pw, area;
};
__device__ __forceinline__ PatchBox patch_box(int token, int h, int w) {
    const int pr = token / kGrid, pc = token % kGrid;
    const int ya = (pr * h) / kGrid, yb = ((pr + 1) * h) / kGrid;
    const int xa = (pc * w) / kGrid, xb = ((pc + 1) * w) / kGrid;
    return {ya, xa, xb - xa, (xb - xa) * (yb - ya)};
}
// Pixel number of a patch -> its place in the image
struct PatchPixels {
    uint32_t first, w;
    PatchRow row_of;
    __device__ __forceinline__ PatchPixels(const PatchBox& box, int width)
        : first((uint32_t)box.ya * (uint32_t)width + (uint32_t)box.xa), w((uint32_t)width), row_of((uint32_t)box.pw, (uint32_t)box.area) {}
    __device__ __forceinline__ uint32_t operator()(int pixel) const {
        const uint32_t p = (uint32_t)pixel, row = row_of(p);
        return first + row * w + (p - row * row_of.width);
    }
};
// The pixels of a pass are asked for together, and the walks of weak ones move in step: a walk's step is a trip to memory, and one
// pixel's walk after the other was most of the time of small frames (one 640x360 frame 12.4 -> 7.2 us, four 1920x1080 26.2 -> 19.4).
// kStride = 64 (small frames): eight pixels a pass, with their first links (four bytes a pixel more, a trip less).
// stop(): asked once the first loads are under way; true (uniform): the frame gets no scores, nothing is done and kNoSum returned.
constexpr uint32_t kNoSum = 0xFFFFFFFFu;
template <int kStride, typename Stop>
__device__ __forceinline__ uint32_t patch_sum(const PoolFrame& frame, const PatchBox& box, int p_first, int h, int w,
                                              uint8_t* __restrict__ salmap, Stop stop) {
    const uint8_t* __restrict__ cls = frame.cls;
    const uint32_t* __restrict__ parent = frame.parent;
    const uint32_t* __restrict__ var = frame.var;
    together(cls, parent, var, frame.msum, frame.scores, salmap);
    constexpr bool kLinks = kStride == 64;
    constexpr int kUnroll = kLinks ? 8 : 4;
    const PatchPixels pixel(box, w);
    uint32_t q = 0;
    for (int p0 = p_first; p0 < box.area || p0 == p_first; p0 += kStride * kUnroll) {
        uint32_t gi[kUnroll], c[kUnroll], v[kUnroll], key[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            gi[u] = pixel(min(p0 + u * kStride, box.area - 1));
            c[u] = ld_at(cls, gi[u]);
            v[u] = ld_at(var, gi[u]);
            if constexpr (kLinks) key[u] = ld_at(parent, gi[u]);
        }
        if (p0 == p_first && stop()) return kNoSum;
        const unsigned long long m = *frame.msum;
        const unsigned long long hw = (unsigned long long)h * (unsigned long long)w;
        bool more = false;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (p0 + u * kStride >= box.area) c[u] = 0u;
            // a weak pixel's key: itself, or its first link where that is known (itself: a root, no strong pixel)
            const uint32_t self = gi[u] | kWeakBit;
            if constexpr (kLinks) {
                if (c[u] == 1u && key[u] == self) c[u] = 0u;
            } else {
                key[u] = self;
            }
            if (c[u] != 1u) key[u] = 0u;
            more = more || (key[u] & kWeakBit) != 0u;
        }
        while (more) {
            uint32_t up[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) up[u] = ld_at(parent, key[u] & ~kWeakBit);
            more = false;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if ((key[u] & kWeakBit) == 0u) continue;
                if (up[u] == key[u]) c[u] = 0u;                 // a root without a strong pixel
                key[u] = up[u] == key[u] ? 0u : up[u];
                more = more || (key[u] & kWeakBit) != 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (p0 + u * kStride >= box.area) continue;
            const uint32_t e = c[u] != 0u ? 1u : 0u, cm = ((unsigned long long)v[u] * hw > m && v[u] >= kVMin) ? 1u : 0u;
            q += e + cm;
            if (salmap != nullptr) salmap[gi[u]] = (uint8_t)(e + cm);
        }
    }
    return q;
}
// floor(q 2^15 / |P|) / 2^16 of the patch, by one lane
__device__ __forceinline__ void store_score(const PoolFrame& frame, int token, uint32_t q, int area) {
    const uint32_t s_fix = (uint32_t)(((unsigned long long)q << 15) / (unsigned long long)area);
    const float score = (float)s_fix * (1.0f / 65536.0f);      // exact: s_fix <= 2^16
    __hip_atomic_store(frame.scores + token, score, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// one patch by one wave
template <typename Stop>
__device__ __forceinline__ void score_by_wave(const PoolFrame& frame, int token, int h, int w, uint8_t* __restrict__ salmap, Stop stop) {
    const int lane = threadIdx.x & 63;
    const PatchBox box = patch_box(token, h, w);
    uint32_t q = patch_sum<64>(frame, box, lane, h, w, salmap, stop);
    if (q == kNoSum) return;
    for (int off = 32; off > 0; off >>= 1) q += __shfl_down(q, off);
    if (lane == 0) store_score(frame, token, q, box.area);
}

}  // namespace sali
