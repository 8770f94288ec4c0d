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
#include "hysteresis.h"
#include "tier_body.h"

namespace sali {

namespace {

constexpr int kHalo = 4;
constexpr int kReg = kTile + 2 * kHalo;        // 40: gray region
constexpr int kRegB = kTile + 4;               // 36: blur / LAB region (halo 2)
constexpr int kRegM = kTile + 2;               // 34: gradient-magnitude region (halo 1)

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }


}  // namespace

// gray only, blockIdx.y = frame of the batch: what the flow needs of a frame.  The rest of the spatial
// filter waits until the reuse rule has spoken.  Sixteen pixels per thread (48 bytes in, 16 out) where
// the caller's image is 16-byte aligned, else pixel by pixel.
__global__ __launch_bounds__(256) void k_gray(PrepBatch f, int n) {
    const uint8_t* __restrict__ rgb = f.rgb[blockIdx.y];
    uint8_t* __restrict__ y8 = f.y8[blockIdx.y];
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

// #{dP_i < tau_t} over the thread's share of one image's 576 patch motions (block of 256 threads); the
// loads are independent and issued together
__device__ __forceinline__ int count_static(const float* dp, float tau_t) {
    float v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int i = (int)threadIdx.x + 256 * k;
        v[k] = i < kTokens ? __hip_atomic_load(dp + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tau_t;
    }
    return (v[0] < tau_t ? 1 : 0) + (v[1] < tau_t ? 1 : 0) + (v[2] < tau_t ? 1 : 0);
}

// Eq. 6 and the reuse rule for frame b of a launch, evaluated by a whole block of 256 threads from the
// per-patch motions that an earlier kernel left (dp[b] NULL: no predecessor, never redundant): the
// kernels of the spatial filter ask this first and leave at once for a redundant frame (Algorithm 1
// skips its saliency).  Same counts and the same fp32 quotient as the tail kernel that writes the gate,
// so all of them take the same decision.  s_cnt: four ints of LDS.
__device__ __forceinline__ bool frame_redundant(const float* const* dp, int b, const GateParams& gp, int* s_cnt) {
    const int b0 = b - b % gp.tiles;
    if (dp[b0] == nullptr) return false;
    int n = 0;
    for (int j = 0; j < gp.tiles; ++j) n += count_static(dp[b0 + j], gp.tau_t);
    for (int off = 32; off > 0; off >>= 1) n += __shfl_down(n, off);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = n;
    __syncthreads();
    const int n_static = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    __syncthreads();
    return (float)n_static / (float)(kTokens * gp.tiles) > gp.theta_r;
}

// 256 threads per 32x32 tile.  Workgroups are kept this small so that they find room on compute units that a
// bandwidth kernel of another stream keeps busy.
//
// Four 1920x1080 frames: 107 us, one 640x360 frame: 16; bound by the trips of a block's stages (image and tables
// from memory, then LDS; 20 waves per compute unit), the vector ALU 61 % busy.  Taken tap by tap, byte
// by byte, with clamped coordinates, the stencils were 612 instructions per pixel instead of 305, the ALU
// 90 % busy, and the kernel took 150 and 24 us.  So each
// stage takes strips of four pixels as words: byte dot products along rows, packed 16-bit arithmetic down
// columns, separable sums kept in LDS where neighbouring rows share them, gradients as 16-bit pairs whose
// squared magnitude is one dot product.  No stage clamps coordinates: a cell outside the image holds what the
// definition wants to see there (gray and colour of the clamped coordinate as loaded; blurred values copied
// from the clamped cell, gradient 0), which only blocks on the image border have to arrange.
constexpr int kPrepThreads = 256;
constexpr int kPrepPx = kTile * kTile / kPrepThreads;                          // 4
constexpr int kQuadsY = kReg / 4;                                              // 10 quads of a gray row
constexpr int kPrepQuads = (kReg * kQuadsY + kPrepThreads - 1) / kPrepThreads; // 2 per thread
constexpr int kStripsB = kRegB / 4;                                            // 9 strips of a blurred row
constexpr int kGradW = 36;                                                     // gradient row: 34 cells, whole strips
constexpr int kLutWords = kColourLutBytes / 4;
constexpr int kLutQuads = (kLutWords / 4 + kPrepThreads - 1) / kPrepThreads;
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
    // gray image and its row sums; from the hysteresis on the tile's union-find links (key = local index | weak bit)
    union {
        struct {
            uint32_t y[kReg][kQuadsY];
            uint2 h[kReg][kStripsB];
        } gray;
        uint32_t lbl[kTile * kTile];
    };
    // blurred image
    union {
        uint32_t b[kRegB][kStripsB];
        uint8_t b8[kRegB][kRegB];
    };
    __attribute__((aligned(16))) uint32_t grad[kRegM][kGradW];      // (gx, gy) as 16-bit halves
    __attribute__((aligned(16))) uint8_t lab[3][kRegB][kRegB];
    unsigned long long sum[kPrepThreads / 64];
    int gate[4];
    uint32_t row[kTile];        // a tile row's edge candidates, a bit each
    uint32_t n_contacts;
};

// bytes i and i + 1 of the eight in (lo, hi) as 16-bit halves
__device__ __forceinline__ short2_t byte_pair(uint32_t lo, uint32_t hi, int i) {
    const uint32_t sel = 0x0c000c00u | (uint32_t)i | ((uint32_t)(i + 1) << 16);
    return __builtin_bit_cast(short2_t, __builtin_amdgcn_perm(hi, lo, sel));
}
__device__ __forceinline__ int grad_m2(uint32_t g) {
    const short2_t v = __builtin_bit_cast(short2_t, g);
    return __builtin_amdgcn_sdot2(v, v, 0, false);
}

__global__ __launch_bounds__(kPrepThreads) void k_prep(PrepBatch f, int h, int w, GateParams gp,
                                                       const uint32_t* __restrict__ lut_words, int lo2, int hi2) {
    // blockIdx.z = frame of the batch
    const uint8_t* __restrict__ rgb = f.rgb[blockIdx.z];
    uint8_t* __restrict__ cls_out = f.cls[blockIdx.z];
    uint32_t* __restrict__ var_out = f.var[blockIdx.z];
    uint32_t* __restrict__ parent_out = f.parent[blockIdx.z];
    unsigned long long* msum_acc = f.msum_acc[blockIdx.z];
    unsigned long long* msum_clear = f.msum_clear[blockIdx.z];
    __shared__ PrepShared sh;
    uint32_t (&s_lbl)[kTile * kTile] = sh.lbl;

    const int tid = threadIdx.x;
    const int x0 = blockIdx.x * kTile, y0 = blockIdx.y * kTile;
    const bool border = x0 == 0 || y0 == 0 || x0 + kTile + kHalo > w || y0 + kTile + kHalo > h;      // uniform

    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0 && msum_clear != nullptr) *msum_clear = 0ull;

    // stage 1a: RGB of the 40x40 region, four pixels (twelve bytes at any address) at a time, coordinates clamped.
    // These loads and those of the colour tables are issued before the reuse rule is looked at, so that its
    // memory round trip and theirs overlap: most frames are not redundant.
    uint32_t crgb[kPrepQuads][3];
#pragma unroll
    for (int k = 0; k < kPrepQuads; ++k) {
        const int p = min(tid + k * kPrepThreads, kReg * kQuadsY - 1);
        const int x = x0 - kHalo + 4 * (p % kQuadsY);
        const uint8_t* row = rgb + (size_t)clampi(y0 - kHalo + p / kQuadsY, 0, h - 1) * w * 3;
        if (x >= 0 && x + 3 < w) {
            __builtin_memcpy(crgb[k], row + 3 * x, 12);
        } else {
            uint32_t c[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) c[i] = row[3 * clampi(x + i / 3, 0, w - 1) + i % 3];
#pragma unroll
            for (int i = 0; i < 3; ++i) crgb[k][i] = c[4 * i] | (c[4 * i + 1] << 8) | (c[4 * i + 2] << 16) | (c[4 * i + 3] << 24);
        }
    }
    u32x4 lut[kLutQuads];
#pragma unroll
    for (int k = 0; k < kLutQuads; ++k)
        lut[k] = reinterpret_cast<const u32x4*>(lut_words)[min(tid + k * kPrepThreads, kLutWords / 4 - 1)];
    {
        // no saliency for a redundant frame; the frame's first block leaves the decision for the kernels
        // after this one, whose blocks are too small to count 576 patches each
        const bool skip = frame_redundant(f.dp, blockIdx.z, gp, sh.gate);
        if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *f.skip[blockIdx.z] = skip ? 1u : 0u;
        if (skip) return;
    }
    // colour tables -> LDS, gray of the region
#pragma unroll
    for (int k = 0; k < kLutQuads; ++k) {
        const int i = tid + k * kPrepThreads;
        if (i < kLutWords / 4) reinterpret_cast<u32x4*>(sh.lut)[i] = lut[k];
    }
#pragma unroll
    for (int k = 0; k < kPrepQuads; ++k) {
        const int p = tid + k * kPrepThreads;
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
            const int p = tid + k * kPrepThreads;
            const int ry = p / kQuadsY - 2, quad = p % kQuadsY;          // row of the region, cells 4 quad - 2 ..
            if (ry < 0 || ry >= kRegB) continue;
            uint32_t lab[3] = {0u, 0u, 0u};                              // four pixels, a byte each
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                auto byte = [&](int j) { return (crgb[k][j >> 2] >> (8 * (j & 3))) & 0xFFu; };
                const int lr = s_lin[byte(3 * i)], lg = s_lin[byte(3 * i + 1)], lb = s_lin[byte(3 * i + 2)];
                const int tx = (1777 * lr + 1541 * lg + 778 * lb + 2048) >> 12;
                const int ty = (871 * lr + 2929 * lg + 296 * lb + 2048) >> 12;
                const int tz = (73 * lr + 448 * lg + 3575 * lb + 2048) >> 12;
                const int fx = s_fl[tx], fy = s_fl[ty], fz = s_fl[tz];
                lab[0] |= (uint32_t)s_l8[ty] << (8 * i);
                lab[1] |= (uint32_t)clampi((500 * (fx - fy) + 4194304 + 16384) >> 15, 0, 255) << (8 * i);
                lab[2] |= (uint32_t)clampi((200 * (fy - fz) + 4194304 + 16384) >> 15, 0, 255) << (8 * i);
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
    for (int p = tid; p < kReg * kStripsB; p += kPrepThreads) {
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
    for (int p = tid; p < kRegB * kStripsB; p += kPrepThreads) {
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
        sh.b[ry][sx] = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
    }
    // stage 4a: colour variance, 25 * sum v^2 - (sum v)^2 over 5x5 per channel: sums over the five cells of a row
    // (the tables are done with: their memory holds these)
    for (int p = tid; p < kRegB * (kTile / 4); p += kPrepThreads) {
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
        for (int p = tid; p < kRegB * kRegB; p += kPrepThreads) {
            const int ry = p / kRegB, rx = p % kRegB;
            const int cy = clampi(y0 - 2 + ry, 0, h - 1) - (y0 - 2), cx = clampi(x0 - 2 + rx, 0, w - 1) - (x0 - 2);
            if (cy != ry || cx != rx) sh.b8[ry][rx] = sh.b8[cy][cx];
        }
        __syncthreads();
    }

    // stage 3: Sobel gradients of the 34x34 region; cells outside the image hold 0 (that is what
    // non-maximum suppression wants to see there)
    for (int p = tid; p < kRegM * kStripsB; p += kPrepThreads) {
        const int ry = p / kStripsB, sx = p % kStripsB;
        short2_t gx[2], gy[2];
        short2_t d[3][2], sm[3][2];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const uint32_t w0 = sh.b[ry + a][sx], w1 = sx + 1 < kStripsB ? sh.b[ry + a][sx + 1] : 0u;
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
    unsigned long long local_sum = 0ull;
    {
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
            uint32_t* dst = var_out + (size_t)gy * w + gx0;
            if (gx0 + 3 < w && (w & 3) == 0) {
                *reinterpret_cast<uint4*>(dst) = make_uint4(v[0], v[1], v[2], v[3]);
                local_sum += (unsigned long long)v[0] + v[1] + v[2] + v[3];
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
    for (int off = 32; off > 0; off >>= 1) local_sum += __shfl_down(local_sum, off);
    if ((tid & 63) == 0) sh.sum[tid >> 6] = local_sum;
    __syncthreads();
    // block sum of V -> one atomic
    if (tid == 0) {
        unsigned long long t = 0ull;
        for (int k = 0; k < kPrepThreads / 64; ++k) t += sh.sum[k];
        atomicAdd(msum_acc, t);
    }

    // stage 5: non-maximum suppression + class.  Four pixels per thread: pixel p = tid + 256 q sits in tile row
    // p / 32, so a wave always holds two complete tile rows.
    const int tx = tid % kTile;
    const int gx = x0 + tx;
    int cls[kPrepPx];
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) {
        const int ty = (tid + q * kPrepThreads) / kTile;
        const int gy = y0 + ty;
        cls[q] = 0;
        if (gy < h && gx < w) {
            const uint32_t* at = &sh.grad[ty + 1][tx + 1];
            const short2_t v = __builtin_bit_cast(short2_t, *at);
            const int sgx = v.x, sgy = v.y;
            const int xx = __mul24(sgx, sgx), yy = __mul24(sgy, sgy), m2 = xx + yy;
            const int ax = abs(sgx), ay = abs(sgy);
            const int s2 = __mul24(ax + ay, ax + ay);
            int step;                         // first-listed neighbour; the second is its mirror
            if (s2 < 2 * xx) step = -1;
            else if (s2 < 2 * yy) step = -kGradW;
            else if (__mul24(sgx, sgy) > 0) step = -kGradW - 1;
            else step = -kGradW + 1;
            const int n1 = grad_m2(at[step]), n2 = grad_m2(at[-step]);
            if (m2 > n1 && m2 >= n2) cls[q] = m2 >= hi2 ? 2 : (m2 >= lo2 ? 1 : 0);
            cls_out[(size_t)gy * w + gx] = (uint8_t)cls[q];
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
        const int p = tid + q * kPrepThreads;
        const int ty = p / kTile;
        const unsigned long long cand64 = __ballot(cls[q] != 0);
        const unsigned long long strong64 = __ballot(cls[q] == 2);
        const uint32_t row_c = (uint32_t)((tid & 32) ? (cand64 >> 32) : cand64);
        const uint32_t row_s = (uint32_t)((tid & 32) ? (strong64 >> 32) : strong64);
        head_key[q] = (uint32_t)p | (cls[q] == 1 ? kWeakBit : 0u);
        left_is_cand[q] = false;
        if (cls[q] != 0) {
            const uint32_t zeros = ~row_c;
            const uint32_t below = zeros & ((1u << tx) - 1u);
            const uint32_t above = (tx == 31) ? 0u : (zeros & ~((2u << tx) - 1u));
            const int start = below == 0u ? 0 : 32 - __builtin_clz(below);
            const int end = above == 0u ? 31 : __builtin_ctz(above) - 1;
            const uint32_t run = (end == 31 ? 0xFFFFFFFFu : ((2u << end) - 1u)) & ~((1u << start) - 1u);
            const uint32_t strong_in_run = row_s & run;
            head_key[q] = strong_in_run != 0u ? (uint32_t)(ty * kTile + __builtin_ctz(strong_in_run))
                                              : ((uint32_t)(ty * kTile + start) | kWeakBit);
            left_is_cand[q] = tx > 0 && ((row_c >> (tx - 1)) & 1u) != 0u;
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
            const int ty = (tid + q * kPrepThreads) / kTile;
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
                    const uint32_t at = first + (uint32_t)__popcll(m[q][side] & ~(~0ull << (tid & 63)));
                    auto pack = [](uint32_t key) { return (key & 0x3FFu) | (key >> 21 & 0x400u); };
                    sh.contact[at] = pack(head_key[q]) | (pack(other[q][side]) << 16);
                }
                first += (uint32_t)__popcll(m[q][side]);
            }
    }
    __syncthreads();
    for (uint32_t i = tid; i < sh.n_contacts; i += kPrepThreads) {
        const uint32_t c = sh.contact[i];
        auto unpack = [](uint32_t v) { return (v & 0x3FFu) | (v << 21 & kWeakBit); };
        uf_spread_strong<__HIP_MEMORY_SCOPE_WORKGROUP>(s_lbl, unpack(c & 0xFFFFu), unpack(c >> 16));
    }
    __syncthreads();
    // each pixel's global link: the global key of a strong pixel of its component or, without one, of the
    // component's smallest key in this tile (itself for pixels that are no edge candidates).  Tile-local
    // row-major order agrees with image row-major order, so "smallest" means the same in both.  The four
    // walks of a thread go in step, and every pixel's link follows its walk: all walks of the tile move at
    // once, so what a walk meets has been shortened as often as itself (no root changes any more).
    uint32_t root[kPrepPx];
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) root[q] = cls[q] != 0 ? head_key[q] : (uint32_t)(tid + q * kPrepThreads);
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
            __hip_atomic_store(&s_lbl[tid + q * kPrepThreads], up[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (!moved) break;
    }
#pragma unroll
    for (int q = 0; q < kPrepPx; ++q) {
        const int ty = (tid + q * kPrepThreads) / kTile;
        if (y0 + ty >= h || gx >= w) continue;
        const uint32_t rl = root[q] & ~kWeakBit;
        const size_t rg = (size_t)(y0 + (int)(rl / kTile)) * w + (x0 + (int)(rl % kTile));
        parent_out[(size_t)(y0 + ty) * w + gx] = (uint32_t)rg | (root[q] & kWeakBit);
    }
}

// hysteresis, cross-tile part; blockIdx.y = frame of the batch.  A thread per border pixel: with a thread per
// image pixel, nearly all of them idle, and walks to the root also between strong components sixteen 640x360
// frames took 44 us in the pipeline, one frame alone 16.8; now 23.5 and 9.6 (chains of trips past the L2).
__global__ __launch_bounds__(256) void k_union(PrepBatch f, int h, int w, int n_items) {
    if (*f.skip[blockIdx.y] != 0u) return;          // redundant frame, says the pre-pass
    const int item = blockIdx.x * 256 + threadIdx.x;
    if (item < n_items) union_border(f.cls[blockIdx.y], f.parent[blockIdx.y], h, w, item);
}

// Gate (Eq. 6), tier assignment and compaction indices of frame `b` of a launch of `n_frames`, by
// one block of 256 threads, after every patch score and patch motion of the frame has been written:
// n_static = #{dP_i < tau_t}, R = n_static / 576, redundant iff R > theta_R; a frame without
// predecessor (no flow) is never redundant.  The last such block of the launch (arrival counter,
// nobody waits) writes the frame-table rows and advances the pool cursors in video order.
__device__ __forceinline__ void pool_tail(TierShared& sh, int* s_cnt, const PoolBatch& f, int b, int n_frames,
                                          float tau_t, float theta_r, const TierLaunch& tl, uint32_t* batch_done) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // gate: n_static = #{dP_i < tau_t}, R = n_static / 576, redundant iff R > theta_R; a frame
    // without predecessor (no flow) is never redundant
    const bool have_flow = f.flow[b] != nullptr;
    // the scores are asked for now, with the patch motions: one memory round trip instead of two on the
    // critical path of the batch (a redundant frame does not use them)
    const TierScores scores = tier_load_scores(f.scores[b]);
    // a tiled frame's patches are those of all its tiles (entries b0 .. b0 + tiles - 1 of the launch): the
    // block of every tile counts them all and so reaches the frame's one decision on its own
    const int tiles = tl.tiles;
    const int b0 = b - b % tiles;
    int n = 0;
    if (have_flow)
        for (int j = 0; j < tiles; ++j) n += count_static(f.dp[b0 + j], tau_t);
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
        *f.gate[b] = gt;
        int32_t* out = reinterpret_cast<int32_t*>(f.tcounts[b]);
        __hip_atomic_store(out + 0, tc.state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            __hip_atomic_store(out + 1 + t, tc.cnt[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < 3; ++j)
            __hip_atomic_store(out + 5 + j, tc.q[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();                // counts, tiers, slots and order lists before the arrival
        const bool last = atomicAdd(batch_done, 1u) == (uint32_t)n_frames - 1u;
        if (last) {
            __threadfence();
            *batch_done = 0u;
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
        if ((int)threadIdx.x < n_frames) {
            const int32_t* in = reinterpret_cast<const int32_t*>(f.tcounts[threadIdx.x]);
            TierCounts rec = {};
            rec.state = __hip_atomic_load(in + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int t = 0; t < 4; ++t) rec.cnt[t] = __hip_atomic_load(in + 1 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            all[threadIdx.x] = rec;
        }
        CursorRegs cr = {};
        if (threadIdx.x == 0) cr = cursor_load(tl.cur);
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
    CursorRegs cr = {};
    if (threadIdx.x == 0) cr = cursor_load(tl.cur);
    if (threadIdx.x < 3) sh.tau[threadIdx.x] = tl.cur->adapt_tau[threadIdx.x];
    __syncthreads();
    for (int i = 0; i < n_frames; ++i) {
        // the frame's hand-over record, the same words for every thread
        const int32_t* in = reinterpret_cast<const int32_t*>(f.tcounts[i]);
        TierCounts tci = {};
        tci.state = __hip_atomic_load(in + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int q[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) q[j] = __hip_atomic_load(in + 5 + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool ranked = tci.state == 3;
        if (ranked)
            tci = tier_assign_adaptive(sh, tier_load_scores(f.scores[i]), tl.tier + (size_t)i * kTokens,
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
template <int kWaves, bool kMotion>
__global__ __launch_bounds__(kTierThreads) void k_pool(PoolBatch f, int h, int w, uint8_t* __restrict__ salmap) {
    static_assert(kTierThreads == 256, "four waves, one patch each");
    static_assert(kWaves == 1 || kWaves == 4, "");
    __shared__ uint32_t s_pq[kTierThreads / 64];
    __shared__ float s_pm[kTierThreads / 64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (!kMotion && *f.skip[blockIdx.y] != 0u) return;      // redundant frame, says the pre-pass
    {
        // blockIdx.y = frame of the batch
        const uint8_t* __restrict__ cls = f.cls[blockIdx.y];
        const uint32_t* __restrict__ parent = f.parent[blockIdx.y];
        const uint32_t* __restrict__ var = f.var[blockIdx.y];
        const float2* __restrict__ flow = f.flow[blockIdx.y];
        const int token = kWaves == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
        const int pr = token / kGrid, pc = token % kGrid;
        const int ya = (pr * h) / kGrid, yb = ((pr + 1) * h) / kGrid;
        const int xa = (pc * w) / kGrid, xb = ((pc + 1) * w) / kGrid;
        const int pw = xb - xa, area = pw * (yb - ya);
        if (kMotion && flow == nullptr) {           // no predecessor: no motion
            if (lane == 0 && (kWaves == 1 || wave == 0))
                __hip_atomic_store(f.dp_out[blockIdx.y] + token, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        unsigned long long m = 0ull;
        if (!kMotion) m = *f.msum[blockIdx.y];
        const unsigned long long hw = (unsigned long long)h * (unsigned long long)w;
        uint32_t q = 0;
        float mag = 0.0f;
        // four pixels per pass, all their loads issued before any is used (the loop is bound by
        // memory latency, not by work)
        constexpr int kStride = 64 * kWaves, kUnroll = 4;
        for (int p0 = (kWaves == 1 ? lane : (int)threadIdx.x); p0 < area; p0 += kStride * kUnroll) {
            size_t gi[kUnroll];
            int c[kUnroll];
            uint32_t v[kUnroll];
            float2 d[kUnroll];
            bool ok[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int p = p0 + u * kStride;
                ok[u] = p < area;
                const int pp = ok[u] ? p : 0;
                gi[u] = (size_t)(ya + pp / pw) * w + (xa + pp % pw);
                if (kMotion) {
                    d[u] = flow[gi[u]];
                } else {
                    c[u] = cls[gi[u]];
                    v[u] = var[gi[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (!ok[u]) continue;
                if (kMotion) {
                    mag += d[u].x * d[u].x + d[u].y * d[u].y;
                } else {
                    uint32_t e = 0;
                    if (c[u] == 2) e = 1;
                    else if (c[u] == 1) e = uf_stays_weak(parent, (uint32_t)gi[u] | kWeakBit) ? 0u : 1u;
                    const uint32_t cm = ((unsigned long long)v[u] * hw > m && v[u] >= kVMin) ? 1u : 0u;
                    q += e + cm;
                    if (salmap != nullptr) salmap[gi[u]] = (uint8_t)(e + cm);
                }
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            if (kMotion) mag += __shfl_down(mag, off);
            else q += __shfl_down(q, off);
        }
        if (kWaves == 4) {
            if (lane == 0) {
                s_pq[wave] = q;
                s_pm[wave] = mag;
            }
            __syncthreads();
            q = s_pq[0] + s_pq[1] + s_pq[2] + s_pq[3];
            mag = (s_pm[0] + s_pm[1]) + (s_pm[2] + s_pm[3]);
        }
        if (lane == 0 && (kWaves == 1 || wave == 0)) {
            if (kMotion) {
                __hip_atomic_store(f.dp_out[blockIdx.y] + token, sqrtf(mag / (float)area), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const uint32_t s_fix = (uint32_t)(((unsigned long long)q << 15) / (unsigned long long)area);
                const float score = (float)s_fix * (1.0f / 65536.0f);      // exact: s_fix <= 2^16
                __hip_atomic_store(f.scores[blockIdx.y] + token, score, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// the tail as a launch of its own: one block per frame
__global__ __launch_bounds__(kTierThreads) void k_pool_tail(PoolBatch f, float tau_t, float theta_r, TierLaunch tl,
                                                            uint32_t* batch_done) {
    __shared__ TierShared sh;
    __shared__ int s_cnt[kTierThreads / 64];
    pool_tail(sh, s_cnt, f, (int)blockIdx.x, (int)gridDim.x, tau_t, theta_r, tl, batch_done);
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_gray(const PrepBatch& f, int n, int h, int w, hipStream_t s) {
    const int px = h * w;
    hipLaunchKernelGGL(k_gray, dim3((px + 4095) / 4096, n), dim3(256), 0, s, f, px);
    return hipGetLastError();
}

hipError_t launch_prep(const PrepBatch& f, int n, int h, int w, GateParams gp, const void* d_lut,
                       int lo2, int hi2, hipStream_t s) {
    dim3 grid((w + kTile - 1) / kTile, (h + kTile - 1) / kTile, n);
    hipLaunchKernelGGL(k_prep, grid, dim3(kPrepThreads), 0, s, f, h, w, gp,
                       static_cast<const uint32_t*>(d_lut), lo2, hi2);
    return hipGetLastError();
}

hipError_t launch_union(const PrepBatch& f, int n, int h, int w, hipStream_t s) {
    const int items = border_items(h, w);
    if (items == 0) return hipSuccess;              // a single tile
    hipLaunchKernelGGL(k_union, dim3((items + 255) / 256, n), dim3(256), 0, s, f, h, w, items);
    return hipGetLastError();
}

hipError_t launch_motion(const PoolBatch& f, int n, int h, int w, hipStream_t s) {
    // patches of up to 1024 pixels: one wave each
    if ((long long)h * w <= 1024ll * kTokens) {
        hipLaunchKernelGGL((k_pool<1, true>), dim3(kTokens / 4, n), dim3(kTierThreads), 0, s, f, h, w, nullptr);
    } else {
        hipLaunchKernelGGL((k_pool<4, true>), dim3(kTokens, n), dim3(kTierThreads), 0, s, f, h, w, nullptr);
    }
    return hipGetLastError();
}

hipError_t launch_pool(const PoolBatch& f, int n, int h, int w, uint8_t* d_salmap_or_null,
                       const TierLaunch* tier_or_null, GateParams gp, uint32_t* d_done_counter, hipEvent_t done_or_null, hipStream_t s) {
    TierLaunch t = {};
    if (tier_or_null != nullptr) t = *tier_or_null;
    if ((long long)h * w <= 1024ll * kTokens) {
        hipLaunchKernelGGL((k_pool<1, false>), dim3(kTokens / 4, n), dim3(kTierThreads), 0, s, f, h, w, d_salmap_or_null);
    } else {
        hipLaunchKernelGGL((k_pool<4, false>), dim3(kTokens, n), dim3(kTierThreads), 0, s, f, h, w, d_salmap_or_null);
    }
    if (tier_or_null != nullptr) {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        launch_recording(done_or_null, k_pool_tail, dim3(n), dim3(kTierThreads), s, f, gp.tau_t, gp.theta_r, t, d_done_counter);
    }
    return hipGetLastError();
}

}  // namespace sali
