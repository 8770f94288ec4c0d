// Dense polynomial-expansion optical flow, per-patch motion and the redundancy gate for gfx950.
//
// Temporal Filtering via Optical Flow (Eq. 5, Eq. 6, reuse rule R_frame > theta_R) and
// Implementation Details (Farneback's algorithm, pyramid scale 0.5).  fp32 throughout, on small
// images; the design goal is few launches and no spilled intermediates.
//
//   k_expand     pyramid (5x5 binomial [1 4 6 4 1]/16, stride 2; level 0 is gray / 255) and
//                polynomial expansion of up to three levels in ONE launch: 16x16 tiles, the pyramid
//                values a tile needs are rebuilt from the RGB frame in LDS; separable moments,
//                closed-form solution of the 6-unknown weighted least-squares fit
//   k_pyr_pair, k_polyexp   the same for more than three levels and larger frames: gray image and two
//                pyramid levels per launch, the pyramid in HBM, then the expansion of all levels
//   k_flow_tile, k_flow_small   one displacement update: per cell of a tile (32x32, 32x16 or 16x16, whichever takes
//                the fewest rounds of blocks) + 5-pixel halo, sample the new frame's expansion bilinearly at
//                x + prior, build A^T A (3 values) and A^T db (2 values) in LDS, separable 11x11 Gaussian
//                aggregation (on the matrix cores for the larger tiles), 2x2 ridge solve.  The coarse-to-fine
//                transfer (2 * bilinear of the coarser flow) is folded into the first update of a level, so G/h
//                fields never touch HBM.  Tiles are handed to the XCDs in contiguous runs so that neighbours share
//                an L2.
//   k_flow_fused  three updates of a small level in one launch (halo recomputed)
//   k_patch_motion, k_gate   per patch RMS flow magnitude (Eq. 5); static patches counted, the gate (Eq. 6).
//                Stand-alone flow call only: the chained step has them in its pooling kernels.
//
// The batched kernels take the frame as a grid dimension.  All stencils replicate the border.

#include <type_traits>

#include "sali_internal.h"
#include "saliency_body.h"

namespace sali {

namespace {

constexpr int kT = 32;                       // tile side of the expansion kernel
constexpr int kPR = kT + 2 * kPolyN;             // 38
constexpr int kPW = 40;                      // row of the region in whole quads: columns x0 - 4 .. x0 + 35

__device__ __forceinline__ uint32_t pix(int y, int w, int x) {          // y * w + x, both factors below 2^24
    return __umul24((uint32_t)y, (uint32_t)w) + (uint32_t)x;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// Two pyramid levels of every frame of the batch (blockIdx.z) in one launch: a block makes a 32x32 tile of
// level `lvl` and the 16x16 tile of level lvl + 1 under it (where there is one) from the source below, whose
// 76x73 patch it holds in LDS.  kRgb: the source is the frame itself; the block converts its patch to gray
// and also writes its 64x64 pixels of the gray image, so the frame is read once and no gray pass precedes.  The
// first level is then an exact integer sum (weights 1 4 6 4 1 squared, at most 256 * 255) and one division.
// Four 1920x1080 frames, five levels: 18 + 7.5 us for gray and four levels.  A thread per output with 25 byte
// loads and divisions each, a launch per level, after a gray pass: 8.7 + 41.6 + 9.9 + 4.8 + 4.8 us.
namespace {
constexpr int kPyrT = 32;                       // tile side of the first level
constexpr int kPyrR = kPyrT + 3;                // 35: cells of it that the second level reads
constexpr int kPyrRows = 2 * (kPyrR - 1) + 5;   // 73: source rows under them
constexpr int kPyrCols = 76;                    // source columns: from 64 bx - 8 (whole quads), 73 used
}  // namespace

template <bool kRgb>
__global__ __launch_bounds__(256) void k_pyr_pair(int tiles_x, int tiles_y, int n, int lvl, LevelGeom g, PyrBatch f) {
    using Cell = typename std::conditional<kRgb, uint8_t, float>::type;
    using Sum = typename std::conditional<kRgb, uint16_t, float>::type;
    __shared__ __align__(16) Cell s_src[kPyrRows][kPyrCols];
    __shared__ Sum s_h[kPyrRows][kPyrR + 1];            // horizontal sums
    __shared__ float s_l1[kPyrR][kPyrR + 1];
    const BlockId blk = xcd_block_id(tiles_x, tiles_y, n);
    const PyrFrame& frame = f.frame[blk.z];
    const int sh = g.h[lvl - 1], sw = g.w[lvl - 1], h1 = g.h[lvl], w1 = g.w[lvl];
    float* __restrict__ pyr = frame.pyr;
    together(sh, sw, h1, w1, frame.rgb, frame.y8, pyr, g.off[lvl - 1], g.off[lvl], g.levels);
    const int tid = threadIdx.x;
    const int qy = 64 * blk.y - 6, qx = 64 * blk.x - 8;         // origin of the patch
    constexpr int kQuads = kPyrCols / 4, kItems = kPyrRows * kQuads, kN = (kItems + 255) / 256;
    if constexpr (kRgb) {
        // a thread takes four pixels (twelve bytes, the compiler is told nothing about their alignment) at a
        // time and has all its loads in flight before the first is used
        const uint8_t* __restrict__ rgb = frame.rgb;
        uint32_t v[kN][3];
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int p = min(tid + 256 * k, kItems - 1);
            const int x = qx + 4 * (p % kQuads);
            load_rgb_quad(rgb + (size_t)clampi(qy + p / kQuads, 0, sh - 1) * sw * 3, x, sw, v[k]);
        }
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int p = tid + 256 * k;
            if (p < kItems) *reinterpret_cast<uint32_t*>(&s_src[p / kQuads][4 * (p % kQuads)]) = gray_of_quad(v[k]);
        }
    } else {
        const float* __restrict__ src = pyr + g.off[lvl - 1];
        constexpr int kCells = kPyrRows * kPyrCols;
#pragma unroll 8
        for (int p = tid; p < kCells; p += 256) {
            const int gy = clampi(qy + p / kPyrCols, 0, sh - 1), gx = clampi(qx + p % kPyrCols, 0, sw - 1);
            s_src[p / kPyrCols][p % kPyrCols] = src[(size_t)gy * sw + gx];
        }
    }
    __syncthreads();
    if constexpr (kRgb) {
        uint8_t* __restrict__ y8 = frame.y8;
#pragma unroll
        for (int k = 0; k < 4; ++k) {                           // 64 rows of sixteen quads
            const int p = tid + 256 * k;
            const int gy = 64 * blk.y + p / 16, gx = 64 * blk.x + 4 * (p % 16);
            if (gy >= sh || gx >= sw) continue;
            const uint32_t quad = *reinterpret_cast<const uint32_t*>(&s_src[6 + p / 16][8 + 4 * (p % 16)]);
            uint8_t* dst = y8 + (size_t)gy * sw + gx;
            if ((sw & 3) == 0) {
                *reinterpret_cast<uint32_t*>(dst) = quad;
            } else {
                for (int i = 0; i < 4 && gx + i < sw; ++i) dst[i] = (uint8_t)(quad >> (8 * i));
            }
        }
    }
    // Cells of the 35x35 region hold the value at the clamped coordinate of their place, as the patch does: a
    // replicate-border stencil centred on an in-image pixel reads exactly that.
    const int oy1 = kPyrT * blk.y - 2, ox1 = kPyrT * blk.x - 2;
    for (int p = tid; p < kPyrRows * kPyrR; p += 256) {
        const int ry = p / kPyrR, rx = p % kPyrR;
        const Cell* c = &s_src[ry][2 * clampi(ox1 + rx, 0, w1 - 1) - qx];
        if constexpr (kRgb) s_h[ry][rx] = (uint16_t)(c[-2] + c[2] + 4 * (c[-1] + c[1]) + 6 * c[0]);
        else s_h[ry][rx] = (c[-2] + c[2]) * (1.0f / 16) + (c[-1] + c[1]) * (4.0f / 16) + c[0] * (6.0f / 16);
    }
    __syncthreads();
    for (int p = tid; p < kPyrR * kPyrR; p += 256) {
        const int ry = p / kPyrR, rx = p % kPyrR;
        const int cy = 2 * clampi(oy1 + ry, 0, h1 - 1) - qy;
        float v;
        if constexpr (kRgb) {
            const uint32_t sum = (uint32_t)s_h[cy - 2][rx] + s_h[cy + 2][rx] + 4u * ((uint32_t)s_h[cy - 1][rx] + s_h[cy + 1][rx]) +
                                 6u * s_h[cy][rx];
            v = (float)sum / 65280.0f;
        } else {
            v = (s_h[cy - 2][rx] + s_h[cy + 2][rx]) * (1.0f / 16) + (s_h[cy - 1][rx] + s_h[cy + 1][rx]) * (4.0f / 16) +
                s_h[cy][rx] * (6.0f / 16);
        }
        s_l1[ry][rx] = v;
        const int gy = oy1 + ry, gx = ox1 + rx;
        if (ry >= 2 && ry < 2 + kPyrT && rx >= 2 && rx < 2 + kPyrT && gy < h1 && gx < w1)
            pyr[g.off[lvl] + (size_t)gy * w1 + gx] = v;
    }
    if (lvl + 1 >= g.levels) return;
    __syncthreads();
    const int h2 = g.h[lvl + 1], w2 = g.w[lvl + 1];
    const int ty = tid / 16, tx = tid % 16, gy = 16 * blk.y + ty, gx = 16 * blk.x + tx;
    if (gy >= h2 || gx >= w2) return;
    const float k[5] = {1.0f / 16, 4.0f / 16, 6.0f / 16, 4.0f / 16, 1.0f / 16};
    float acc = 0.0f;
#pragma unroll
    for (int a = 0; a < 5; ++a) {
        float row = 0.0f;
#pragma unroll
        for (int b = 0; b < 5; ++b) row += k[b] * s_l1[2 * ty + a][2 * tx + b];
        acc += k[a] * row;
    }
    pyr[g.off[lvl + 1] + (size_t)gy * w2 + gx] = acc;
}

// ---------------------------------------------------------------------------------------------
// Polynomial expansion f(x + d) ~ c + b.d + d^T A d over the 7x7 Gaussian-weighted window.
// With separable symmetric weights (sum 1, second moment m2, fourth moment m4) the normal
// equations decouple:  b = (sx, sy) / m2,  A_xx = (sxx - m2 s0) / (m4 - m2^2),  A_yy likewise,
// A_xy = sxy / (2 m2^2), where s* are the weighted correlations of f with 1, x, y, x^2, y^2, xy.
//
// Bound by the vector ALU, then by its writes (20 bytes a pixel): two 1920x1080 frames of five levels 26.5 us, 4.1 TB/s.  Cell by cell, with
// clamped coordinates, byte loads, a division each and 28 instructions a moment (values under the symmetric weights are now summed and subtracted
// in pairs first): 31.6.
//
// The launch that completes the expansions may carry the saliency pre-pass of its frames (Ride = PrepRide): blocks
// 0 .. ride.blocks - 1, so that these, the longest, start first.  Neither needs anything of the other.
namespace {
struct PolyexpShared {
    __attribute__((aligned(16))) float f[kPR][kPW], v[3][kT][kPW];
};
// the moments of seven values under the symmetric weights, from their sums and differences in pairs
struct PolyTaps {
    float g[4], kg[4], kkg[4];      // g_k, k g_k, k^2 g_k
};
__device__ __forceinline__ PolyTaps poly_taps(const FlowWeights& fw) {
    PolyTaps t;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        t.g[k] = fw.poly_g[kPolyN + k];
        t.kg[k] = t.g[k] * (float)k;
        t.kkg[k] = t.g[k] * (float)(k * k);
    }
    return t;
}
__device__ __forceinline__ float moment0(const PolyTaps& t, float f0, const float (&sum)[3]) {
    return t.g[0] * f0 + t.g[1] * sum[0] + t.g[2] * sum[1] + t.g[3] * sum[2];
}
__device__ __forceinline__ float moment1(const PolyTaps& t, const float (&diff)[3]) { return t.kg[1] * diff[0] + t.kg[2] * diff[1] + t.kg[3] * diff[2]; }
__device__ __forceinline__ float moment2(const PolyTaps& t, const float (&sum)[3]) { return t.kkg[1] * sum[0] + t.kkg[2] * sum[1] + t.kkg[3] * sum[2]; }
// LDS of a block that is either kind
template <typename Own, typename Ride>
struct WithPrep {
    union {
        Own own;
        PrepShared prep;
    };
};
template <typename Own>
struct WithPrep<Own, NoRide> {
    Own own;
};
// Is this block one of the `riders`?  Then it does its tile; the others get their number among the launch's own blocks (per_frame
// a frame, frame by frame).  Without riders the grid is (per_frame, frames).
template <int NT, typename Shared>
__device__ __forceinline__ bool ride_prep(Shared& sh, const PrepRide& ride, int riders, int, int& block) {
    block = (int)blockIdx.x - riders;
    if (block >= 0) return false;
    const int tiles = ride.tiles_x * ride.tiles_y, frame = (int)blockIdx.x / tiles, t = (int)blockIdx.x - frame * tiles;
    prep_tile<false, NT>(sh.prep, ride.f, t % ride.tiles_x, t / ride.tiles_x, frame, ride.h, ride.w, GateParams{}, ride.lut, ride.lo2, ride.hi2);
    return true;
}
template <int NT, typename Shared>
__device__ __forceinline__ bool ride_prep(Shared&, const NoRide&, int, int per_frame, int& block) {
    block = (int)blockIdx.x + per_frame * (int)blockIdx.y;
    return false;
}
}  // namespace

template <typename Ride>
__global__ __launch_bounds__(256) void k_polyexp(int riders, int per_frame, LevelGeom g, FlowWeights fw, PyrBatch f, Ride ride) {
    __shared__ WithPrep<PolyexpShared, Ride> sh;
    int block;
    if (ride_prep<256>(sh, ride, riders, per_frame, block)) return;
    int frame = (int)blockIdx.y, tile = (int)blockIdx.x;
    if constexpr (!std::is_same_v<Ride, NoRide>) {
        frame = block / per_frame;
        tile = block - frame * per_frame;
    }
    const PyrFrame& fr = f.frame[frame];
    const uint8_t* __restrict__ y8 = fr.y8;
    const float* __restrict__ pyr = fr.pyr;
    float4* __restrict__ A_out = fr.A;
    float* __restrict__ b_out = fr.b;
    together(y8, pyr, A_out, b_out);
    float (&s_f)[kPR][kPW] = sh.own.f;
    float (&s_v)[3][kT][kPW] = sh.own.v;

    int lvl = 0;
#pragma unroll
    for (int l = 1; l < kMaxLevels; ++l) lvl += l < g.levels && tile >= g.tile_start[l] ? 1 : 0;
    const int h = g.h[lvl], w = g.w[lvl];
    const int first = g.tile_start[lvl], tiles_x = g.tiles_x[lvl];
    const int64_t level_off = g.off[lvl];
    together(h, w, first, tiles_x, level_off);
    const int t = tile - first;
    const int x0 = (t % tiles_x) * kT, y0 = (t / tiles_x) * kT;
    const float* src = pyr + level_off;
    const int tid = threadIdx.x;

    // The region, a quad of columns at a time: 38 rows of ten.  Out-of-image cells hold the value at the clamped coordinate, which is exactly
    // what a replicate-border stencil centred on an in-image pixel reads.
    constexpr int kQuads = kPW / 4, kItems = kPR * kQuads, kN = (kItems + 255) / 256;
    auto region = [&](auto quad_at) {
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int p = min(tid + 256 * k, kItems - 1);               // the last ones are made again, the same
            const int gy = clampi(y0 - kPolyN + p / kQuads, 0, h - 1), x = x0 - 4 + 4 * (p % kQuads);
            *reinterpret_cast<float4*>(&s_f[p / kQuads][4 * (p % kQuads)]) = quad_at((size_t)gy * w, x);
        }
    };
    if (lvl == 0) {
        region([&](size_t row, int x) {
            uint32_t q;
            if (x >= 0 && x + 3 < w) {
                __builtin_memcpy(&q, y8 + row + x, 4);
            } else {
                q = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) q |= (uint32_t)y8[row + clampi(x + i, 0, w - 1)] << (8 * i);
            }
            return make_float4(whole_over<255>(q & 0xFFu), whole_over<255>((q >> 8) & 0xFFu), whole_over<255>((q >> 16) & 0xFFu), whole_over<255>(q >> 24));
        });
    } else {
        region([&](size_t row, int x) {
            float4 q;
            if (x >= 0 && x + 3 < w) {
                __builtin_memcpy(&q, src + row + x, 16);
            } else {
                q = make_float4(src[row + clampi(x, 0, w - 1)], src[row + clampi(x + 1, 0, w - 1)], src[row + clampi(x + 2, 0, w - 1)],
                                src[row + clampi(x + 3, 0, w - 1)]);
            }
            return q;
        });
    }
    __syncthreads();

    // vertical moments: a quad of columns, two rows
    const PolyTaps taps = poly_taps(fw);
    for (int p = tid; p < (kT / 2) * kQuads; p += 256) {
        const int ty = 2 * (p / kQuads), c = 4 * (p % kQuads);
        float f[8][4];
#pragma unroll
        for (int k = 0; k < 8; ++k) *reinterpret_cast<float4*>(f[k]) = *reinterpret_cast<const float4*>(&s_f[ty + k][c]);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            float m[3][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float sum[3], diff[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    sum[k] = f[r + 4 + k][i] + f[r + 2 - k][i];
                    diff[k] = f[r + 4 + k][i] - f[r + 2 - k][i];
                }
                m[0][i] = moment0(taps, f[r + 3][i], sum);
                m[1][i] = moment1(taps, diff);
                m[2][i] = moment2(taps, sum);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) *reinterpret_cast<float4*>(&s_v[j][ty + r][c]) = make_float4(m[j][0], m[j][1], m[j][2], m[j][3]);
        }
    }
    __syncthreads();

    // horizontal moments and the fit: a thread's four pixels lie in a column, eight rows apart
    const int tx = tid % kT, gx = x0 + tx;
    if (gx >= w) return;
#pragma unroll
    for (int r = 0; r < kT / 8; ++r) {
        const int ty = tid / kT + 8 * r, gy = y0 + ty;
        if (gy >= h) break;
        float v[3][7];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 7; ++k) v[j][k] = s_v[j][ty][tx + 1 + k];
        float sum[3][3], diff[3][3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                sum[j][k] = v[j][4 + k] + v[j][2 - k];
                diff[j][k] = v[j][4 + k] - v[j][2 - k];
            }
        const float s0 = moment0(taps, v[0][3], sum[0]), sx = moment1(taps, diff[0]), sxx = moment2(taps, sum[0]);
        const float sy = moment0(taps, v[1][3], sum[1]), sxy = moment1(taps, diff[1]), syy = moment0(taps, v[2][3], sum[2]);
        const size_t gi = level_off + (size_t)gy * w + gx;
        const float axx = (sxx - fw.m2 * s0) * fw.inv_den;
        const float ayy = (syy - fw.m2 * s0) * fw.inv_den;
        const float axy = sxy * fw.inv_2m2sq;
        A_out[gi] = make_float4(axx, axy, ayy, sx * fw.inv_m2);
        b_out[gi] = sy * fw.inv_m2;
    }
}

// ---------------------------------------------------------------------------------------------
// Pyramid + expansion in one launch for up to three levels: a block owns one 16x16 tile of level 2 or two tiles of level 1 or 0 and
// rebuilds the pyramid values it needs from the RGB frame in LDS (level 1 from a 47x47
// gray patch, level 2 from a 47x47 level-1 patch built from a 97x97 gray patch).  This recomputes
// some pyramid pixels but removes two dependent launches and all pyramid traffic.
//
// The level-2 tile is the launch's length: trip for its patch, two pyramid stages, moments (3.4, 2.6, 0.6 and 0.8 of 8.9 us on 256 threads
// with a byte read per tap).  On 512 threads, its first stage by byte dot products, a launch for two 336x336 frames takes 10.2 us instead
// of 13.4, for one frame with the pre-pass 13.3 instead of 18.2.
namespace {
constexpr int kET = 16;                        // tile side
constexpr int kER = kET + 2 * kPolyN;          // 22: region the expansion stencil reads
constexpr int kEP = 2 * (kER - 1) + 5;         // 47: region one level below that feeds it
constexpr int kEQ = 2 * (kEP - 1) + 5;         // 97: region two levels below
constexpr int kExpandThreads = 512, kExpandHalf = kExpandThreads / 2;
// The 47-wide float patch of a level-2 tile is de-interleaved: even columns from float 24 of a row on, row stride 59, so
// that the stage reading it (22 cells per row) sees addresses linear in its thread index (pyr_level_lds:
// 2 * 59 = 22 mod 32).  The gray patches stay in bytes, plain layout, rows of 112 and 52 bytes: a stage that reads one takes two
// words per row and cell, neighbouring cells half a word apart.
constexpr int kEvenP = 24, kEPS = 59;
constexpr int kEQB = 112, kEPB = 52;
static_assert(kEvenP + (kEP + 1) / 2 <= kEPS && kEvenP >= kEP / 2, "a row holds both halves");
static_assert(kEQB % 4 == 0 && kEQB >= (kEQ + 3) / 4 * 4 && kEPB % 4 == 0 && kEPB >= (kEP + 3) / 4 * 4, "byte rows");

// LDS patches that feed a pyramid stage keep the odd columns of a row in its first part and the even
// columns from kEven on (kEven = 0: plain layout): the stage reads columns 2 * cx + {-2..2}, a stride
// of two over the lanes, which in the plain layout puts two lanes on every bank (measured: bank-conflict
// cycles were 45 % of the kernel's LDS cycles); de-interleaved, every tap is a unit-stride read.
template <int kEven>
__device__ __forceinline__ int lds_col(int c) {
    return kEven == 0 ? c : (c & 1 ? 0 : kEven) + (c >> 1);
}

// one level of the 5x5 binomial pyramid, LDS to LDS.  dst cell i (i < kN) stands for the
// coordinate clamp(o_dst + i) of the upper level and reads src cells 2 * that + {-2..2} - o_src
// (o_src is even, so the parity of a tap's column is the parity of the tap).  Threads take the cells in
// row-major order, kLanesPerRow (>= kN) lanes per row; with 2 * kSrcStride = kLanesPerRow (mod 32) the
// address of a tap is thread index + constant, i.e. free of bank conflicts.
template <int kSrcStride, int kSrcEven, int kDstStride, int kDstEven, int kN, int kLanesPerRow>
__device__ __forceinline__ void pyr_level_lds(const float* src, int o_src_y, int o_src_x, float* dst, int o_dst_y,
                                              int o_dst_x, int dh, int dw) {
    static_assert((2 * kSrcStride - kLanesPerRow) % 32 == 0, "tap addresses must be linear in the thread index");
    const float k[5] = {1.0f / 16, 4.0f / 16, 6.0f / 16, 4.0f / 16, 1.0f / 16};
    for (int p = threadIdx.x; p < kN * kLanesPerRow; p += kExpandThreads) {
        const int ry = p / kLanesPerRow, rx = p % kLanesPerRow;
        if (rx >= kN) continue;
        const int cy = clampi(o_dst_y + ry, 0, dh - 1), cx = clampi(o_dst_x + rx, 0, dw - 1);
        const int sy = 2 * cy - o_src_y, sx = 2 * cx - o_src_x;
        float acc = 0.0f;
#pragma unroll
        for (int a = -2; a <= 2; ++a) {
            float row = 0.0f;
#pragma unroll
            for (int b = -2; b <= 2; ++b) row += k[b + 2] * src[(sy + a) * kSrcStride + lds_col<kSrcEven>(sx + b)];
            acc += k[a + 2] * row;
        }
        dst[ry * kDstStride + lds_col<kDstEven>(rx)] = acc;
    }
}
// Patch of kSide x kSide pixels with origin (qy, qx) (coordinates clamped to the image) as gray, straight from the frame: a
// gray image of its own would be a launch before this one that nothing else reads.  put(row, column, four gray bytes) for
// every quad of columns.  All of a thread's loads are issued before the first one is used: written as one loop the
// compiler waits for every one in turn, and next to a kernel that saturates the memory system each takes
// microseconds.
template <int kSide, int NT, typename Put>
__device__ __forceinline__ void load_gray_patch(const uint8_t* __restrict__ rgb, int h0, int w0, int qy, int qx, int tid, Put put) {
    constexpr int kQuads = (kSide + 3) / 4, kItems = kSide * kQuads, kN = (kItems + NT - 1) / NT;
    uint32_t v[kN][3];
#pragma unroll
    for (int k = 0; k < kN; ++k) {
        const int p = min(tid + NT * k, kItems - 1);
        load_rgb_quad(rgb + (size_t)clampi(qy + p / kQuads, 0, h0 - 1) * w0 * 3, qx + 4 * (p % kQuads), w0, v[k]);
    }
#pragma unroll
    for (int k = 0; k < kN; ++k) {
        const int p = tid + NT * k;
        if (p < kItems) put(p / kQuads, 4 * (p % kQuads), gray_of_quad(v[k]));
    }
}
// as gray / 255, row stride kSide
template <int kSide, int NT>
__device__ __forceinline__ void load_gray_floats(const uint8_t* __restrict__ rgb, int h0, int w0, int qy, int qx, int tid,
                                                 float* __restrict__ dst) {
    load_gray_patch<kSide, NT>(rgb, h0, w0, qy, qx, tid, [&](int row, int col, uint32_t quad) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (col + i < kSide) dst[row * kSide + col + i] = whole_over<255>((quad >> (8 * i)) & 0xFFu);
    });
}
// as bytes, rows of kRowBytes
template <int kSide, int kRowBytes, int NT>
__device__ __forceinline__ void load_gray_bytes(const uint8_t* __restrict__ rgb, int h0, int w0, int qy, int qx, int tid,
                                                uint32_t* __restrict__ dst) {
    load_gray_patch<kSide, NT>(rgb, h0, w0, qy, qx, tid, [&](int row, int col, uint32_t quad) { dst[row * (kRowBytes / 4) + col / 4] = quad; });
}

// First pyramid level from a byte patch: the 5x5 binomial sum in integers (weights
// 1 4 6 4 1 squared: at most 256 * 255, exact) and one division by 256 * 255, i.e. the level-1 value of
// gray / 255 rounded once.  dst cell i stands for the coordinate clamp(o_dst + i), as in pyr_level_lds; its leftmost tap lies at an even
// column of the patch (o_src is even), so the five taps of a row are in two words.
template <int kRowBytes, int kDstStride, int kDstEven, int kN, int NT>
__device__ __forceinline__ void pyr_level_from_bytes(const uint32_t* src, int o_src_y, int o_src_x, float* dst, int o_dst_y, int o_dst_x,
                                                     int dh, int dw, int tid) {
    const uint32_t k[5] = {1u, 4u, 6u, 4u, 1u};
#pragma unroll 2
    for (int p = tid; p < kN * kN; p += NT) {
        const int ry = p / kN, rx = p % kN;
        const int cy = clampi(o_dst_y + ry, 0, dh - 1), cx = clampi(o_dst_x + rx, 0, dw - 1);
        const int c = 2 * cx - o_src_x - 2, top = 2 * cy - o_src_y - 2;
        const uint32_t* at = src + top * (kRowBytes / 4) + (c >> 2);
        const uint32_t shift = 8u * ((uint32_t)c & 3u);                 // 0 or 16
        uint32_t acc = 0u;
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            const uint32_t w0 = at[a * (kRowBytes / 4)], w1 = at[a * (kRowBytes / 4) + 1];
            const uint32_t four = __builtin_amdgcn_alignbit(w1, w0, shift), fifth = (w1 >> shift) & 0xFFu;
            acc += k[a] * __builtin_amdgcn_udot4(four, 0x04060401u, fifth, false);
        }
        dst[ry * kDstStride + lds_col<kDstEven>(rx)] = whole_over<65280>(acc);
    }
}

struct ExpandTile {                     // a tile of level 0 or 1, half a block
    uint32_t pb[kEP * (kEPB / 4)];      // gray patch of a level-1 tile, bytes
    // unpadded rows: both the pass that writes these arrays and the pass that reads them then see
    // addresses linear in the thread index (the horizontal pass pairs rows eight apart, see below)
    float f[kER][kER];
    float v[3][kET][kER];               // vertical moments
};
struct ExpandTile2 {                    // a tile of level 2, the whole block
    uint32_t qb[kEQ * (kEQB / 4)];      // gray patch, bytes; vertical moments later
    float p[kEP * kEPS];                // level-1 patch
    float f[kER][kER];
};
union ExpandShared {
    ExpandTile half[2];
    ExpandTile2 whole;
};
static_assert(sizeof(float) * 3 * kET * kER <= sizeof(uint32_t) * kEQ * (kEQB / 4), "moments fit into the byte patch");

}  // namespace

// c0, c1, c2: a frame's tiles of each level
template <typename Ride>
__global__ __launch_bounds__(kExpandThreads) void k_expand(int riders, int n_frames, int c0, int c1, int c2, int tx0, int tx1, int tx2,
                                                           LevelGeom g, FlowWeights fw, ExpandBatch f, Ride ride) {
    __shared__ WithPrep<ExpandShared, Ride> sh;
    const int b0 = (c0 + 1) / 2, b1 = (c1 + 1) / 2;             // blocks of a frame's levels 0 and 1
    int idx;
    if (ride_prep<kExpandThreads>(sh, ride, riders, c2 + b1 + b0, idx)) return;
    // Work order.  A level-2 tile costs about ten times a level-0 tile (97 x 97 gray pixels, two pyramid
    // stages) and there are sixteen level-0 tiles for each: with the tiles of a frame in level order the
    // heavy ones start last and the launch ends with a few of them on an idle chip (22 us per four
    // 336x336 frames, 10 of them that tail).  So the linear block id is cut into runs, heaviest first,
    // each run over all frames of the batch: level-2 tiles, level-1 tiles, level-0 tiles.
    const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kExpandHalf);
    int lvl, t, frame, count;
    if (idx < n_frames * c2) {
        lvl = 2;
        count = c2;
        frame = idx / c2;
        t = idx - frame * c2;
    } else if ((idx -= n_frames * c2) < n_frames * b1) {
        lvl = 1;
        count = c1;
        frame = idx / b1;
        t = 2 * (idx - frame * b1) + half;
    } else {
        idx -= n_frames * b1;
        lvl = 0;
        count = c0;
        frame = idx / b0;
        t = 2 * (idx - frame * b0) + half;
    }
    const bool spare = t >= count;                              // the second tile of a last block: done again, not stored
    t = min(t, count - 1);
    const ExpandFrame& fr = f.frame[frame];
    const uint8_t* __restrict__ rgb = fr.rgb;
    float4* __restrict__ A_out = fr.A;
    float* __restrict__ b_out = fr.b;
    together(rgb, A_out, b_out, g.h[0], g.w[0], g.h[1], g.w[1], g.h[2], g.w[2], g.off[1], g.off[2]);
    const int tiles_x = lvl == 0 ? tx0 : (lvl == 1 ? tx1 : tx2);
    const int h = lvl == 0 ? g.h[0] : (lvl == 1 ? g.h[1] : g.h[2]), w = lvl == 0 ? g.w[0] : (lvl == 1 ? g.w[1] : g.w[2]);
    const int64_t level_off = lvl == 0 ? 0 : (lvl == 1 ? g.off[1] : g.off[2]);
    const int x0 = (t % tiles_x) * kET, y0 = (t / tiles_x) * kET;
    const int oy = y0 - kPolyN, ox = x0 - kPolyN;   // origin of s_f in this level's coordinates
    const int tid = threadIdx.x % kExpandHalf;
    const int h0 = g.h[0], w0 = g.w[0];
    float (*s_f)[kER] = lvl == 2 ? sh.own.whole.f : sh.own.half[half].f;
    float (*s_v)[kET][kER] = lvl == 2 ? reinterpret_cast<float (*)[kET][kER]>(sh.own.whole.qb) : sh.own.half[half].v;

    if (lvl == 0) {
        load_gray_floats<kER, kExpandHalf>(rgb, h, w, oy, ox, tid, &s_f[0][0]);
    } else if (lvl == 1) {
        const int qy = 2 * oy - 2, qx = 2 * ox - 2;              // origin of the gray patch (47 x 47)
        uint32_t* s_pb = sh.own.half[half].pb;
        load_gray_bytes<kEP, kEPB, kExpandHalf>(rgb, h0, w0, qy, qx, tid, s_pb);
        __syncthreads();
        pyr_level_from_bytes<kEPB, kER, 0, kER, kExpandHalf>(s_pb, qy, qx, &s_f[0][0], oy, ox, h, w, tid);
    } else {
        const int h1 = g.h[1], w1 = g.w[1];
        const int py = 2 * oy - 2, px = 2 * ox - 2;              // origin of the level-1 patch (47 x 47)
        const int qy = 2 * py - 2, qx = 2 * px - 2;              // origin of the gray patch (97 x 97)
        load_gray_bytes<kEQ, kEQB, kExpandThreads>(rgb, h0, w0, qy, qx, (int)threadIdx.x, sh.own.whole.qb);
        __syncthreads();
        pyr_level_from_bytes<kEQB, kEPS, kEvenP, kEP, kExpandThreads>(sh.own.whole.qb, qy, qx, sh.own.whole.p, py, px, h1, w1, (int)threadIdx.x);
        __syncthreads();
        pyr_level_lds<kEPS, kEvenP, kER, 0, kER, kER>(sh.own.whole.p, py, px, &s_f[0][0], oy, ox, h, w);
    }
    __syncthreads();

    // vertical moments, then horizontal moments and the closed-form fit (as in k_polyexp)
    const int step = lvl == 2 ? kExpandThreads : kExpandHalf;
    for (int p = lvl == 2 ? (int)threadIdx.x : tid; p < kET * kER; p += step) {
        const int ty = p / kER, rx = p % kER;
        float v0 = 0.0f, v1 = 0.0f, v2 = 0.0f;
#pragma unroll
        for (int k = -kPolyN; k <= kPolyN; ++k) {
            const float f = s_f[ty + kPolyN + k][rx] * fw.poly_g[k + kPolyN];
            v0 += f;
            v1 += f * (float)k;
            v2 += f * (float)(k * k);
        }
        s_v[0][ty][rx] = v0;
        s_v[1][ty][rx] = v1;
        s_v[2][ty][rx] = v2;
    }
    __syncthreads();
    if (spare || (lvl == 2 && half != 0)) return;
    {
        // a group of 32 lanes takes the rows r and r + 8 (16 lanes each): 8 rows of 22 floats are 176 =
        // 16 (mod 32) floats apart, so the two rows lie on disjoint banks
        const int pair = tid / kET, tx = tid % kET;
        const int ty = (pair >> 1) + 8 * (pair & 1);
        const int gy = y0 + ty, gx = x0 + tx;
        if (gy < h && gx < w) {
            float s0 = 0, sx = 0, sxx = 0, sy = 0, sxy = 0, syy = 0;
#pragma unroll
            for (int k = -kPolyN; k <= kPolyN; ++k) {
                const float gk = fw.poly_g[k + kPolyN];
                const float a0 = s_v[0][ty][tx + kPolyN + k] * gk;
                const float a1 = s_v[1][ty][tx + kPolyN + k] * gk;
                const float a2 = s_v[2][ty][tx + kPolyN + k] * gk;
                s0 += a0;
                sx += a0 * (float)k;
                sxx += a0 * (float)(k * k);
                sy += a1;
                sxy += a1 * (float)k;
                syy += a2;
            }
            const size_t gi = level_off + (size_t)gy * w + gx;
            A_out[gi] = make_float4((sxx - fw.m2 * s0) * fw.inv_den, sxy * fw.inv_2m2sq, (syy - fw.m2 * s0) * fw.inv_den,
                                    sx * fw.inv_m2);
            b_out[gi] = sy * fw.inv_m2;
        }
    }
}

// ---------------------------------------------------------------------------------------------
namespace {

// Prior displacement of a pixel in the first update of a level that is not the coarsest: 2 * the coarser flow at (y / 2, x / 2), bilinear,
// coordinates clamped to it.  The weights are 1 and 0 or both a half, and past the last row or column (an odd pixel of an even size)
// both samples are the last one.
struct CoarseCell {
    float2 a, b, c, d;
};
__device__ __forceinline__ float2 transfer_of(const CoarseCell& v) {
    // each pair's mean is exact but for one rounding of the sum, as is 2 * the mean of the two
    const float tx = 0.5f * (v.a.x + v.b.x), ty = 0.5f * (v.a.y + v.b.y), bx = 0.5f * (v.c.x + v.d.x), by = 0.5f * (v.c.y + v.d.y);
    return make_float2(tx + bx, ty + by);
}

// The coarser flow under a region of a finer level that starts at (ry, rx) (odd) and is 2 (CX - 1) x 2 (CY - 1) pixels large, in LDS.  A cell of
// it serves up to sixteen of the loads that priors took one by one (four a pixel), which were half as much
// work for the load path as the samples: first updates of 3 x 1920x1080 128 -> 107 us, one 35 -> 31, 15 x 640x360 57 -> 49.
template <int CX, int CY>
struct CoarsePatch {
    float2 v[CX * CY];
};
template <int NT, int CX, int CY>
__device__ __forceinline__ void load_coarse(CoarsePatch<CX, CY>& patch, const float2* __restrict__ coarse, int ry, int rx, int ch, int cw) {
    for (int p = threadIdx.x; p < CX * CY; p += NT)
        patch.v[p] = ld_at(coarse, pix(clampi((ry >> 1) + p / CX, 0, ch - 1), cw, clampi((rx >> 1) + p % CX, 0, cw - 1)));
}
template <int CX, int CY>
__device__ __forceinline__ float2 transfer_from(const CoarsePatch<CX, CY>& patch, int ry, int rx, int y, int x, int ch, int cw) {
    const int r0 = ((y >> 1) - (ry >> 1)) * CX, r1 = (min((y >> 1) + (y & 1), ch - 1) - (ry >> 1)) * CX;
    const int c0 = (x >> 1) - (rx >> 1), c1 = min((x >> 1) + (x & 1), cw - 1) - (rx >> 1);
    return transfer_of({patch.v[r0 + c0], patch.v[r0 + c1], patch.v[r1 + c0], patch.v[r1 + c1]});
}

// size of a level and the coordinates of its last row and column, in scalar registers
struct Extent {
    int h, w;
    float last_y, last_x;
};
__device__ __forceinline__ Extent extent_of(int h, int w) {
    auto uniform = [](float v) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v))); };
    return {h, w, uniform((float)(h - 1)), uniform((float)(w - 1))};
}

// the old frame's expansion at a pixel
struct OldCell {
    float4 A;
    float by;
};
__device__ __forceinline__ OldCell old_cell(const float4* __restrict__ A1, const float* __restrict__ b1, uint32_t gi) {
    return {ld_at(A1, gi), ld_at(b1, gi)};
}

// A^T A (xx, xy, yy) and A^T db (x, y) of the pixel (gy, gx) with prior displacement dp: the old frame's
// expansion there, the new frame's sampled at the pixel + dp.  The upper left of the four samples is clamped to the
// last but one row and column (an image level has at least two of each; at the border the weight of the other
// row or column is then exactly one), so that the others lie at fixed distances from it: no coordinates, products and
// offsets of their own, and the two samples of a row of b in one load.  Which sums are fused is written out, here and in
// flow_solve: left to the compiler it depended on the code around, and kernels for other sizes of the same level must agree bit by bit.
__device__ __forceinline__ void flow_terms(const OldCell& old, const float4* __restrict__ A2, const float* __restrict__ b2, const Extent& e,
                                           int gy, int gx, float2 dp, float (&t)[5]) {
#pragma clang fp contract(off)
    const int h = e.h, w = e.w;
    const float4 a1 = old.A;
    const float b1y = old.by;
    const float sy = __builtin_amdgcn_fmed3f((float)gy + dp.y, 0.0f, e.last_y);       // not a number: 0
    const float sx = __builtin_amdgcn_fmed3f((float)gx + dp.x, 0.0f, e.last_x);
    const int iy0 = min((int)sy, h - 2), ix0 = min((int)sx, w - 2);
    const float wy = sy - (float)iy0, wx = sx - (float)ix0;
    const uint32_t i0 = pix(iy0, w, ix0), i1 = i0 + (uint32_t)w;
    const float4 a00 = ld_at(A2, i0), a01 = ld_at(A2 + 1, i0), a10 = ld_at(A2, i1), a11 = ld_at(A2 + 1, i1);
    float c0[2], c1[2];                      // four-byte alignment only
    __builtin_memcpy(c0, reinterpret_cast<const char*>(b2) + i0 * 4u, 8);
    __builtin_memcpy(c1, reinterpret_cast<const char*>(b2) + i1 * 4u, 8);
    const float w00 = (1.0f - wx) * (1.0f - wy), w01 = wx * (1.0f - wy), w10 = (1.0f - wx) * wy, w11 = wx * wy;
    auto sampled = [&](float v00, float v01, float v10, float v11) {
        return __builtin_fmaf(v11, w11, __builtin_fmaf(v10, w10, __builtin_fmaf(v01, w01, v00 * w00)));
    };
    const float a2xx = sampled(a00.x, a01.x, a10.x, a11.x), a2xy = sampled(a00.y, a01.y, a10.y, a11.y);
    const float a2yy = sampled(a00.z, a01.z, a10.z, a11.z), b2x = sampled(a00.w, a01.w, a10.w, a11.w);
    const float b2y = sampled(c0[0], c0[1], c1[0], c1[1]);
    const float axx = 0.5f * (a1.x + a2xx), axy = 0.5f * (a1.y + a2xy), ayy = 0.5f * (a1.z + a2yy);
    const float dbx = __builtin_fmaf(axy, dp.y, __builtin_fmaf(axx, dp.x, -0.5f * (b2x - a1.w)));
    const float dby = __builtin_fmaf(ayy, dp.y, __builtin_fmaf(axy, dp.x, -0.5f * (b2y - b1y)));
    t[0] = __builtin_fmaf(axx, axx, axy * axy);
    t[1] = axy * (axx + ayy);
    t[2] = __builtin_fmaf(ayy, ayy, axy * axy);
    t[3] = __builtin_fmaf(axx, dbx, axy * dby);
    t[4] = __builtin_fmaf(axy, dbx, ayy * dby);
}

// the displacement from the windowed sums of the terms and the prior (ridge term centred on the prior).  The two
// quotients share one reciprocal, refined to the last place, and each gets a step of its own (at most half a unit in
// the last place and a little more); the ridge term keeps the determinant above 1e-8, so nothing has to be scaled as
// a general division does.
__device__ __forceinline__ float2 flow_solve(float g11, float g12, float g22, float h1, float h2, float2 dp) {
#pragma clang fp contract(off)
    const float lam = __builtin_fmaf(kLamRel * 0.5f, g11 + g22, kLamAbs);
    const float m11 = g11 + lam, m22 = g22 + lam;
    const float r1 = __builtin_fmaf(lam, dp.x, h1), r2 = __builtin_fmaf(lam, dp.y, h2);
    const float det = __builtin_fmaf(m11, m22, -(g12 * g12));
    float inv = __builtin_amdgcn_rcpf(det);
    inv = __builtin_fmaf(__builtin_fmaf(-det, inv, 1.0f), inv, inv);
    const float nx = __builtin_fmaf(m22, r1, -(g12 * r2)), ny = __builtin_fmaf(m11, r2, -(g12 * r1));
    const float qx = nx * inv, qy = ny * inv;
    return make_float2(__builtin_fmaf(__builtin_fmaf(-det, qx, nx), inv, qx), __builtin_fmaf(__builtin_fmaf(-det, qy, ny), inv, qy));
}

// Window passes on the matrix cores.  v_mfma_f32_4x4x1f32 is sixteen independent outer products of four weights and
// four values; with the lane's weight k of the window's row `lane % 4` as the one operand and a value of the
// lane's own as the other, fourteen of them give every lane four neighbouring outputs of the eleven-tap window,
//   out[i] = sum_k w[k - i] v[k],  i = 0..3,
// from the fourteen values under them, in fp32, lane by lane: what 44 multiply-adds of the vector ALU do, which then
// is free for the warped samples.  Lanes do not mix, but all 64 must be there: the weights come from all of a block of
// four, so callers keep their control flow uniform over the wave and let idle lanes repeat an item.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kFirOut = 4, kFirIn = 2 * kWinR + kFirOut;              // 14

struct FirWeights {
    float k[kFirIn];
};
constexpr int kFirTable = kFirIn + 3;
// three zeros, the window, three zeros, in LDS (written by the first threads, one barrier before its use)
__device__ __forceinline__ void fir_table(float* s_w, const FlowWeights& fw) {
    if (threadIdx.x < kFirTable) {
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k <= 2 * kWinR; ++k) v = (int)threadIdx.x == 3 + k ? fw.win_g[k] : v;
        s_w[threadIdx.x] = v;
    }
}
__device__ __forceinline__ FirWeights fir_weights(const float* s_w) {
    FirWeights w;
#pragma unroll
    for (int k = 0; k < kFirIn; ++k) w.k[k] = s_w[k + 3 - (threadIdx.x & 3)];
    return w;
}
__device__ __forceinline__ f32x4 fir4(const FirWeights& w, const float* v) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < kFirIn; ++k) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(w.k[k], v[k], acc, 0, 0, 0);
    return acc;
}
// N windows abreast: consecutive products do not wait for one another (one window's follow each other every four cycles at best)
template <int N>
__device__ __forceinline__ void fir4_abreast(const FirWeights& w, const float (&v)[N][16], f32x4* acc) {
    __builtin_amdgcn_sched_barrier(0);      // all reads ahead of the products: taken as they go they cost an LDS trip every few
#pragma unroll
    for (int n = 0; n < N; ++n) acc[n] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < kFirIn; ++k)
#pragma unroll
        for (int n = 0; n < N; ++n) acc[n] = __builtin_amdgcn_mfma_f32_4x4x1f32(w.k[k], v[n][k], acc[n], 0, 0, 0);
}
// four outputs of the row pass from sixteen floats at p (16-byte aligned; the last two come with the fourth load and are not used)
__device__ __forceinline__ f32x4 fir4_row(const FirWeights& w, const float* p) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(v + 4 * i) = *reinterpret_cast<const f32x4*>(p + 4 * i);
    return fir4(w, v);
}
// four outputs of the column pass, rows `stride` apart
__device__ __forceinline__ f32x4 fir4_column(const FirWeights& w, const float* p, int stride) {
    float v[kFirIn];
#pragma unroll
    for (int k = 0; k < kFirIn; ++k) v[k] = p[k * stride];
    return fir4(w, v);
}

}  // namespace

// One update of a small level: 16x16 tiles on 256 threads.  Here the block is a short chain and the chip is not full,
// so the window passes stay on the vector ALU with one output per lane (84x84 x 4 frames 5.8 us a launch, with the
// matrix cores' four outputs per lane 6.7: a quarter of the lanes at work, each on a serial chain).
constexpr int kSmallTile = 16, kSmallThreads = 256;
__global__ __launch_bounds__(kSmallThreads) void k_flow_small(int tiles_x, int tiles_y, int n, int h, int w, int ch, int cw, int prior_mode,
                                                              FlowWeights fw, FlowBatch f) {
    // blk.z = frame of the batch, (blk.x, blk.y) = tile
    const BlockId blk = xcd_block_id(tiles_x, tiles_y, n);
    const FlowFrame fr = f.frame[blk.z];
    together(fr.A1, fr.A2, fr.b1, fr.b2, fr.d_in, fr.d_out);
    const Extent extent = extent_of(h, w);
    constexpr int T = kSmallTile, NT = kSmallThreads, R = T + 2 * kWinR;       // 26: tile and halo
    // A group of 32 lanes of a window pass reads two rows (16 lanes each), which must lie 16 banks apart.  The two
    // rows of a group are eight apart (window_item) and the rows are unpadded: 8 * 26 = 16 mod 32; the pass that
    // writes the terms then sees addresses linear in the thread index, and a block takes 17 136 bytes, so that eight
    // blocks fill every wave slot of a compute unit.
    static_assert((8 * R) % 32 == 16, "rows eight apart sit 16 banks apart");
    __shared__ float s_in[5][R][R];
    __shared__ float2 s_dp[T][T];            // prior of the tile's own pixels, for the solve
    __shared__ CoarsePatch<R / 2 + 1, R / 2 + 1> s_coarse;

    const int tid = threadIdx.x;
    const int x0 = blk.x * T, y0 = blk.y * T;
    if (prior_mode == 1) {
        load_coarse<NT>(s_coarse, fr.d_in, y0 - kWinR, x0 - kWinR, ch, cw);
        __syncthreads();
    }

    // per-cell A^T A and A^T db at the clamped coordinate of the cell
#pragma unroll 2
    for (int p = tid; p < R * R; p += NT) {
        const int ry = p / R, rx = p % R;
        const int gy = clampi(y0 - kWinR + ry, 0, h - 1), gx = clampi(x0 - kWinR + rx, 0, w - 1);
        const OldCell old = old_cell(fr.A1, fr.b1, pix(gy, w, gx));
        const float2 dp = prior_mode == 0 ? make_float2(0.0f, 0.0f)
                          : prior_mode == 1 ? transfer_from(s_coarse, y0 - kWinR, x0 - kWinR, gy, gx, ch, cw) : ld_at(fr.d_in, pix(gy, w, gx));
        if (ry >= kWinR && ry < kWinR + T && rx >= kWinR && rx < kWinR + T) s_dp[ry - kWinR][rx - kWinR] = dp;
        float t[5];
        flow_terms(old, fr.A2, fr.b2, extent, gy, gx, dp, t);
#pragma unroll
        for (int c = 0; c < 5; ++c) s_in[c][ry][rx] = t[c];
    }
    __syncthreads();
    // Item p of a pass over n_rows rows of 16 outputs: the 32 lanes of a group take rows r and r + 8, first the whole
    // blocks of 16 rows, then the rest (ten rows in the row pass: two pairs, six rows with an idle half each).
    auto window_item = [](int p, int n_rows, int& row, int& col) {
        const int g = p >> 5, half = (p >> 4) & 1;
        col = p & 15;
        const int full = n_rows / 16, base = 16 * full;
        if (g < 8 * full) {
            row = (g >> 3) * 16 + (g & 7) + 8 * half;
            return true;
        }
        const int rest = n_rows - base, gg = g - 8 * full, npair = rest > 8 ? rest - 8 : 0;
        if (gg < npair) {
            row = base + gg + 8 * half;
            return true;
        }
        row = base + npair + (gg - npair);
        return half == 0 && row < base + (rest > 8 ? 8 : rest);
    };
    {
        // Row pass of the separable Gaussian window, in place: every thread keeps the sums of its (at most two) outputs
        // in registers until all taps of all threads are read, then writes them over the terms at [ry][tx].
        constexpr int kRowItems = 2;
        static_assert(32 * (8 + 2 + 6) <= kRowItems * NT, "26 rows: eight pairs, two pairs and six singles");
        float racc[kRowItems][5];
#pragma unroll
        for (int q = 0; q < kRowItems; ++q) {
            int ry, tx;
            const bool mine = window_item(tid + q * NT, R, ry, tx);
#pragma unroll
            for (int c = 0; c < 5; ++c) racc[q][c] = 0.0f;
            if (mine) {
#pragma unroll
                for (int k = 0; k <= 2 * kWinR; ++k) {
                    const float wk = fw.win_g[k];
#pragma unroll
                    for (int c = 0; c < 5; ++c) racc[q][c] += wk * s_in[c][ry][tx + k];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRowItems; ++q) {
            int ry, tx;
            if (window_item(tid + q * NT, R, ry, tx)) {
#pragma unroll
                for (int c = 0; c < 5; ++c) s_in[c][ry][tx] = racc[q][c];
            }
        }
        __syncthreads();
    }

    // column pass + ridge solve
    int ty, tx;
    window_item(tid, T, ty, tx);
    const int gy = y0 + ty, gx = x0 + tx;
    if (gy >= h || gx >= w) return;
    float acc[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k <= 2 * kWinR; ++k) {
        const float wk = fw.win_g[k];
#pragma unroll
        for (int c = 0; c < 5; ++c) acc[c] += wk * s_in[c][ty + k][tx];
    }
    *reinterpret_cast<float2*>(reinterpret_cast<char*>(fr.d_out) + pix(gy, w, gx) * 8u) =
        flow_solve(acc[0], acc[1], acc[2], acc[3], acc[4], s_dp[ty][tx]);
}

// ---------------------------------------------------------------------------------------------
// One update of a large level: tiles 32 wide on 512 threads, the window passes on the matrix cores.
//
// Three 1920x1080 frames: 84 to 90 us an update, one: 28, fifteen 640x360: 44.  With the windows on the vector ALU (110
// multiply-adds and as many LDS reads a pixel and 1.6 rows of halo, 32x16 tiles, per-cell index arithmetic, divisions)
// 518 vector instructions a pixel kept the ALU 91 % busy: 102, 37 and 59 us.  Now it is 45 % busy (260 instructions)
// and the trips of the warped samples bound the kernel: 12 000 of a block's 21 000 cycles.  Everything that costs a block
// or a wave shows: 16 waves a block (32x32 on 1024 threads) 100 us, registers spilled under the 64 that eight waves per
// SIMD leave 94 to 140 (five fields' products in step, or marching down a strip while ten rows of sums stay in LDS),
// 48-wide tiles 104 to 121; 64x32 on 1024 threads is as fast but needs sixteen free wave slots on one compute unit.  The
// same windows as banded matrix products
// (v_mfma_f32_16x16x4f32, the row pass's result the column pass's operand) took 100: 28 and 32 terms for eleven.
constexpr int kTileX = 32, kTileThreads = 512;
//
// kFirst: the first update of a level (prior_mode 0 or 1), whose priors come from the coarser level's flow, staged in LDS: 107, 31 and 49 us.  The
// others know that a prior is one load.  Both have the priors of all the thread's cells before the first sample.
template <int TY, bool kFirst>
__global__ __launch_bounds__(kTileThreads, 8) void k_flow_tile(int tiles_x, int tiles_y, int n, int h, int w, int ch, int cw, int first_mode,
                                                               FlowWeights fw, FlowBatch f) {
    const int prior_mode = kFirst ? first_mode : 2;
    const BlockId blk = xcd_block_id(tiles_x, tiles_y, n);
    const FlowFrame fr = f.frame[blk.z];
    together(fr.A1, fr.A2, fr.b1, fr.b2, fr.d_in, fr.d_out);
    const Extent extent = extent_of(h, w);
    const float2* __restrict__ d_in = fr.d_in;
    float2* __restrict__ d_out = fr.d_out;
    constexpr int TX = kTileX, NT = kTileThreads, RX = TX + 2 * kWinR, RY = TY + 2 * kWinR;
    constexpr int P = (RX + 3) / 4 * 4;              // row stride: the row pass reads sixteen bytes at a time
    // With the coarser flow a block takes 40 900 bytes: still four per compute unit.
    constexpr int CX = RX / 2 + 1, CY = RY / 2 + 1;
    static_assert(kWinR % 2 == 1 && TX % 2 == 0 && TY % 2 == 0, "the region starts at an odd and ends at an even coordinate");
    __shared__ __align__(16) float s_in[5][RY * P];
    __shared__ typename std::conditional<kFirst, CoarsePatch<CX, CY>, NoRide>::type s_coarse;
    __shared__ float s_w[kFirTable];
    const int tid = threadIdx.x, wave0 = tid & ~63;
    const int x0 = blk.x * TX, y0 = blk.y * TY;
    fir_table(s_w, fw);
    if constexpr (kFirst) {
        if (prior_mode == 1) {
            load_coarse<NT>(s_coarse, d_in, y0 - kWinR, x0 - kWinR, ch, cw);
            __syncthreads();
        }
    }
    // priors of N pixels of a column, rows row_of(0 .. N - 1), all asked for before the first is used
    auto priors = [&](int px, auto row_of, auto& prior) {
        constexpr int N = sizeof(prior) / sizeof(float2);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if constexpr (!kFirst) prior[k] = ld_at(d_in, pix(row_of(k), w, px));
            else if (prior_mode == 0) prior[k] = make_float2(0.0f, 0.0f);
            else prior[k] = transfer_from(s_coarse, y0 - kWinR, x0 - kWinR, row_of(k), px, ch, cw);
        }
    };
    {
        // per-cell terms at the clamped coordinate of the cell: a thread stays in its column (of 504 threads, twelve
        // rows at a time), so that only the row's coordinate changes
        constexpr int kRows = NT / RX, kSteps = (RY + kRows - 1) / kRows;
        const int rx = tid % RX, r0 = tid / RX;
        const int gx = clampi(x0 - kWinR + rx, 0, w - 1);
        if (r0 < kRows) {
            float2 prior[kSteps];
            priors(gx, [&](int k) { return clampi(y0 - kWinR + min(r0 + k * kRows, RY - 1), 0, h - 1); }, prior);
#pragma unroll
            for (int k = 0; k < kSteps; ++k) {
                const int ry = r0 + k * kRows;
                if (k == kSteps - 1 && ry >= RY) continue;
                const int gy = clampi(y0 - kWinR + ry, 0, h - 1);
                __builtin_amdgcn_sched_barrier(0);      // cell by cell: two interleaved need more registers than there are
                float t[5];
                flow_terms(old_cell(fr.A1, fr.b1, pix(gy, w, gx)), fr.A2, fr.b2, extent, gy, gx, prior[k], t);
#pragma unroll
                for (int c = 0; c < 5; ++c) s_in[c][ry * P + rx] = t[c];
            }
        }
    }
    __syncthreads();
    const FirWeights wt = fir_weights(s_w);
    // the priors of the four pixels the thread solves for, asked for again (they are in the cache) ahead of the row pass
    constexpr int kSolve = TX * (TY / kFirOut);      // items of the column pass: whole waves
    static_assert(kSolve <= NT && kSolve % 64 == 0, "one column item per thread, in whole waves");
    const int tx = tid % TX, ty = kFirOut * (tid / TX);
    const int gx = x0 + tx;
    float2 dp[kFirOut];
    if (wave0 < kSolve) {
        priors(min(gx, w - 1), [&](int i) { return min(y0 + ty + i, h - 1); }, dp);
    }
    {
        // Row pass, in place: the sums stay in registers until all of the block's taps are read.  A second array
        // would cost a quarter of the blocks per compute unit.
        constexpr int kItems = RY * (TX / kFirOut);
        static_assert(kItems <= NT, "one row item per thread");
        const int item = min(tid, kItems - 1);
        const int at = (item / (TX / kFirOut)) * P + kFirOut * (item % (TX / kFirOut));
        f32x4 r[5];
        if (wave0 < kItems) {
#pragma unroll
            for (int c = 0; c < 5; ++c) r[c] = fir4_row(wt, &s_in[c][at]);
        }
        __syncthreads();
        if (tid < kItems) {
#pragma unroll
            for (int c = 0; c < 5; ++c) *reinterpret_cast<f32x4*>(&s_in[c][at]) = r[c];
        }
        __syncthreads();
    }
    if (wave0 >= kSolve) return;
    f32x4 acc[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) acc[c] = fir4_column(wt, &s_in[c][ty * P + tx], P);
#pragma unroll
    for (int i = 0; i < kFirOut; ++i) {
        const int gy = y0 + ty + i;
        if (gy < h && gx < w)
            *reinterpret_cast<float2*>(reinterpret_cast<char*>(d_out) + pix(gy, w, gx) * 8u) =
                flow_solve(acc[0][i], acc[1][i], acc[2][i], acc[3][i], acc[4][i], dp[i]);
    }
}

// ---------------------------------------------------------------------------------------------
// Three updates of a level in one launch.  An update of a pixel needs the terms, hence the priors, of the
// pixels within five of it, so a block that makes a TX x TY tile of the third update makes 10 more rows and
// columns of the second and 20 more of the first (the warped samples come from memory wherever they lie).
// That is several times the work per pixel of a launch per update, and it pays where a level is so
// small that its blocks, one per compute unit, leave the chip idle and an update is a chain of
// launch, trips to memory and window passes: 84x84 18.1 -> 11.5 us for three updates (tile 16x8), 168x168
// 18.0 -> 12.4, two frames of it 18.1 -> 14.9 (16x16), 336x336 19.2 -> 17.5 (32x16); now 10.2, 11.2
// and 17.2 (arguments in one trip, coarser flow in LDS, row passes on the matrix cores).  With more than one
// block per compute unit it loses (168x168 x 4: 21.5 against 27).  All of that on an idle chip, one launch after
// the other; next to kernels that fill the wave slots a block of 1024 threads waits longer for room than the three
// launches take.  The results are the same bits (tests/test_gpu_step.py: calls of one to sixteen frames, whose levels take other
// kernels).
// Cells outside the image stand for the clamped coordinate, as in k_flow_tile.
constexpr int kFusedUpdates = 3;
constexpr int kFusedThreads = 1024;

template <int TX, int TY>
struct FusedTile {
    static constexpr int SX = TX + 10 * kFusedUpdates, SY = TY + 10 * kFusedUpdates;      // the first update's terms
    static constexpr int PX = SX - 10, PY = SY - 10;                                      // the first update's results
    static constexpr int SP = (SX + 3) / 4 * 4, kFloats = 5 * SY * SP;
    alignas(16) float in[kFloats];
    float2 p[SY * SX];          // priors of the first update, then of the third
    float2 q[PY * PX];          // priors of the second update
    CoarsePatch<SX / 2 + 1, SY / 2 + 1> coarse;
    float w[kFirTable];
};

// Update I of the block: terms of its region plus five cells all round, window passes, solve; the priors
// (region of the terms, row-major) come from `prior`, the results go to `next` or, the last ones, to d_out.
// The row pass runs on the matrix cores, as in k_flow_tile, over quads of outputs of one field, dealt to all waves: 1.5 -> 1.2, 0.92 ->
// 0.76 and 0.56 -> 0.32 us of a 168x168 level's three updates.  The column pass stays on the vector ALU, two outputs an item: on the
// matrix cores, five fields and four outputs a lane, it is a chain of 70 products and four solves on a quarter of the waves (0.6 -> 0.84 us
// of the last update).  A region that is no multiple of four has outputs past its end, which nothing uses, and the zero weights of its
// last outputs meet cells past its end.  Those must be finite: terms of other cells or of an earlier update, or the padding of the first update's rows, which is cleared.
template <int TX, int TY, int I>
__device__ __forceinline__ void fused_update(FusedTile<TX, TY>& sh, float2* prior, float2* next, const FlowFrame& f,
                                             const Extent& extent, int ch, int cw, int prior_mode, int x0, int y0, FirWeights& wt, const FlowWeights& fw) {
    constexpr int kLeft = kFusedUpdates - 1 - I, NT = kFusedThreads;
    constexpr int DX = TX + 10 * kLeft, DY = TY + 10 * kLeft, RX = DX + 10, RY = DY + 10;
    constexpr int P = (RX + 3) / 4 * 4;             // row stride: the row pass reads sixteen bytes at a time
    const int tid = threadIdx.x, wave0 = tid & ~63;
    const int ox = x0 - 5 * (kLeft + 1), oy = y0 - 5 * (kLeft + 1), h = extent.h, w = extent.w;
    if constexpr (I == 0) {
        static_assert(5 * kFusedUpdates % 2 == 1 && TX % 2 == 0 && TY % 2 == 0, "the region starts at an odd and ends at an even coordinate");
        if (prior_mode == 1) {
            load_coarse<NT>(sh.coarse, f.d_in, oy, ox, ch, cw);
            __syncthreads();
        }
    }
    {
        // a thread stays in its column, kRows rows at a time, and asks for all that does not depend on the prior first, then
        // for the priors of all its cells
        constexpr int kRows = NT / RX, kSteps = (RY + kRows - 1) / kRows;
        const int rx = tid % RX, r0 = tid / RX;
        const int gx = clampi(ox + rx, 0, w - 1);
        if (r0 < kRows) {
            OldCell old[kSteps];
            float2 dp[kSteps];
#pragma unroll
            for (int k = 0; k < kSteps; ++k)
                old[k] = old_cell(f.A1, f.b1, pix(clampi(oy + min(r0 + k * kRows, RY - 1), 0, h - 1), w, gx));
            auto row = [&](int k) { return clampi(oy + min(r0 + k * kRows, RY - 1), 0, h - 1); };
#pragma unroll
            for (int k = 0; k < kSteps; ++k) {
                if constexpr (I > 0) dp[k] = prior[(row(k) - oy) * RX + (gx - ox)];     // in the region: the tile meets the image
                else if (prior_mode == 0) dp[k] = make_float2(0.0f, 0.0f);
                else if (prior_mode == 1) dp[k] = transfer_from(sh.coarse, oy, ox, row(k), gx, ch, cw);
                else dp[k] = ld_at(f.d_in, pix(row(k), w, gx));
            }
#pragma unroll
            for (int k = 0; k < kSteps; ++k) {
                const int ry = r0 + k * kRows;
                if (k == kSteps - 1 && ry >= RY) continue;
                if constexpr (I == 0) prior[ry * RX + rx] = dp[k];
                float t[5];
                flow_terms(old[k], f.A2, f.b2, extent, clampi(oy + ry, 0, h - 1), gx, dp[k], t);
#pragma unroll
                for (int c = 0; c < 5; ++c) sh.in[(c * RY + ry) * P + rx] = t[c];
            }
        }
    }
    __syncthreads();
    if constexpr (I == 0) wt = fir_weights(sh.w);
    {
        // Row pass in place, as in k_flow_tile, an item four outputs of one field: the rows of the five fields follow one another.
        constexpr int kQuads = (DX + 3) / 4, kItems = 5 * RY * kQuads, kN = (kItems + NT - 1) / NT;
        static_assert((5 * RY - 1) * P + 4 * (kQuads - 1) + 16 <= FusedTile<TX, TY>::kFloats, "reads end inside the array");
        f32x4 r[kN];
        auto rows = [&](auto count) {
            float v[count()][16];
#pragma unroll
            for (int n = 0; n < count(); ++n) {
                const int item = min(tid + n * NT, kItems - 1);
                const float* p = &sh.in[(item / kQuads) * P + 4 * (item % kQuads)];
#pragma unroll
                for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(v[n] + 4 * i) = *reinterpret_cast<const f32x4*>(p + 4 * i);
            }
            fir4_abreast<count()>(wt, v, r);
        };
        // whole waves have either all of their kN items or all but the last
        if (wave0 + (kN - 1) * NT < kItems) rows(std::integral_constant<int, kN>{});
        else if constexpr (kN > 1) rows(std::integral_constant<int, kN - 1>{});
        __syncthreads();
#pragma unroll
        for (int n = 0; n < kN; ++n) {
            const int item = tid + n * NT;
            if (item < kItems) *reinterpret_cast<f32x4*>(&sh.in[(item / kQuads) * P + 4 * (item % kQuads)]) = r[n];
        }
        __syncthreads();
    }
    // Column pass, two outputs an item: twelve reads a field for two outputs
    static_assert(DY % 2 == 0, "pairs");
    for (int p = tid; p < (DY / 2) * DX; p += NT) {
        const int ty0 = 2 * (p / DX), tx = p % DX;
        float acc[5][2];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            float v[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) v[k] = sh.in[(c * RY + ty0 + k) * P + tx];
            acc[c][0] = acc[c][1] = 0.0f;
#pragma unroll
            for (int k = 0; k <= 2 * kWinR; ++k) {
                acc[c][0] += fw.win_g[k] * v[k];
                acc[c][1] += fw.win_g[k] * v[k + 1];
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int ty = ty0 + j;
            const float2 d = flow_solve(acc[0][j], acc[1][j], acc[2][j], acc[3][j], acc[4][j], prior[(ty + kWinR) * RX + tx + kWinR]);
            if constexpr (kLeft == 0) {
                const int gy = y0 + ty, gx = x0 + tx;
                if (gy < h && gx < w) *reinterpret_cast<float2*>(reinterpret_cast<char*>(f.d_out) + pix(gy, w, gx) * 8u) = d;
            } else {
                next[ty * DX + tx] = d;
            }
        }
    }
    if constexpr (kLeft > 0) __syncthreads();
}

// Riders of a launch, its blocks after the flow's: a tile of the pre-pass per block, a border pixel per thread, or a patch per
// wave.  At 336x336 the flow leaves room for them: its own blocks are at most one per compute unit.
namespace {
template <typename Shared>
__device__ __forceinline__ void ride_flow(Shared& sh, const PrepRide& r, int block) {
    const int tiles = r.tiles_x * r.tiles_y, b = block / tiles, t = block - b * tiles;
    prep_tile<false, kFusedThreads>(sh.prep, r.f, t % r.tiles_x, t / r.tiles_x, b, r.h, r.w, GateParams{}, r.lut, r.lo2, r.hi2);
}
template <typename Shared>
__device__ __forceinline__ void ride_flow(Shared&, const UnionRide& r, int block) {
    const int b = block / r.blocks_per_frame;
    union_item(r.f.frame[b], r.h, r.w, (block - b * r.blocks_per_frame) * kFusedThreads + (int)threadIdx.x, r.n_items, [] { return false; });
}
template <typename Shared>
__device__ __forceinline__ void ride_flow(Shared&, const ScoreRide& r, int block) {
    const int b = block / r.blocks_per_frame;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (int token = (block - b * r.blocks_per_frame) * (kFusedThreads / 64) + wave; token < kTokens;
         token += r.blocks_per_frame * (kFusedThreads / 64))
        score_by_wave(r.f.frame[b], token, r.h, r.w, nullptr, [] { return false; });
}
// LDS: the pre-pass needs some of its own, the other riders none
template <typename Own, typename Ride>
struct FlowShared : WithPrep<Own, NoRide> {};
template <typename Own>
struct FlowShared<Own, PrepRide> : WithPrep<Own, PrepRide> {};
}  // namespace

// tiles_x x tiles_y tiles of n frames: the grid, or the first blocks of a one-dimensional grid that ends with the riders
template <int TX, int TY, typename Ride>
__global__ __launch_bounds__(kFusedThreads) void k_flow_fused(int tiles_x, int tiles_y, int n, int h, int w, int ch, int cw, int prior_mode,
                                                              FlowWeights fw, FlowBatch f, Ride ride) {
    __shared__ FlowShared<FusedTile<TX, TY>, Ride> lds;
    BlockId blk;
    if constexpr (std::is_same_v<Ride, NoRide>) {
        blk = xcd_block_id(tiles_x, tiles_y, n);
    } else {
        const int own = tiles_x * tiles_y * n;
        if ((int)blockIdx.x >= own) {
            ride_flow(lds, ride, (int)blockIdx.x - own);
            return;
        }
        blk = xcd_block_id((int)blockIdx.x, tiles_x, tiles_y, n);
    }
    const FlowFrame fr = f.frame[blk.z];
    together(fr.A1, fr.A2, fr.b1, fr.b2, fr.d_in, fr.d_out);
    const Extent extent = extent_of(h, w);
    FusedTile<TX, TY>& sh = lds.own;
    const int x0 = blk.x * TX, y0 = blk.y * TY;
    fir_table(sh.w, fw);
    constexpr int kPad = FusedTile<TX, TY>::SP - FusedTile<TX, TY>::SX;
    if constexpr (kPad > 0) {
        for (int p = threadIdx.x; p < 5 * FusedTile<TX, TY>::SY * kPad; p += kFusedThreads)
            sh.in[(p / kPad + 1) * FusedTile<TX, TY>::SP - 1 - p % kPad] = 0.0f;
    }
    FirWeights wt;
    fused_update<TX, TY, 0>(sh, sh.p, sh.q, fr, extent, ch, cw, prior_mode, x0, y0, wt, fw);
    fused_update<TX, TY, 1>(sh, sh.q, sh.p, fr, extent, ch, cw, prior_mode, x0, y0, wt, fw);
    fused_update<TX, TY, 2>(sh, sh.p, sh.q, fr, extent, ch, cw, prior_mode, x0, y0, wt, fw);
}

// ---------------------------------------------------------------------------------------------
// Eq. 5 of the stand-alone flow call: each patch's motion, and the flow field in the caller's layout (two
// planes).  kWaves = 1: one wave per patch, four patches per block; kWaves = 4: the block works on one patch
// (large frames).  Four pixels a lane are asked for together: the loop is bound by trips to memory; without
// divisions by the patch's width (PatchPixels) 1920x1080 takes 8.0 us, 9.6 before.
template <int kWaves>
__global__ __launch_bounds__(256) void k_patch_motion(const float2* __restrict__ flow, int h, int w, float* __restrict__ dp_out,
                                                      float* __restrict__ flow_uv) {
    __shared__ float s_sum[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int token = kWaves == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
    const PatchBox box = patch_box(token, h, w);
    const PatchPixels pixel(box, w);
    constexpr int kStride = 64 * kWaves, kUnroll = 4;
    float acc = 0.0f;
    for (int p0 = (kWaves == 1 ? lane : (int)threadIdx.x); p0 < box.area; p0 += kStride * kUnroll) {
        uint32_t gi[kUnroll];
        float2 d[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            gi[u] = pixel(min(p0 + u * kStride, box.area - 1));
            d[u] = ld_at(flow, gi[u]);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (p0 + u * kStride >= box.area) continue;
            acc += d[u].x * d[u].x + d[u].y * d[u].y;
            if (flow_uv != nullptr) {
                flow_uv[gi[u]] = d[u].x;
                flow_uv[(size_t)h * w + gi[u]] = d[u].y;
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off);
    if (kWaves == 4) {
        if (lane == 0) s_sum[wave] = acc;
        __syncthreads();
        acc = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
    }
    if (lane == 0 && (kWaves == 1 || wave == 0)) dp_out[token] = sqrtf(acc / (float)box.area);
}

// Eq. 6, one block.  A launch of its own: as the work of the last block to finish it needed a device-scope
// fence in every block, and with the pixels of a patch taken one at a time the call's last kernel took
// 14.3 us (with its neighbours' tails) at 336x336 and 33 us at 1920x1080; motion and gate now take 3.3 and 9.4 us
// plus 2 to 4 for the gate.
__global__ __launch_bounds__(256) void k_gate(const float* __restrict__ dp, float tau_t, float theta_r, sali_gate* gate) {
    __shared__ int s_cnt[4];
    int n = 0;
    for (int i = threadIdx.x; i < kTokens; i += 256) n += dp[i] < tau_t ? 1 : 0;
    for (int off = 32; off > 0; off >>= 1) n += __shfl_down(n, off);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int n_static = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        const float r = (float)n_static / (float)kTokens;
        sali_gate gt;
        gt.n_static = n_static;
        gt.r_frame = r;
        gt.redundant = (r > theta_r) ? 1 : 0;
        gt.reserved = 0;
        *gate = gt;
    }
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_pyramid(const PyrBatch& f, int n, const LevelGeom& g, hipStream_t s) {
    for (int lvl = 1; lvl < g.levels; lvl += 2) {
        const dim3 grid((g.w[lvl] + kPyrT - 1) / kPyrT, (g.h[lvl] + kPyrT - 1) / kPyrT, n);
        const int sharing = frames_sharing_runs((int)grid.x, (int)grid.y, n);
        if (lvl == 1) hipLaunchKernelGGL(k_pyr_pair<true>, grid, dim3(256), 0, s, (int)grid.x, (int)grid.y, sharing, lvl, g, f);
        else hipLaunchKernelGGL(k_pyr_pair<false>, grid, dim3(256), 0, s, (int)grid.x, (int)grid.y, sharing, lvl, g, f);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_polyexp(const PyrBatch& f, int n, LevelGeom g, FlowWeights fw, const PrepRide* ride_or_null, hipEvent_t done_or_null,
                          hipStream_t s) {
    const int per_frame = g.tile_start[g.levels];
    if (ride_or_null != nullptr)
        launch_recording(done_or_null, k_polyexp<PrepRide>, dim3(ride_or_null->blocks + per_frame * n), dim3(256), s, ride_or_null->blocks,
                         per_frame, g, fw, f, *ride_or_null);
    else
        launch_recording(done_or_null, k_polyexp<NoRide>, dim3(per_frame, n), dim3(256), s, 0, per_frame, g, fw, f, NoRide{});
    return hipGetLastError();
}

hipError_t launch_expand(const ExpandBatch& f, int n, LevelGeom g, FlowWeights fw, const PrepRide* ride_or_null, hipEvent_t done_or_null,
                         hipStream_t s) {
    // up to three levels, 16x16 tiles, one launch
    int tx[3] = {1, 1, 1}, tiles[3] = {0, 0, 0};
    for (int l = 0; l < 3 && l < g.levels; ++l) {
        tx[l] = (g.w[l] + kET - 1) / kET;
        tiles[l] = tx[l] * ((g.h[l] + kET - 1) / kET);
    }
    const int per_frame = tiles[2] + (tiles[1] + 1) / 2 + (tiles[0] + 1) / 2;
    if (ride_or_null != nullptr)
        launch_recording(done_or_null, k_expand<PrepRide>, dim3(ride_or_null->blocks + per_frame * n), dim3(kExpandThreads), s,
                         ride_or_null->blocks, n, tiles[0], tiles[1], tiles[2], tx[0], tx[1], tx[2], g, fw, f, *ride_or_null);
    else
        launch_recording(done_or_null, k_expand<NoRide>, dim3(per_frame, n), dim3(kExpandThreads), s, 0, n, tiles[0], tiles[1], tiles[2], tx[0],
                         tx[1], tx[2], g, fw, f, NoRide{});
    return hipGetLastError();
}

namespace {

constexpr int kComputeUnits = 256;

long long tiles_of(int tx, int ty, int n, int h, int w) { return (long long)((w + tx - 1) / tx) * ((h + ty - 1) / ty) * n; }

// Tile of the launch that makes three updates of a level at once: the smallest whose blocks fit one per compute unit.
// Also for batches: of 100 clips with the image side next to K/V kernels three, of two frames a call, are 3 to 5 %
// slower than with single frames fused only, small frames up to 26 % faster, the median 1 % faster.
enum class Fused { no, t16x8, t16x16, t32x16 };
Fused fused_tile(int n, int h, int w, int wanted) {
    if (wanted < kFusedUpdates) return Fused::no;
    if (tiles_of(16, 8, n, h, w) <= kComputeUnits) return Fused::t16x8;
    if (tiles_of(16, 16, n, h, w) <= kComputeUnits) return Fused::t16x16;
    return tiles_of(32, 16, n, h, w) <= kComputeUnits ? Fused::t32x16 : Fused::no;
}

// Blocks per frame that a piece of the spatial filter gets beside `own` blocks of the flow's, 0: no room.  The flow's blocks fit
// a compute unit each, by registers or LDS, and take 10 us and more; the riders get the other units, all at once.  A tile of
// the pre-pass (one per block) takes 10 us, a block of border pixels 5, a patch of a wave's 5: up to three per wave.
// (In two rounds of blocks, 36 a frame on 25 units, the scores made the flow's launch at 336x336 5 us longer.)
int rider_blocks(FlowRider rider, const FlowRiders& r, long long own) {
    const long long room = own < kComputeUnits ? (kComputeUnits - own) / r.n : 0;
    constexpr int kAll = kTokens / (kFusedThreads / 64);
    if (rider == FlowRider::scores) return room >= kAll ? kAll : (room >= kAll / 3 ? (int)room : 0);
    const int want = rider == FlowRider::prepass ? r.prep->tiles_x * r.prep->tiles_y
                                                 : (border_items(r.h, r.w) + kFusedThreads - 1) / kFusedThreads;
    return want <= room ? want : 0;
}

template <int TX, int TY>
hipError_t launch_fused(const FlowBatch& f, int n, int h, int w, int ch, int cw, int prior_mode, const FlowWeights& fw, FlowRider rider,
                        const FlowRiders* r, hipStream_t s) {
    const int gx = (w + TX - 1) / TX, gy = (h + TY - 1) / TY, own = gx * gy * n;
    auto go = [&](const auto& ride, dim3 grid) {
        hipLaunchKernelGGL((k_flow_fused<TX, TY, std::decay_t<decltype(ride)>>), grid, dim3(kFusedThreads), 0, s, gx, gy, n, h, w, ch, cw,
                           prior_mode, fw, f, ride);
        return hipGetLastError();
    };
    if (rider == FlowRider::none) return go(NoRide{}, dim3(gx, gy, n));
    const int per = rider_blocks(rider, *r, own), blocks = per * r->n;
    if (rider == FlowRider::prepass) return go(*r->prep, dim3(own + blocks));
    if (rider == FlowRider::hysteresis) return go(UnionRide{blocks, r->h, r->w, border_items(r->h, r->w), per, r->prep->f}, dim3(own + blocks));
    return go(ScoreRide{blocks, r->h, r->w, per, *r->pool}, dim3(own + blocks));
}

}  // namespace

bool flow_launch_carries(FlowRider rider, const FlowRiders& riders, int n, int h, int w, int wanted) {
    long long own = 0;
    switch (fused_tile(n, h, w, wanted)) {
        case Fused::no: return false;
        case Fused::t16x8: own = tiles_of(16, 8, n, h, w); break;
        case Fused::t16x16: own = tiles_of(16, 16, n, h, w); break;
        case Fused::t32x16: own = tiles_of(32, 16, n, h, w); break;
    }
    return rider_blocks(rider, riders, own) > 0;
}

hipError_t launch_flow_updates(const FlowBatch& level0, int n, int64_t level_off, int h, int w, int ch, int cw,
                               int prior_mode, int wanted, int* done, const FlowWeights& fw, FlowRider rider, const FlowRiders* riders,
                               hipStream_t s) {
    FlowBatch f = {};
    for (int i = 0; i < n; ++i) {
        f.frame[i] = level0.frame[i];
        f.frame[i].A1 += level_off;
        f.frame[i].A2 += level_off;
        f.frame[i].b1 += level_off;
        f.frame[i].b2 += level_off;
    }
    *done = kFusedUpdates;
    switch (fused_tile(n, h, w, wanted)) {
        case Fused::no: break;
        case Fused::t16x8: return launch_fused<16, 8>(f, n, h, w, ch, cw, prior_mode, fw, rider, riders, s);
        case Fused::t16x16: return launch_fused<16, 16>(f, n, h, w, ch, cw, prior_mode, fw, rider, riders, s);
        case Fused::t32x16: return launch_fused<32, 16>(f, n, h, w, ch, cw, prior_mode, fw, rider, riders, s);
    }
    *done = 1;
#define SALI_FLOW_LAUNCH(KERNEL, TX, TY, NT)                                                                              \
    hipLaunchKernelGGL(KERNEL, dim3((w + TX - 1) / TX, (h + TY - 1) / TY, n), dim3(NT), 0, s, (w + TX - 1) / TX, (h + TY - 1) / TY, \
                       frames_sharing_runs((w + TX - 1) / TX, (h + TY - 1) / TY, n), h, w, ch, cw, prior_mode, fw, f)
    // The shape whose rounds of blocks cost least.  A round is a block per compute unit; launches of 1, 2, 3 .. rounds
    // measured over thirteen frame sizes and their halves (42x42 to 1920x1080, one to fifteen frames, an idle chip, in us) lie on a line each, the
    // first update of a level and the others:
    //   32x32 tiles   8.5  11.7  14.6  17.9 .. 30 (eight)    6.7  10.1  12.3  15.9 .. 27        least work per pixel: 1.7 cells
    //   32x16 tiles   7.0   9.6  11.6  13.5                  5.9   7.8   9.6  11.4              2.1 cells
    //   16x16 tiles   6.6   7.3   8.3  10.2  12.1            5.5   6.3   7.5   8.8   9.6        2.6 cells, the shortest block
    // The costs below are lines through both (as they were before the coarser flow was staged in LDS).  Of 288 launches they choose a shape that is
    // more than 3 % slower than the best for 24, at most 22 % (first update of 84x84 x 15 frames 9.9 us, in 16x16 tiles 8.1).
    auto rounds = [&](int tx, int ty) { return (tiles_of(tx, ty, n, h, w) + kComputeUnits - 1) / kComputeUnits; };
    const long long cost32 = 93 + 60 * rounds(kTileX, 32), cost16 = 95 + 36 * rounds(kTileX, 16),
                    cost_small = 94 + 22 * rounds(kSmallTile, kSmallTile);             // twentieths of a us
    if (cost_small <= cost16 && cost_small <= cost32) SALI_FLOW_LAUNCH(k_flow_small, kSmallTile, kSmallTile, kSmallThreads);
    else if (cost16 <= cost32 && prior_mode != 2) SALI_FLOW_LAUNCH((k_flow_tile<16, true>), kTileX, 16, kTileThreads);
    else if (cost16 <= cost32) SALI_FLOW_LAUNCH((k_flow_tile<16, false>), kTileX, 16, kTileThreads);
    else if (prior_mode != 2) SALI_FLOW_LAUNCH((k_flow_tile<32, true>), kTileX, 32, kTileThreads);
    else SALI_FLOW_LAUNCH((k_flow_tile<32, false>), kTileX, 32, kTileThreads);
#undef SALI_FLOW_LAUNCH
    return hipGetLastError();
}

hipError_t launch_patch_gate(const float2* d_flow, int h, int w, float tau_t, float theta_r, float* d_dp,
                             sali_gate* d_gate, float* d_flow_uv_or_null, hipStream_t s) {
    // a wave per patch of up to 256 pixels (one trip of four loads a lane), the block beyond
    if ((long long)h * w <= 256ll * kTokens)
        hipLaunchKernelGGL(k_patch_motion<1>, dim3(kTokens / 4), dim3(256), 0, s, d_flow, h, w, d_dp, d_flow_uv_or_null);
    else
        hipLaunchKernelGGL(k_patch_motion<4>, dim3(kTokens), dim3(256), 0, s, d_flow, h, w, d_dp, d_flow_uv_or_null);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gate, dim3(1), dim3(256), 0, s, d_dp, tau_t, theta_r, d_gate);
    return hipGetLastError();
}

}  // namespace sali
