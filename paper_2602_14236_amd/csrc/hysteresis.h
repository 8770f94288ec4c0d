// Hysteresis of the Canny stage as a lock-free union-find, shared by the saliency kernels
// (Implementation Details: Canny edge detection).
// A pixel's key is its index with bit 31 set for weak pixels; links always point to the smaller
// key, so a walk along links meets a strong key iff the component has one.
#pragma once

#include "sali_internal.h"

namespace sali {

constexpr int kTile = 32;                       // tile side of the saliency pre-pass
constexpr uint32_t kWeakBit = 0x80000000u;

// union-find on a parent array (LDS or global); key = index | weak bit; links go to smaller keys
template <int kScope>
__device__ __forceinline__ uint32_t uf_load(const uint32_t* parent, uint32_t idx) {
    return __hip_atomic_load(parent + idx, __ATOMIC_RELAXED, kScope);
}

// Joins the components of two pixels as far as the classes need it: "has a strong pixel" must reach the weak
// components; two that are strong already are not joined, and a walk ends at the first strong key, whose
// component's root is strong (keys decrease along links and strong keys are the smaller ones).  Both walks
// of a pair go in step: a step is a trip to LDS or, at agent scope, past the L2.
template <int kScope>
__device__ __forceinline__ void uf_spread_strong(uint32_t* parent, uint32_t ka, uint32_t kb) {
    for (;;) {
        uint32_t before_a = ka, before_b = kb;
        for (;;) {
            uint32_t pa = ka, pb = kb;
            if (ka & kWeakBit) pa = uf_load<kScope>(parent, ka & ~kWeakBit);
            if (kb & kWeakBit) pb = uf_load<kScope>(parent, kb & ~kWeakBit);
            if (pa == ka && pb == kb) break;        // two roots or strong keys
            if constexpr (kScope == __HIP_MEMORY_SCOPE_WORKGROUP) {
                // in LDS a passed node is linked on to its grandparent on the way, which keeps the paths short
                if (pa != ka && before_a != ka) atomicMin(parent + (before_a & ~kWeakBit), pa);
                if (pb != kb && before_b != kb) atomicMin(parent + (before_b & ~kWeakBit), pb);
                before_a = ka;
                before_b = kb;
            }
            ka = pa;
            kb = pb;
        }
        if (ka == kb || ((ka | kb) & kWeakBit) == 0u) return;
        if (ka < kb) { const uint32_t t = ka; ka = kb; kb = t; }      // ka is the larger key: a weak root
        const uint32_t old = atomicMin(parent + (ka & ~kWeakBit), kb);
        if (old == ka) return;      // ka was a root and now points at kb
        ka = old;                   // somebody linked ka first: join where it pointed with kb (the smaller is ka's link)
    }
}

// Pixels that have neighbours across a border of the pre-pass's tiles (pairs inside a tile were joined in LDS
// there): first the last rows of all tile rows but the lowest, pixel by pixel, then the last columns of all
// tile columns but the rightmost.  Each looks at the three pixels across;
// where runs of candidates touch along the border the contact is made once, by the first pair.
__host__ __device__ inline int border_rows(int h, int w) { return ((h - 1) / kTile) * w; }
__host__ __device__ inline int border_items(int h, int w) { return border_rows(h, w) + ((w - 1) / kTile) * h; }

// (`there`: the item exists; stop(), uniform: asked once the classes are under way, true leaves everything as it is)
template <typename Stop>
__device__ __forceinline__ void union_border(const uint8_t* __restrict__ cls, uint32_t* parent, int h, int w, int item, bool there, Stop stop) {
    const int n_rows = border_rows(h, w);
    const bool row = item < n_rows;
    const int i = row ? item : item - n_rows, len = row ? w : h;
    const int k = i / len, at = i - k * len;                        // border k, place along it
    const int x = row ? at : kTile * k + kTile - 1, y = row ? kTile * k + kTile - 1 : at;
    const int gi = y * w + x, across = row ? w : 1, along = row ? 1 : w;
    // c[0][1] = this pixel, c[0][0] / c[0][2] = the ones beside it along the border, c[1][] = across
    int c[2][3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const bool in = at + j >= 1 && at + j <= len;
        c[0][j] = in ? cls[gi + (j - 1) * along] : 0;
        c[1][j] = in ? cls[gi + across + (j - 1) * along] : 0;
    }
    if (stop() || !there || c[0][1] == 0) return;
    const uint32_t me = (uint32_t)gi | (c[0][1] == 1 ? kWeakBit : 0u);
    // Straight across, unless the pair before makes that contact: it lies in the same two tiles, whose pixels
    // are joined in LDS (so not for the first pair of a tile: round a corner of four tiles each contact
    // would count on the others).  A diagonal only if neither the pixel straight across nor the one beside this
    // pixel leads there.
    const bool straight = c[1][1] != 0 && !(at % kTile != 0 && c[0][0] != 0 && c[1][0] != 0);
    if (straight) uf_spread_strong<__HIP_MEMORY_SCOPE_AGENT>(parent, me, (uint32_t)(gi + across) | (c[1][1] == 1 ? kWeakBit : 0u));
    if (c[1][1] != 0) return;
#pragma unroll
    for (int j = 0; j < 3; j += 2)
        if (c[1][j] != 0 && c[0][j] == 0)
            uf_spread_strong<__HIP_MEMORY_SCOPE_AGENT>(parent, me, (uint32_t)(gi + across + (j - 1) * along) | (c[1][j] == 1 ? kWeakBit : 0u));
}

}  // namespace sali
