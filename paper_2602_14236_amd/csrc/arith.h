// Arithmetic of the kernels that the host can run too (tests/test_device_arithmetic.py does).
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define SALI_BOTH __host__ __device__ __forceinline__
#else
#define SALI_BOTH inline
#endif

namespace sali {

constexpr int kAttnPartials = 256;          // partial softmax states per head in the attention kernel

// Hand-over of a head's partials to the last of its `parts` blocks.  Every number of parts has a counter of its own, which wraps to zero at that
// number (atomicInc), so it is at zero whenever as many blocks have arrived as were launched, also after launches that overlapped
// each other against the rules: their results are lost, those of later ones are not.  A head's counters are 1 KB, so that two heads' lie in
// different memory lines: additions to one line are made one after the other wherever they come from, and with the counters of 32
// heads side by side 2000 arrivals took 20 us.
SALI_BOTH size_t arrival_counter(int head_set, int parts) { return (size_t)head_set * kAttnPartials + (size_t)(parts - 1); }
SALI_BOTH bool last_arrival(uint32_t before, int parts) { return before >= (uint32_t)parts - 1u; }

// v / kDiv, correctly rounded, for whole v from 0 to kDiv (255 and 65280: every value checked): the product with the rounded reciprocal,
// corrected by its remainder
template <int kDiv>
SALI_BOTH float whole_over(uint32_t v) {
    constexpr float kInv = 1.0f / kDiv;
    const float x = (float)v, q = x * kInv;
    return __builtin_fmaf(__builtin_fmaf(-(float)kDiv, q, x), kInv, q);
}

// Row of a patch's pixel by a product: exact for numbers below 2^16 and rows of 2 to 2^16 pixels
// (larger patches divide: from 6000 pixels a side on)
struct PatchRow {
    uint32_t width, inverse;
    bool small;
    SALI_BOTH PatchRow(uint32_t pixels_a_row, uint32_t area)
        : width(pixels_a_row), inverse(0xFFFFFFFFu / pixels_a_row + 1u), small(area <= 65536u && pixels_a_row > 1u) {}
    SALI_BOTH uint32_t operator()(uint32_t pixel) const { return small ? (uint32_t)((uint64_t)pixel * inverse >> 32) : pixel / width; }
};

}  // namespace sali
