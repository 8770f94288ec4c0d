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

}  // namespace sali
