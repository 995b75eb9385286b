// Slots of a bucket: workgroups take runs of them by adding their counts to
// the bucket's 32-bit fill counter.  Plain C++ (constexpr, so usable in device
// code too): the rule is tested on the host.  Not installed.
#pragma once

#include <stdint.h>

namespace spv {

// Whether a run of n slots fits a bucket of cap slots of which `taken` were
// taken before it.  The counter is read as unsigned, and nothing is added to
// it here: base + taken + n in 32 bits goes negative, and passes a test against
// the bucket's end, once repeated x indices have brought the counter past 2^31.
constexpr bool slots_fit(int32_t taken, int32_t n, int32_t cap) {
    return (uint32_t)taken <= (uint32_t)cap && (uint32_t)n <= (uint32_t)cap - (uint32_t)taken;
}

// What keeps the counter itself from wrapping.  The scatter adds at most W <=
// nnz products.  The expansion has no count of all products; there a workgroup
// stops at the first chunk with a run that does not fit, so past a bucket's
// slots (at most INT32_MAX) every workgroup adds one chunk at most.
constexpr int kExpandMaxGrid = 4096;    // workgroups
constexpr int kExpandMaxChunk = 8192;   // products
static_assert((uint64_t)INT32_MAX + (uint64_t)kExpandMaxGrid * kExpandMaxChunk <= UINT32_MAX, "fill counters wrap");

}  // namespace spv
