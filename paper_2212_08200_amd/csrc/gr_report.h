// Counters that the host polls (declarations; see gr_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace gr {

// Copies a counter slot to `to` (pinned host memory, the slot's layout), then
// stores tag in to[kSlotWords].
hipError_t launch_report(const unsigned long long *slot, unsigned long long *to, unsigned long long tag, hipStream_t st);

}  // namespace gr
