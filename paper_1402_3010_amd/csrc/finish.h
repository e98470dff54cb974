// Launcher of the kernel that ends a call with few pairs (finish.hip).
#pragma once

#include "apss_internal.h"

namespace apss {

// Most pairs that one launch sorts and hands over.
constexpr int64_t kFinishPairs = 32768;

struct FinishArgs {
  const uint64_t* key;  // raw pairs of the join kernels, in any order, distinct
  const float* sim;
  int64_t cap;          // raw pairs that the buffers hold
  int bj;               // key = i << bj | j
  int bits;             // keys are below 2^bits
  uint32_t* out_i;      // room entries each (device or pinned host memory)
  uint32_t* out_j;
  float* out_sim;
  int64_t room;
  const unsigned long long* counters;  // [C_NUM]
  const unsigned long long* checks;    // [2] error bits and first bad row of the call's rows, or NULL
  unsigned long long* host;            // [C_NUM + 2] pinned host copy of the counters and the checks
};

// The counters (and 0, 0 for checks that there are not) to the host; and, if there are at most kFinishPairs, cap and
// room pairs and no check has failed, the pairs in order of (i, j) to out_*.
hipError_t launch_finish(const FinishArgs& a, hipStream_t s);
// True when launch_finish delivered a join's pairs.
inline bool finish_delivers(int64_t matches, int64_t cap, int64_t room) {
  return matches <= kFinishPairs && matches <= cap && matches <= room;
}

}  // namespace apss
