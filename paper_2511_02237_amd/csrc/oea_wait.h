// Budget of a bounded wait: how often data that other workgroups produce may be asked for again.
#pragma once
#include <stdint.h>

namespace oea {

// One budget serves everything a wavefront waits for in a row, so that several waits together take no longer
// than one, and once it is used up every further wait gives up at its first look.
struct WaitBudget {
  uint32_t left;
  // to be asked when a look has found something missing: true if there may be another one
  __host__ __device__ bool again() {
    if (left == 0) return false;
    --left;
    return true;
  }
};

}  // namespace oea
