// Internal declarations shared by the host-side entry points of libpolarquant.
// Nothing here is part of the public ABI (that is include/polarquant.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pq_plan.hpp"

namespace pq {

// Remembers the hipError_t of a failed call for pq_last_hip_error().
int record_hip_error(hipError_t e);

// True when this build has kernels for the layout.
bool layout_supported(const pq_layout* l);

// An encoder's work-groups (256 threads) are one a (token group, KV head) in a one-dimensional grid, which HIP limits to
// 2^32 - 1 threads: launch(first group, groups) is called for as many ranges of token groups as that takes.
template <typename F>
hipError_t for_group_ranges(int64_t n_groups, int32_t n_kv_heads, F launch) {
  const int64_t most = ((int64_t{1} << 24) - 1) / n_kv_heads;            // 256 and more: n_kv_heads < 2^16
  hipError_t e = hipSuccess;
  for (int64_t first = 0; first < n_groups && e == hipSuccess; first += most)
    e = launch(first, n_groups - first < most ? n_groups - first : most);
  return e;
}

}  // namespace pq
