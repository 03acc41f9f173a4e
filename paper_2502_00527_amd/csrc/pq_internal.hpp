// Internal declarations shared by the host-side entry points of libpolarquant.
// Nothing here is part of the public ABI (that is include/polarquant.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "polarquant.h"

namespace pq {

constexpr int kHeadDim = 128;          // d
constexpr int kPairs = kHeadDim / 2;   // P: pair j = dims (j, j + 64)
constexpr int kGroup = 128;            // g: tokens per page / quantization group
constexpr int kPairsPerUnit = 16;      // one packed unit = 16 pairs of one token
constexpr int kBlocks = kPairs / kPairsPerUnit;
constexpr int kMaxAngleBins = 32;      // t <= 5

// Remembers the hipError_t of a failed call for pq_last_hip_error().
int record_hip_error(hipError_t e);

// True when this build has kernels for the layout.
bool layout_supported(const pq_layout* l);

// How the context of a sequence is cut into chunks of pages; one work-group
// handles one (sequence, KV head, chunk).  Pure function of the launch shape so
// that the workspace size and both decode stages agree.
struct ChunkPlan {
  int32_t pages_per_chunk;
  int32_t n_chunks;   // per sequence, for max_seq_len
  // chunks from number n_big on are pages_small long (attention kernel of the uniform grid; otherwise
  // n_big is n_chunks)
  int32_t n_big;
  int32_t pages_small;
};
ChunkPlan plan_chunks(int32_t n_seqs, int32_t n_kv_heads, int32_t max_seq_len);

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
