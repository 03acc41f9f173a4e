// What the host knows of a launch and plans with: sizes of the format, the chunk plans, the workspace they need, and
// which attention launches are cut into chunks on the device (pq_decode_cut.hpp).  Plain C++ but for
// __host__ __device__: tests build it for the CPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "polarquant.h"

namespace pq {

constexpr int kHeadDim = 128;          // d
constexpr int kPairs = kHeadDim / 2;   // P: pair j = dims (j, j + 64)
constexpr int kGroup = 128;            // g: tokens per page / quantization group
constexpr int kPairsPerUnit = 16;      // one packed unit = 16 pairs of one token
constexpr int kBlocks = kPairs / kPairsPerUnit;
constexpr int kMaxAngleBins = 32;      // t <= 5

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

// Chunks of the grouped quantizer's attention kernel, and the size of the workspace for all: one
// work-group per (sequence, KV head, chunk).  Chunks are whole pages, a
// multiple of the 4 wavefronts of a work-group; they shrink from 32 pages
// until the launch has at least the 512 work-groups that are resident at
// once (2 per compute unit).  Long chunks amortise the table build and keep
// each wavefront's page pipeline running; measured on MI355X, a target of 512
// beat 2048 by 4 % at 16 x 32K and by 16 % for one 128K sequence.
inline ChunkPlan plan_chunks(int32_t n_seqs, int32_t n_kv_heads, int32_t max_seq_len) {
  const int64_t max_pages = (static_cast<int64_t>(max_seq_len) + kGroup - 1) / kGroup;
  const int64_t units = static_cast<int64_t>(n_seqs) * n_kv_heads;
  constexpr int64_t kWantGroups = 512;
  int32_t ppc = 32;
  while (ppc > 4 && units * ((max_pages + ppc - 1) / ppc) < kWantGroups) ppc >>= 1;
  ChunkPlan p;
  p.pages_per_chunk = ppc;
  p.n_chunks = static_cast<int32_t>((max_pages + ppc - 1) / ppc);
  p.n_big = p.n_chunks;
  p.pages_small = ppc;
  return p;
}

// Most chunks of a unit that are combined in the kernel: arrivals at one word are taken one after
// the other by the memory system, and whoever combines n partials waits for their loads.
constexpr int kMergeFan = 16;
constexpr int kBalancedFan = 32;              // (launches cut on the device have no other way)
constexpr int kBalancedSeqs = 512;            // most sequences of theirs
constexpr int kComputeUnits = 256;            // MI355X
constexpr int kResidentGroups = 2 * kComputeUnits;   // work-groups of the attention kernel

// Lengths of chunks, in pages: the first n_big chunks of a sequence are `big` long, the others `small`.
// Starting and ending a chunk costs about as much as streaming 8 pages: chunks are as long as they
// can be without leaving compute units idle at the end.  `share` is a resident work-group's part of
// the launch's pages, `longest` the longest sequence.  Measured (pages per chunk: microseconds;
// "48 + 16": 48, the last quarter in chunks of 16):
//   up to 16 pages a share   248 units x 2 .. 24 pages   8: 51, 16: 44, 24: 47;  8 x 1024  8: 64, 16: 61, 24: 68
//   fp16 values              256 x 64      24: 110, 32: 110, 44: 107.5, 64: 110;  128 x 256  32: 210, 44: 212, 64: 208
//                            512 x 8 .. 128  24: 240, 44: 238, 64: 239, 64 + 24: 233
//   quantized values         256 x 4 .. 64   16: 54, 24: 43.4, 24 + 8: 44, 32: 55;  128 x 256  32: 131, 64: 126, 48 + 16: 125
// (With fp16 values a work-group that is left alone streams faster; with quantized ones it does not.)
struct ChunkLengths {
  int big, small, n_big;
};
constexpr int kWaveRound = 4;                 // pages: one for each wavefront of a work-group
__host__ __device__ inline int whole_rounds(int pages) { return (pages + kWaveRound - 1) / kWaveRound * kWaveRound; }
__host__ __device__ inline ChunkLengths chunk_lengths(int share, int longest, bool fp16_values) {
  ChunkLengths c;
  c.n_big = longest;                                       // more than there are
  if (longest < 2 * kWaveRound) {
    c.big = c.small = longest > 1 ? longest : 1;           // less than two pages a wavefront: one chunk, nothing to merge
  } else if (share <= 16) {
    c.big = c.small = share <= 4 ? 4 : (share <= 8 ? 8 : 16);
  } else if (fp16_values && share <= 64) {
    const int p = whole_rounds(share * 4 / 3);
    c.big = c.small = p < 64 ? p : 64;
  } else {
    const int b = share < 96 ? whole_rounds(share * 3 / 4) : 64, s = share < 96 ? whole_rounds(share / 4) : 24;
    c.big = b < 64 ? b : 64;
    c.small = s < 8 ? 8 : (s > 24 ? 24 : s);
    const int n = longest * 4 / 5 / c.big;
    c.n_big = n > 1 ? n : 1;
  }
  return c;
}

// Work-groups of four pages each that the shape could have, as far as 768 (the workspace's size is
// stated in them).
constexpr int64_t kCountedGroups = 768;
inline int64_t four_page_groups(const pq_layout* l, int32_t n_seqs, int32_t max_seq_len) {
  const int64_t max_pages = (static_cast<int64_t>(max_seq_len) + kGroup - 1) / kGroup;
  const int64_t bound = static_cast<int64_t>(n_seqs) * l->n_kv_heads * max_pages;   // pages x KV heads, at most
  return std::min<int64_t>(kCountedGroups, (bound + 3) / 4);
}

// Pages enough for at least 256 work-groups; the second: and on the uniform angle grid.
inline bool large_launch(const pq_layout* l, int32_t n_seqs, int32_t max_seq_len) {
  return n_seqs <= 4096 && four_page_groups(l, n_seqs, max_seq_len) >= kComputeUnits;
}
inline bool large_uniform_launch(const pq_layout* l, int32_t n_seqs, int32_t max_seq_len) {
  return l->angle_quantizer == PQ_ANGLE_UNIFORM && large_launch(l, n_seqs, max_seq_len);
}

// Grouped angle quantizer: query heads per KV head from which on the kernels of pq_decode_matrix.hpp take over.  They make
// the keys' coordinates, whatever the number of heads (about 11 instructions a symbol); the vector unit's take 3 + heads, and
// heads times as many for the values.  Vector unit against matrix cores, microseconds: 3 heads, which are two passes of the
// former, 16 x 16K tokens 231 / 116.  2 heads 16 x 16K 117 / 114, with 4-bit values 78.5 / 82, one sequence of 1000 14.7 / 14.5; 1 head 114 /
// 114, 76 / 81, 13.5 / 14.2.
constexpr int kGroupedMatrixHeads = 3;
inline bool grouped_on_matrix(const pq_layout* l, int group_total) { return l->angle_quantizer == PQ_ANGLE_GROUPED && group_total >= kGroupedMatrixHeads; }

inline size_t workspace_slots(const pq_layout* l, int32_t n_seqs, int32_t n_q_heads, int32_t max_seq_len) {
  const ChunkPlan plan = plan_chunks(n_seqs, l->n_kv_heads, max_seq_len);
  const size_t units = static_cast<size_t>(n_seqs) * l->n_kv_heads;
  const size_t chunk_slots = static_cast<size_t>(n_seqs) * n_q_heads * plan.n_chunks;
  return std::max(chunk_slots, (static_cast<size_t>(four_page_groups(l, n_seqs, max_seq_len)) + units) * (n_q_heads / l->n_kv_heads));
}

// Chunk plan of the uniform angle grid's attention kernel for launches that are cut on the host, as if
// every sequence had max_seq_len tokens (chunk_lengths() says why chunks are as long as they are).
// The two-stage entry points, whose second one does not know the values' width, use the fp16 plan.
inline ChunkPlan plan_uniform(const pq_layout* l, int32_t v_bits, int32_t n_seqs, int32_t n_q_heads, int32_t max_seq_len) {
  const int64_t max_pages = (static_cast<int64_t>(max_seq_len) + kGroup - 1) / kGroup;
  const int64_t units = static_cast<int64_t>(n_seqs) * l->n_kv_heads;
  const int64_t share = std::min<int64_t>(1 << 20, (units * max_pages + kResidentGroups - 1) / kResidentGroups);
  const ChunkLengths len = chunk_lengths(static_cast<int>(share), static_cast<int>(max_pages), v_bits == 16);
  int64_t big = len.big, small = len.small, n_big = big == small ? 0 : len.n_big;
  // as many partials as the workspace holds (its own plan has max_pages / 32 chunks or more)
  const int64_t most = static_cast<int64_t>(workspace_slots(l, n_seqs, n_q_heads, max_seq_len)) / (static_cast<int64_t>(n_seqs) * n_q_heads);
  auto chunks = [&] {
    const int64_t first = std::min(n_big, (max_pages + big - 1) / big), rest = max_pages - n_big * big;
    return first + (rest > 0 ? (rest + small - 1) / small : 0);
  };
  while (chunks() > most && small < max_pages) {
    small += 4;
    if (small > big) {
      big = small;
      n_big = 0;
    }
  }
  ChunkPlan p;
  p.pages_per_chunk = static_cast<int32_t>(big);
  p.pages_small = static_cast<int32_t>(small);
  p.n_chunks = static_cast<int32_t>(chunks());
  p.n_big = static_cast<int32_t>(n_big == 0 && big == small ? p.n_chunks : n_big);
  return p;
}
inline ChunkPlan plan_attention(const pq_layout* l, int32_t v_bits, int32_t n_seqs, int32_t n_q_heads, int32_t max_seq_len) {
  return l->angle_quantizer == PQ_ANGLE_UNIFORM ? plan_uniform(l, v_bits, n_seqs, n_q_heads, max_seq_len)
                                                : plan_chunks(n_seqs, l->n_kv_heads, max_seq_len);
}

// How a launch is cut into chunks on the device by the sequences' real lengths (BalancedPlan).  places: of the grid, per KV head; 0:
// the launch is cut on the host.  fit_chunks: how many chunks per KV head are resident at once, if that cut
// (BalancedPlan::cut_resident) is tried; spare_chunks: chunks per KV head beyond one a sequence that the general rule may make, 0 if the
// launch has the host's chunks where the other cut will not do.
// Three kinds of launches: sequences of at least two chunks that leave places on the compute units (fit_chunks > 0), from four pages a
// resident work-group on (below, chunks are one round long); launches where a resident work-group may have kCutShare pages or more, for the general
// rule, up to three work-groups a resident one or as many as the workspace has partials for (a launch may be of both kinds); and the
// others, cut as if every sequence had max_seq_len tokens.  With fewer than 16 units the host's cut has more chunks per unit than are combined in the kernel (but for launches
// of kCutShare pages, whose chunks may be 32 of a unit); above 512 sequences reading all lengths in every work-group costs more
// than uneven chunks do among so many.  The grouped quantizer's matrix kernels have the first kind and the last one.
constexpr int64_t kCutShare = 48;
struct DeviceCut {
  int32_t places, spare_chunks, fit_chunks;
};
// `host`: what plan_attention() gives for the launch.
inline DeviceCut device_cut(const pq_layout* l, const ChunkPlan& host, int32_t v_bits, int32_t n_seqs, int32_t n_q_heads, int32_t max_seq_len) {
  const int64_t units = static_cast<int64_t>(n_seqs) * l->n_kv_heads;
  const int64_t max_pages = (static_cast<int64_t>(max_seq_len) + kGroup - 1) / kGroup;
  const bool uniform = l->angle_quantizer == PQ_ANGLE_UNIFORM;
  if (!(uniform || grouped_on_matrix(l, n_q_heads / l->n_kv_heads)) || !large_launch(l, n_seqs, max_seq_len) || units < kResidentGroups / kBalancedFan || n_seqs > kBalancedSeqs ||
      l->n_kv_heads > kComputeUnits || units * max_pages >= (int64_t{1} << 30))
    return {0, 0, 0};
  const bool large = units * max_pages >= kCutShare * kResidentGroups;
  const int resident = 2 * (kComputeUnits / l->n_kv_heads);
  const int n_chunks = host.n_chunks;
  const bool fit = n_seqs <= 64 && n_seqs < resident && n_chunks >= 2 && n_chunks <= (large && uniform ? kBalancedFan : kMergeFan) &&
                   units * max_pages > kWaveRound * kResidentGroups;
  // (the workspace has room for the host's chunks, and at this size for one partial of each resident work-group; more places than
  // that cost time: 16 sequences of 2K tokens with a max_seq_len of 32K 21.7 us with three work-groups a resident one)
  int places = fit ? std::max(n_seqs * n_chunks, resident) : 0;
  if (!large || !uniform) return {places, 0, fit ? resident : 0};
  const int64_t partials = workspace_slots(l, n_seqs, l->n_kv_heads, max_seq_len) - units;     // (one query head per KV head)
  const int spare = static_cast<int>(std::min<int64_t>(3 * kResidentGroups, partials) / l->n_kv_heads);
  if (!fit) return {n_seqs + spare, spare, 0};
  // as many as the general rule would make of sequences of max_seq_len tokens, as far as there is room: with a shorter last part
  // they may be more than the host's (33 x 12000 tokens, 4-bit values: 99 chunks of 32 pages 112 us, 66 of 48 127)
  const ChunkLengths len = chunk_lengths(static_cast<int>(std::min<int64_t>(1 << 20, (units * max_pages + kResidentGroups - 1) / kResidentGroups)),
                                         static_cast<int>(max_pages), v_bits == 16);
  const int64_t first = std::min<int64_t>(len.n_big, (max_pages + len.big - 1) / len.big), rest = std::max<int64_t>(0, max_pages - first * len.big);
  places = static_cast<int>(std::max<int64_t>(places, std::min<int64_t>(n_seqs * (first + (rest + len.small - 1) / len.small), n_seqs + spare)));
  return {places, std::min(spare, places - n_seqs), resident};
}

// Whether one kernel does all of pq_decode_attention (true), or the merge kernel follows: the
// sequences are one chunk long, the launch is cut on the device, or a large one has few enough chunks per
// unit.  (Grouped quantizer, 16 x 16K tokens: 115.6 -> 114.7 us without the launch, 4 x 8K 23.7 -> 22.7.  Its vector-unit kernel
// leaves partials only.)
inline bool merges_in_kernel(const pq_layout* l, const ChunkPlan& host, const DeviceCut& cut, int32_t n_seqs, int32_t n_q_heads, int32_t max_seq_len) {
  if (l->angle_quantizer != PQ_ANGLE_UNIFORM && !grouped_on_matrix(l, n_q_heads / l->n_kv_heads)) return false;
  return cut.places > 0 || host.n_chunks == 1 || (host.n_chunks <= kMergeFan && large_launch(l, n_seqs, max_seq_len));
}

// Work-groups of 8 wavefronts: sequences of one chunk with more pages than 4 wavefronts take at once, and no more
// units than compute units (two work-groups of 4 share one otherwise).  One sequence of 777 tokens 13.3 -> 12.2 us
// (11.5 now, with a shorter end of the chunk), 16 of them 15.0 -> 14.7; up to 4 pages the wider work-group costs 1 us (300 tokens: 9.7 -> 10.7).  From 8 pages on
// chunk_lengths() makes two chunks: 8 units 13.0, 64 units 13.8 us; one chunk of 8 wavefronts 13.1 and 14.8 (4-bit values 12.7 and 12.7;
// 13.0 and 13.1), but with 256 units, a work-group on every compute unit, 20.0 and 18.5 (4-bit values 15.9, 14.7).
inline bool wide_groups(const pq_layout* l, const ChunkPlan& plan, int32_t n_seqs, int32_t max_seq_len) {
  return l->angle_quantizer == PQ_ANGLE_UNIFORM && plan.n_chunks == 1 && max_seq_len > kWaveRound * kGroup &&
         static_cast<int64_t>(n_seqs) * l->n_kv_heads <= kComputeUnits;
}

}  // namespace pq
