// CPU run of the cut of an attention launch (csrc/pq_decode_cut.hpp) with the host's plan (csrc/pq_plan.hpp), for tests.
// A wavefront is 64 contexts that take turns: each runs to its next wavefront-wide operation, the last one to arrive
// carries it out for all.  They have to arrive at the same one: what the code says of a wavefront is checked with it.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <vector>

namespace lanes {

constexpr int kLanes = 64;
enum Op { kNone, kBallot, kReadLane, kReadFirst, kDpp, kSwap16, kSwap32, kSync };
struct Lane {
  ucontext_t context;
  std::vector<char> stack;
  bool done;
  Op op;
  int a, b, ctrl, rows;
  uint64_t result;
};
Lane lane[kLanes];
ucontext_t scheduler;
int current;
std::function<void(int)> body;

[[noreturn]] void fail(const char* what) {
  fprintf(stderr, "cut_host: %s\n", what);
  abort();
}

// One operation for all lanes.
void carry_out() {
  const Op op = lane[0].op;
  for (const Lane& l : lane)
    if (l.done || l.op != op || l.ctrl != lane[0].ctrl || l.rows != lane[0].rows) fail("the lanes are not at the same operation");
  switch (op) {
    case kBallot: {
      uint64_t bits = 0;
      for (int i = 0; i < kLanes; ++i) bits |= static_cast<uint64_t>(lane[i].a != 0) << i;
      for (Lane& l : lane) l.result = bits;
      break;
    }
    case kReadFirst:
      for (Lane& l : lane) l.result = static_cast<uint32_t>(lane[0].a);
      break;
    case kReadLane:
      for (Lane& l : lane) {
        if (l.b != lane[0].b || l.b < 0 || l.b >= kLanes) fail("readlane of no lane, or not of one");
        l.result = static_cast<uint32_t>(lane[l.b].a);
      }
      break;
    case kDpp:
      for (int i = 0; i < kLanes; ++i) {
        const int row = i / 16, c = i % 16, ctrl = lane[0].ctrl;
        int from;
        if (ctrl < 0x100) from = row * 16 + (c & ~3) + (ctrl >> 2 * (c & 3) & 3);        // quad_perm
        else if (ctrl > 0x110 && ctrl < 0x120) from = c >= ctrl - 0x110 ? i - (ctrl - 0x110) : -1;   // row_shr
        else if (ctrl == 0x140) from = row * 16 + 15 - c;                              // row_mirror
        else if (ctrl == 0x141) from = row * 16 + (c & 8) + 7 - (c & 7);               // row_half_mirror
        else if (ctrl == 0x142) from = row > 0 ? row * 16 - 1 : -1;                    // row_bcast:15
        else if (ctrl == 0x143) from = i >= 32 ? 31 : -1;                              // row_bcast:31
        else fail("an unknown way of reading another lane");
        lane[i].result = static_cast<uint32_t>(from < 0 || !(lane[0].rows >> row & 1) ? 0 : lane[from].a);
      }
      break;
    case kSwap16:                                                      // rows 1 and 3 of a against rows 0 and 2 of b
    case kSwap32:
      for (int i = 0; i < kLanes; ++i) {
        const int half = op == kSwap16 ? 16 : 32;
        const bool upper = (i & half) != 0;
        const uint32_t first = static_cast<uint32_t>(upper ? lane[i - half].b : lane[i].a);
        const uint32_t second = static_cast<uint32_t>(upper ? lane[i].b : lane[i + half].a);
        lane[i].result = first | static_cast<uint64_t>(second) << 32;
      }
      break;
    default: break;
  }
}

uint64_t arrive(Op op, int a, int b, int ctrl, int rows) {
  Lane& l = lane[current];
  l.op = op, l.a = a, l.b = b, l.ctrl = ctrl, l.rows = rows;
  swapcontext(&l.context, &scheduler);
  return l.result;
}

void entry() {
  body(current);
  lane[current].done = true;
  swapcontext(&lane[current].context, &scheduler);
}

void run(std::function<void(int)> f) {
  body = f;
  for (Lane& l : lane) {
    if (l.stack.empty()) l.stack.resize(64 << 10);
    getcontext(&l.context);
    l.context.uc_stack.ss_sp = l.stack.data();
    l.context.uc_stack.ss_size = l.stack.size();
    l.context.uc_link = nullptr;
    l.done = false;
    makecontext(&l.context, entry, 0);
  }
  for (;;) {
    for (current = 0; current < kLanes; ++current) swapcontext(&scheduler, &lane[current].context);
    int ended = 0;
    for (const Lane& l : lane) ended += l.done;
    if (ended == kLanes) return;
    if (ended) fail("some lanes have ended, others have not");
    carry_out();
  }
}

struct Pair {
  uint32_t v[2];
  uint32_t operator[](int i) const { return v[i]; }
};

}  // namespace lanes

#define __host__
#define __device__
#define __forceinline__ inline
#define __syncthreads() ((void)lanes::arrive(lanes::kSync, 0, 0, 0, 0))
inline int amd_readfirstlane(int x) { return static_cast<int>(lanes::arrive(lanes::kReadFirst, x, 0, 0, 0)); }
inline int amd_readlane(int x, int from) { return static_cast<int>(lanes::arrive(lanes::kReadLane, x, from, 0, 0)); }
inline uint64_t amd_ballot(bool x) { return lanes::arrive(lanes::kBallot, x, 0, 0, 0); }
inline int amd_dpp(int old, int x, int ctrl, int rows, int, bool) {
  if (old != 0) lanes::fail("lanes that read none get zero here");
  return static_cast<int>(lanes::arrive(lanes::kDpp, x, 0, ctrl, rows));
}
inline lanes::Pair amd_swap(lanes::Op op, uint32_t a, uint32_t b) {
  const uint64_t r = lanes::arrive(op, static_cast<int>(a), static_cast<int>(b), 0, 0);
  return {{static_cast<uint32_t>(r), static_cast<uint32_t>(r >> 32)}};
}
inline int amd_mbcnt(uint32_t mask, int add, int first) {              // bits of the mask below this lane
  const int n = std::min(std::max(lanes::current - first, 0), 32);
  return add + __builtin_popcountll(mask & ((uint64_t{1} << n) - 1));
}
// off by a unit in the last place, as the hardware's may be
float reciprocal_error = 0.f;
inline float amd_rcp(float x) { return 1.f / x * (1.f + reciprocal_error); }
#define __builtin_amdgcn_readfirstlane amd_readfirstlane
#define __builtin_amdgcn_readlane amd_readlane
#define __builtin_amdgcn_ballot_w64 amd_ballot
#define __builtin_amdgcn_update_dpp amd_dpp
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) amd_swap(lanes::kSwap16, a, b)
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) amd_swap(lanes::kSwap32, a, b)
#define __builtin_amdgcn_mbcnt_lo(mask, add) amd_mbcnt(mask, add, 0)
#define __builtin_amdgcn_mbcnt_hi(mask, add) amd_mbcnt(mask, add, 32)
#define __builtin_amdgcn_rcpf amd_rcp

#include "pq_plan.hpp"

namespace pq {
using std::max;
using std::min;
struct DecodeArgs {
  const int32_t* seq_lens;
  int32_t n_seqs, n_kv_heads, max_seq_len, pages_per_chunk, n_chunks, n_big, pages_small, spare_chunks, fit_chunks;
};
}  // namespace pq

#include "pq_decode_cut.hpp"

// A launch's plan and, if it is cut on the device, its slots of one KV head.
//   plan[0..7]: grid places per KV head, work-groups resident at once per KV head (0: that cut is not tried), whether the
//     kernel merges, pages of the host's longest chunk, its chunks per sequence, the workspace's partials per query head of a
//     KV head, the cut that was made (-1: on the host), slots with a chunk or that may have one.
//   slots[6 u ..]: sequence (-1: slot u has nothing), chunk, first page, pages, the sequence's chunks, chunks of the sequences before it
// Returns the number of slots written.
extern "C" int cut_host(int n_seqs, int n_kv_heads, int n_q_heads, int grouped, int v_bits, const int32_t* lens, int max_seq_len, float error,
                        int64_t* plan, int32_t* slots) {
  using namespace pq;
  reciprocal_error = error;
  pq_layout layout = {};
  layout.head_dim = kHeadDim;
  layout.r_bits = layout.t_bits = 4;
  layout.group_tokens = kGroup;
  layout.n_kv_heads = n_kv_heads;
  layout.angle_quantizer = grouped ? PQ_ANGLE_GROUPED : PQ_ANGLE_UNIFORM;
  const ChunkPlan host = plan_attention(&layout, v_bits, n_seqs, n_q_heads, max_seq_len);
  const DeviceCut cut = device_cut(&layout, host, v_bits, n_seqs, n_q_heads, max_seq_len);
  plan[0] = cut.places > 0 ? cut.places : static_cast<int64_t>(n_seqs) * host.n_chunks;
  plan[1] = cut.fit_chunks;
  plan[2] = merges_in_kernel(&layout, host, cut, n_seqs, n_q_heads, max_seq_len);
  plan[3] = host.pages_per_chunk;
  plan[4] = host.n_chunks;
  plan[5] = static_cast<int64_t>(workspace_slots(&layout, n_seqs, n_q_heads, max_seq_len)) / (n_q_heads / n_kv_heads);
  plan[6] = -1;
  plan[7] = 0;
  if (cut.places == 0) return 0;
  const DecodeArgs a = {lens, n_seqs, n_kv_heads, max_seq_len, host.pages_per_chunk, host.n_chunks, host.n_big, host.pages_small, cut.spare_chunks, cut.fit_chunks};
  std::vector<int32_t> others(kBalancedSeqs);
  for (int s = 0; s < n_seqs; ++s) others[s] = pages_of_len(clamped_len(a, s));   // (the other wavefronts of the work-group)
  lanes::run([&](int id) {
    BalancedPlan p = {};
    p.load(a, id);
    p.store_others(a, others.data(), id);
    const int chunks = p.cut(a, v_bits == 16, grouped != 0);
    if (id == 0) plan[6] = p.kind, plan[7] = chunks;
    if (p.kind == BalancedPlan::kFitted && (p.size0 < 0 || p.size0 > p.pages0 + kWaveRound)) lanes::fail("a lane's pages a chunk are not a number of pages");
    for (int u = 0; u < plan[0]; ++u) {
      int32_t* const to = slots + 6 * u;
      if (id == 0) to[0] = -1;
      int seq = u, chunk = 0;
      if (u >= chunks || (u >= n_seqs && !p.locate(u, seq, chunk))) continue;
      int n_pages = 0, n_chunks = 0, before = 0, first = 0, most = 0;
      seq = uni(seq);
      chunk = uni(chunk);
      p.sequence(seq, n_pages, n_chunks, before);
      p.pages_of_chunk(seq, chunk, first, most);
      if (id == 0) to[0] = seq, to[1] = chunk, to[2] = first, to[3] = min(most, n_pages - first), to[4] = n_chunks, to[5] = before;
    }
  });
  return static_cast<int>(plan[0]);
}
