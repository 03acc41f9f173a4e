// How an attention launch is shared out among its work-groups, and how the pieces of one
// (sequence, KV head) are put together again inside the kernel.
//
// A work-group takes a chunk of one (sequence, KV head)'s pages.  Work-groups are in chunk-major
// order: the KV heads of one page are neighbours in memory and run together, every sequence's first
// chunks run first, and chunks that only longer sequences have come last.  There are about as many as
// are resident at once, or more: the hardware hands them out as others finish, which evens out the
// compute units' different speeds.  (A line of equal shares, one per resident work-group, with the
// units end to end measured 236 against 206 us for 16 x 32K tokens at 4 query heads per KV head: its
// work-groups stream from 512 places at once.)
//
// Lengths are known on the device only.  Launches of sequences that leave places on the compute units, and large ones, cut the
// chunks there, by the pages that really exist (struct BalancedPlan; device_cut() says which launches): the caller's
// max_seq_len may be far above, and one sequence may be far longer than the others.  The grid has a place for every chunk
// that the cut can make and each work-group finds its own; what is left over ends at once.  The other launches are cut on the host, as
// if every sequence had max_seq_len tokens.  8 KV heads, 4 query heads each, microseconds (host cut ->
// device cut): 1 x 128K + 63 x 1K tokens 168 -> 104, with 4-bit values 132 -> 67; 4 x 32K + 28 x 2K
// 133 -> 78; 8 x 4K with a max_seq_len of 32K 39.8 -> 20.8; 64 of 1K .. 16K with one of 64K 270 -> 229.
//
// A unit -- one (sequence, KV head) -- that is one chunk long is finished there.  Otherwise every
// chunk leaves its softmax partial (running maximum, denominator, un-normalised output) in the
// workspace, and either pq_decode_merge_kernel follows (launches cut on the host), or the chunks register at the unit's arrival
// word and whoever registers last combines them, in chunk order (so the result does not depend
// on who that was), and writes the output row.  Nobody waits for anybody.
//
// The arrival word needs no initialisation by the caller: it holds (mark, count), and a word
// without the mark -- memory the library has not used as an arrival word before -- is first made
// (mark, 0).  The last arriver puts the count back to zero, so a word that carries the mark
// always starts a launch at zero.
#pragma once
#include "pq_decode_kernels.hpp"
#include "pq_decode_cut.hpp"

namespace pq {
namespace {

__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// All memory operations this wavefront has issued are complete (for device-coherent stores:
// performed at memory, where every other work-group's device-coherent loads will find them).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Registers one arrival at a word; true for the arrival that completes `n`.  One atomic add in
// the normal case.  If the value it returns does not carry the mark, the word was never an
// arrival word (fresh memory, or memory that held partials of a launch of another shape): it is
// replaced by (mark, 0) -- one compare-and-swap wins, whatever the other arrivals have added to
// the old value meanwhile -- and every arrival that saw the unmarked word registers again.
constexpr uint64_t kArrivalMark = 0x7ff5c0dea11dull << 16;   // 48 bits above the 16-bit count
__device__ __forceinline__ bool arrive(uint64_t* word, int n) {
  unsigned long long* p = reinterpret_cast<unsigned long long*>(word);
  unsigned long long before = atomicAdd(p, 1ull);
  if ((before & ~0xffffull) != kArrivalMark) {
    unsigned long long cur = before + 1ull;
    while ((cur & ~0xffffull) != kArrivalMark) {
      const unsigned long long prev = atomicCAS(p, cur, kArrivalMark);
      if (prev == cur) break;
      cur = prev;
    }
    before = atomicAdd(p, 1ull);
  }
  return static_cast<int>(before & 0xffffull) + 1 == n;
}

// Puts a word's count back to zero (the last arriver, when nobody else will touch the word again).
__device__ __forceinline__ void reset_arrivals(uint64_t* word) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(word), kArrivalMark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kFinishThreads = 256;
// LDS the combination of partials needs (floats): a 4-float accumulator and a denominator per thread.
// A kernel lends memory that is idle at its end (16-byte aligned).
constexpr int kFinishLdsFloats = kFinishThreads * 5;

// End of a chunk.  `partial(h, quad, M, l)` returns the chunk's un-normalised output for query head
// h (of the a.n_heads <= NH this launch serves) and dimensions 4 quad .. 4 quad + 3, and sets the
// head's running maximum M (log2 units) and denominator l.  All threads of the
// work-group call this, the first kFinishThreads do the work; `lent` may be what `partial` reads, `stage` is a word of LDS.
//
// Partials that are combined in the kernel travel between work-groups that may sit on different
// XCDs, each with an L2 of its own.  They are written and read with device-coherent accesses
// (cache policy sc1: performed past the L2s) and ordered by waiting for the stores before the
// arrival is registered -- not by fences, which write back and invalidate whole caches (measured:
// with fences in every work-group the launch takes twice as long).
// The unit's partials: head h (from a.head0 on), chunk c in row row0 + h * stride + c.
template <int NH, typename Partial>
__device__ __forceinline__ void finish_chunk(const DecodeArgs& a, int seq, int kvh, int chunk, int n_chunks_seq, int64_t row0,
                                             int stride, int tid, Partial partial, float* lent, int* stage) {
  const int h = tid >> 5, quad = tid & 31;             // 256 threads: 8 heads x 32 quads
  const bool mine = h < a.n_heads;
  const int64_t head_row = static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0;
  float* const out_rows = a.out + head_row * kHeadDim;
  float M, l;
  f32x4 o;
  if (mine) o = partial(h, quad, M, l);
  if (a.merge_in_kernel && n_chunks_seq == 1) {
    if (mine) {
      const float inv = l > 0.f ? 1.f / l : 0.f;
      reinterpret_cast<float4*>(out_rows)[tid] = make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
    }
    return;
  }
  const uint32_t rows = static_cast<uint32_t>(a.n_heads * stride);
  const __amdgpu_buffer_rsrc_t r_acc = make_rsrc(a.ws_acc + row0 * kHeadDim, rows * (kHeadDim * 4));
  const __amdgpu_buffer_rsrc_t r_ml = make_rsrc(a.ws_ml + row0 * 2, rows * 8);
  if (mine) {
    const uint32_t row = static_cast<uint32_t>(h * stride + chunk);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{f2u(o.x), f2u(o.y), f2u(o.z), f2u(o.w)}, r_acc, row * (kHeadDim * 4) + quad * 16, 0, kAuxDevice);
    if (quad == 0) __builtin_amdgcn_raw_buffer_store_b64(u32x2{f2u(M), f2u(l)}, r_ml, row * 8, 0, kAuxDevice);
  }
  if (!a.merge_in_kernel) return;

  stores_done();                        // the partial has reached memory before the arrival is registered
  __syncthreads();
  uint64_t* const word = a.arrivals + static_cast<int64_t>(seq) * a.n_kv_heads + kvh;
  if (tid == 0) *stage = arrive(word, n_chunks_seq) ? 1 : 0;
  __syncthreads();
  if (*stage == 0) return;

  // last to arrive: combine the chunks.  Thread = (head, slice, 4 dims); a slice takes every
  // kSlices-th chunk, kAtOnce at a time with all their loads under way together.  Maxima are whole
  // numbers or -inf: the weights are exact.
  constexpr int TPH = kFinishThreads / NH;
  constexpr int kSlices = TPH / 32;
  constexpr int kAtOnce = 8;
  static_assert(kSlices == 1 || kSlices == 2, "4 or 8 heads: a head's threads sit in one wavefront");
  const int ch = tid / TPH, slice = (tid % TPH) >> 5;
  const int count = ch < a.n_heads ? n_chunks_seq : 0;   // no partials of heads the launch does not serve
  f32x4 r = {0.f, 0.f, 0.f, 0.f};
  float lt = 0.f, m = kNegInf;
  for (int k0 = slice; k0 < count; k0 += kAtOnce * kSlices) {
    u32x2 ml[kAtOnce];
    u32x4 v[kAtOnce];
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) {
      const uint32_t row = static_cast<uint32_t>(ch * stride + min(k0 + i * kSlices, count - 1));
      ml[i] = __builtin_amdgcn_raw_buffer_load_b64(r_ml, row * 8, 0, kAuxDevice);
      v[i] = __builtin_amdgcn_raw_buffer_load_b128(r_acc, row * (kHeadDim * 4) + quad * 16, 0, kAuxDevice);
    }
    float top = m;
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i)
      if (k0 + i * kSlices < count) top = fmaxf(top, u2f(ml[i].x));
    const float keep = top > kNegInf ? __builtin_amdgcn_exp2f(m - top) : 0.f;
    r *= keep;
    lt *= keep;
    m = top;
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) {
      if (k0 + i * kSlices < count && top > kNegInf) {
        const float wgt = __builtin_amdgcn_exp2f(u2f(ml[i].x) - top);
        r.x = fmaf(wgt, u2f(v[i].x), r.x);
        r.y = fmaf(wgt, u2f(v[i].y), r.y);
        r.z = fmaf(wgt, u2f(v[i].z), r.z);
        r.w = fmaf(wgt, u2f(v[i].w), r.w);
        lt = fmaf(wgt, u2f(ml[i].y), lt);
      }
    }
  }
  if constexpr (kSlices == 2) {
    f32x4* const part_o = reinterpret_cast<f32x4*>(lent);
    float* const part_l = lent + kFinishThreads * 4;
    const float top = fmaxf(m, __shfl_xor(m, 32));
    const float wgt = top > kNegInf ? __builtin_amdgcn_exp2f(m - top) : 0.f;
    if (tid < kFinishThreads) {
      part_o[tid] = r * wgt;
      part_l[tid] = lt * wgt;
    }
    __syncthreads();
    if (slice == 0 && tid < kFinishThreads) {
      r = part_o[tid] + part_o[tid + 32];
      lt = part_l[tid] + part_l[tid + 32];
    }
  }
  if (slice == 0 && ch < a.n_heads) {
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    reinterpret_cast<float4*>(out_rows)[ch * 32 + quad] = make_float4(r.x * inv, r.y * inv, r.z * inv, r.w * inv);
  }
  if (tid == 0) reset_arrivals(word);
}

}  // namespace
}  // namespace pq
