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

namespace pq {

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

namespace {

// A value every lane holds alike, moved to a scalar register (the compiler keeps the results of
// shuffles and integer divisions in vector registers otherwise, one per lane for nothing).
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ int clamped_len(const DecodeArgs& a, int s) {
  return min(a.seq_lens[s], a.max_seq_len);
}
__device__ __forceinline__ int pages_of_len(int L) { return L > 0 ? (L + kGroup - 1) / kGroup : 0; }

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_of_u32(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, true));
}
// Maximum over each half of the wavefront, in all of its lanes.
__device__ __forceinline__ uint32_t half_wave_max_u32(uint32_t x) {
  x = max(x, dpp_of_u32<0xB1>(x));
  x = max(x, dpp_of_u32<0x4E>(x));
  x = max(x, dpp_of_u32<0x141>(x));
  x = max(x, dpp_of_u32<0x140>(x));
  auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return max(r[0], r[1]);
}
__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// Maximum / sum over the wavefront, as a scalar.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  x = half_wave_max_u32(x);
  auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return static_cast<uint32_t>(uni(static_cast<int>(max(s[0], s[1]))));
}
// Sum over the lanes up to and including this one.
__device__ __forceinline__ int wave_prefix(int v) {
  // shifts within the rows of 16, then the rows' last lanes to the rows behind them
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);      // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31 to rows 2 and 3
  return v;
}
__device__ __forceinline__ int wave_sum(int v) {
  uint32_t x = static_cast<uint32_t>(v);
  x += dpp_of_u32<0xB1>(x);
  x += dpp_of_u32<0x4E>(x);
  x += dpp_of_u32<0x141>(x);
  x += dpp_of_u32<0x140>(x);
  auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = r[0] + r[1];
  auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return uni(static_cast<int>(s[0] + s[1]));
}

// The cut of a launch into chunks, made alike by every wavefront of it.  Slot u of a KV head: chunk 0
// of sequence u for the first n_seqs, then the second chunks of the sequences that have one, and so on.
// Sequences 0 .. 63 sit in a register, the others in LDS.
struct BalancedPlan {
  int pages0, n0;                              // sequence `lane`: pages; chunks (0 past the last sequence, 1 if it is empty)
  const int32_t* others;                       // LDS: pages of sequences 64 ..
  int n_seqs, lane;
  ChunkLengths len;
  float per_big, per_small;
  enum Kind { kGeneral, kAlike, kFitted } kind;   // which cut it is (cut_resident)
  int others0, size0;                          // kFitted: chunks behind the first ones, of the sequences up to this lane's; pages a chunk
  int units;                                   // kFitted: compute units for each KV head

  __device__ __forceinline__ void load(const DecodeArgs& a, int lane_) {
    lane = lane_;
    n_seqs = a.n_seqs;
    pages0 = a.seq_lens[min(lane, n_seqs - 1)];                        // the length; waited for in cut()
  }
  // Sequences 64 .. into LDS (kBalancedSeqs words), by the whole work-group; holds a barrier if there are any.
  __device__ __forceinline__ void store_others(const DecodeArgs& a, int32_t* lds, int tid) {
    others = lds;
    if (n_seqs > 64) {
#pragma unroll 1
      for (int s = tid; s < n_seqs; s += 256) lds[s] = pages_of_len(clamped_len(a, s));
      __syncthreads();
    }
  }
  // f(first sequence of the block, pages of this lane's, chunks of this lane's)
  template <typename F>
  __device__ __forceinline__ void for_blocks(F f) const {
    f(0, pages0, n0);
#pragma unroll 1
    for (int s0 = 64; s0 < n_seqs; s0 += 64) {
      const int p = s0 + lane < n_seqs ? others[s0 + lane] : 0;
      f(s0, p, chunks_of(s0 + lane, p));
    }
  }
  // ceil(x / d) for 0 <= x <= 2^24 (every page count), by the reciprocal of d; d >= 4, or x < 8
  static __device__ __forceinline__ int div_up(int x, int d, float inverse) {
    const int q = static_cast<int>(static_cast<float>(x) * inverse);   // off by one at most
    const int rest = x - q * d;
    return q + (rest > 0 ? 1 : 0) + (rest > d ? 1 : 0) - (rest <= -d ? 1 : 0);
  }
  // as chunks_of_pages()
  __device__ __forceinline__ int chunks_of(int seq, int p) const {
    const int rest = max(0, p - len.n_big * len.big);
    const int n = min(div_up(p, len.big, per_big), len.n_big) + div_up(rest, len.small, per_small);
    return seq < n_seqs ? max(1, n) : 0;
  }
  __device__ __forceinline__ void find_chunks() {
    per_big = __builtin_amdgcn_rcpf(static_cast<float>(len.big));
    per_small = __builtin_amdgcn_rcpf(static_cast<float>(len.small));
    n0 = chunks_of(lane, pages0);
  }
  __device__ __forceinline__ int count() {
    find_chunks();
    int sum = 0;
    for_blocks([&](int, int, int n) { sum += n; });
    return wave_sum(sum);
  }
  // after load() and store_others(); returns the chunks per KV head
  __device__ __forceinline__ int cut(const DecodeArgs& a, bool fp16_values) {
    pages0 = lane < n_seqs ? pages_of_len(min(pages0, a.max_seq_len)) : 0;
    kind = kGeneral;
    if (a.fit_chunks > 0) {
      const int slots = cut_resident(a);
      if (slots > 0) return slots;
    }
    int sum = pages0, most = pages0;
#pragma unroll 1
    for (int s = 64 + lane; s < n_seqs; s += 64) {
      sum += others[s];
      most = max(most, others[s]);
    }
    const int total = wave_sum(sum), longest = static_cast<int>(wave_max_u32(static_cast<uint32_t>(most)));
    // Lengths spread over a range (or all alike): as if all were the longest, which is what the rule was
    // measured with.  A few far above the rest: by the pages there are.
    const int even = n_seqs * longest;
    const int pages_per_head = even <= total * 5 / 2 ? even : total;
    len = chunk_lengths((pages_per_head * a.n_kv_heads + kResidentGroups - 1) / kResidentGroups, longest, fp16_values);
    int chunks = count();
    if (chunks > n_seqs + a.spare_chunks || uni(chunks_of(0, longest)) > kBalancedFan) {
      // equal chunks, as short as there is room for: sum of ceil(p / c) <= n_seqs + total / c
      len.big = len.small = whole_rounds(max((total + a.spare_chunks - 1) / a.spare_chunks, (longest + kBalancedFan - 1) / kBalancedFan));
      len.n_big = longest;
      chunks = count();
    }
    return chunks;
  }
  // The cut of a launch of at most 64 sequences that leaves places on the compute units when every sequence has one work-group.
  // If all sequences are equally long nothing has to be counted (kAlike), and if they are as long as the host was told its chunk
  // lengths are the measured ones.  If they are not, what matters is that all chunks start at once and that the two work-groups of a compute unit
  // are not both long ones (kFitted): the shortest whole rounds with no more chunks than are resident together, a sequence's
  // chunks alike, and locate_fitted() says who takes which.  Returns the slots that may have a chunk, 0 if neither will do.
  // Measured (8 KV heads, 4 query heads each, microseconds: chunks cut on the host, or here by chunk_lengths() from 48 pages a
  // share on, and dealt out chunk by chunk -> this):
  //   32 x 512 .. 8K tokens 70.9 -> 61.4, 3+3-bit keys and 2-bit values 42.4 -> 38.7;  8 x 2K .. 30K, 4-bit values 54.1 -> 41.8
  //   grouped quantizer: 12 x 1K .. 16K 80.8 -> 52.9, 8 heads and 4-bit values 81.2 -> 47.2;  20 x 5K .. 10K, 2-bit values 50.8 -> 39.7
  //   6 x 500 .. 12K 36.4 -> 27.1;  30 x 300 .. 2500 29.3 -> 25.2;  16 x 4K .. 32K 142.8 -> 114.3;  8 x 4K .. 8K, 32 KV heads 82.1 -> 77.0
  //   alike: 16 x 2K with a max_seq_len of 32K 20.7 -> 20.8, 16 x 8K 60.0 -> 59.4, 31 x 3000 43.5 -> 43.5;  8 x 8K, 32 KV heads 109.4 -> 109.0
  __device__ __forceinline__ int cut_resident(const DecodeArgs& a) {
    const int max_pages = pages_of_len(a.max_seq_len);
    const int first_pages = uni(pages0);
    if (__builtin_amdgcn_ballot_w64(lane < n_seqs && pages0 != first_pages) == 0) {
      kind = kAlike;
      len.big = a.pages_per_chunk;
      len.small = a.pages_small;
      len.n_big = a.n_big;
      if (first_pages != max_pages) {                                  // shorter ones: as many chunks as there are places
        const int n = a.fit_chunks / n_seqs;
        len.big = len.small = max(kWaveRound, whole_rounds((first_pages + n - 1) / n));
        len.n_big = max_pages;
      }
      find_chunks();
      return n_seqs * uni(n0);
    }
    const int total = wave_sum(pages0);
    // as long as the longest of the host's (with longer ones, work-groups that come as others go are the better balance)
    constexpr int kLongest = 64;
#pragma unroll 1
    for (int c = whole_rounds(max((total + a.fit_chunks - 1) / a.fit_chunks, (max_pages + kBalancedFan - 1) / kBalancedFan)); c <= kLongest; c += 2 * kWaveRound) {
      // two lengths at a time, their counts in the halves of a word
      const int n = lane < n_seqs ? max(1, div_up(pages0, c, __builtin_amdgcn_rcpf(static_cast<float>(c)))) : 0;
      const int m = lane < n_seqs ? max(1, div_up(pages0, c + kWaveRound, __builtin_amdgcn_rcpf(static_cast<float>(c + kWaveRound)))) : 0;
      const int both = wave_sum(n | (m << 16));
      const bool first = (both & 0xffff) <= a.fit_chunks;
      if (first || (both >> 16) <= a.fit_chunks) {
        kind = kFitted;
        n0 = first ? n : m;
        size0 = div_up(pages0, n0, __builtin_amdgcn_rcpf(static_cast<float>(n0)));
        units = kComputeUnits / a.n_kv_heads;
        others0 = wave_prefix(max(n0 - 1, 0));
        return 2 * units;
      }
    }
    return 0;
  }
  // Slot u takes its place on compute unit u % units of its KV head, if work-groups are handed out in order (which they are:
  // of 512 work-groups i and i + 256 shared a unit, 256 times of 256; nothing but time hangs on it).  The first slots have the sequences' first chunks; of the others, the longest chunk goes to the unit
  // with the least to do, the next one to the next.  False: there are no more.
  __device__ __forceinline__ bool locate_fitted(int u, int& seq, int& chunk) const {
    const int alone = max(0, units - n_seqs);                          // units without a first chunk
    int rank = u - n_seqs;
    if (u >= units) {
      const int partner = u - units;
      const bool open = lane < min(n_seqs, units) && lane >= n_seqs - units;           // the units of these sequences' first chunks have a place left
      rank = alone + __builtin_popcountll(__builtin_amdgcn_ballot_w64(open)) + partner - n_seqs;
      if (partner < n_seqs) {
        const int mine = __builtin_amdgcn_readlane(size0, partner);
        rank = alone + __builtin_popcountll(__builtin_amdgcn_ballot_w64(open && (size0 < mine || (size0 == mine && lane < partner))));
      }
    }
    if (rank >= __builtin_amdgcn_readlane(others0, 63)) return false;
    // by the rounds a chunk takes, then second chunks, third ones ...
    const int rounds = (size0 + kWaveRound - 1) / kWaveRound;
    uint64_t have = 0;
    for (int r = uni(static_cast<int>(wave_max_u32(static_cast<uint32_t>(n0 > 1 ? rounds : 0))));; --r) {
      for (chunk = 1;; ++chunk) {
        have = __builtin_amdgcn_ballot_w64(rounds == r && n0 > chunk);
        const int n = __builtin_popcountll(have);
        if (n == 0) break;
        if (rank < n) {
          const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(have >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(have), 0)));
          seq = __builtin_ctzll(__builtin_amdgcn_ballot_w64(rounds == r && n0 > chunk && below == rank));
          return true;
        }
        rank -= n;
      }
      if (r <= 0) return false;                                        // (not reached: rank is below the number of chunks)
    }
  }
  // sequence and chunk of slot u >= n_seqs, u < what the cut returned; false: it has none
  __device__ __forceinline__ bool locate(int u, int& seq, int& chunk) const {
    if (kind == kFitted) return locate_fitted(u, seq, chunk);
    if (kind == kAlike) {
      chunk = uni(static_cast<int>(static_cast<float>(u) * __builtin_amdgcn_rcpf(static_cast<float>(n_seqs))));   // off by one at most
      chunk += u - chunk * n_seqs >= n_seqs ? 1 : (u - chunk * n_seqs < 0 ? -1 : 0);
      seq = u - chunk * n_seqs;
      return true;
    }
    // most chunk numbers c below which at most u slots lie: sum of min(n, c) over the sequences
    int lo = 1, before = n_seqs, hi = kBalancedFan;
#pragma unroll 1
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      int sum = 0;
      for_blocks([&](int, int, int n) { sum += min(n, mid); });
      sum = wave_sum(sum);
      if (sum <= u) {
        lo = mid;
        before = sum;
      } else {
        hi = mid;
      }
    }
    chunk = lo;
    seq = 0;
    int rank = u - before;
    for_blocks([&](int s0, int, int n) {
      const uint64_t have = __builtin_amdgcn_ballot_w64(n > lo);
      const int of_block = __builtin_popcountll(have);
      if (rank >= 0 && rank < of_block) {
        const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(have >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(have), 0)));
        seq = s0 + __builtin_ctzll(__builtin_amdgcn_ballot_w64(n > lo && below == rank));
      }
      rank -= of_block;
    });
    return true;
  }
  // first page and most pages of a chunk
  __device__ __forceinline__ void pages_of_chunk(int seq, int chunk, int& first, int& most) const {
    if (kind == kFitted) {
      most = __builtin_amdgcn_readlane(size0, seq);
      first = chunk * most;
      return;
    }
    const int big = min(chunk, len.n_big);
    first = big * len.big + (chunk - big) * len.small;
    most = chunk < len.n_big ? len.big : len.small;
  }
  // pages and chunks of a sequence, and the chunks of those before it
  __device__ __forceinline__ void sequence(int seq, int& n_pages, int& n_chunks, int& chunks_before) const {
    if (kind != kGeneral) {
      n_pages = __builtin_amdgcn_readlane(pages0, seq);
      n_chunks = __builtin_amdgcn_readlane(n0, seq);
      chunks_before = kind == kAlike ? seq * n_chunks : seq + __builtin_amdgcn_readlane(others0, seq) - (n_chunks - 1);
      return;
    }
    int sum = 0;
    for_blocks([&](int s0, int p, int n) {
      sum += s0 + lane < seq ? n : 0;
      if (seq >= s0 && seq < s0 + 64) {
        n_pages = __builtin_amdgcn_readlane(p, seq - s0);
        n_chunks = __builtin_amdgcn_readlane(n, seq - s0);
      }
    });
    chunks_before = wave_sum(sum);
  }
};

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
