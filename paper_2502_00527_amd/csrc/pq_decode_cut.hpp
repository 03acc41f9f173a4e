// The cut of an attention launch into chunks by the sequences' real lengths, made on the device, and alike, by every
// wavefront of the launch; pq_decode_sched.hpp says why.  Only wavefront-wide operations and arithmetic: tests run it for
// 64 lanes on the CPU.  DecodeArgs and the device functions are declared before it.
#pragma once
#include "pq_plan.hpp"

namespace pq {
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

// The cut of a launch into chunks, made alike by every wavefront of it.  Slot u of a KV head is chunk 0
// of sequence u for the first n_seqs; the others have, by the kind of the cut, the second chunks of the sequences that have one, then
// the third ones and so on (kGeneral), chunk u / n_seqs of sequence u % n_seqs or nothing (kGrid), or the chunk that suits
// the compute unit (kFitted, locate_fitted()).  Sequences 0 .. 63 sit in a register, the others in LDS.
struct BalancedPlan {
  int pages0, n0;                              // sequence `lane`: pages; chunks (0 past the last sequence, 1 if it is empty)
  const int32_t* others;                       // LDS: pages of sequences 64 ..
  int n_seqs, lane;
  ChunkLengths len;
  float per_big, per_small;
  enum Kind { kGeneral, kGrid, kFitted } kind;    // which cut it is; kGrid: slot u is chunk u / n_seqs of sequence u % n_seqs
  int others0;                                 // kGrid, kFitted: chunks behind the first ones, of the sequences up to this lane's
  int size0;                                   // kFitted: pages a chunk
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
  // ceil(x / d) for 0 <= x <= 2^24 (every page count) and d >= 1, by the reciprocal of d; x / d <= 2^22, so that the quotient is
  // off by one at most
  static __device__ __forceinline__ int div_up(int x, int d, float inverse) {
    const int q = static_cast<int>(static_cast<float>(x) * inverse);
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
  __device__ __forceinline__ int cut(const DecodeArgs& a, bool fp16_values, bool grouped) {
    pages0 = lane < n_seqs ? pages_of_len(min(pages0, a.max_seq_len)) : 0;
    kind = kGeneral;
    if (a.fit_chunks > 0) {
      const int slots = cut_resident(a, fp16_values ? kPairedFp16 : (grouped ? kPairedGrouped : kPairedQuantized));
      if (slots > 0) return slots;
      if (a.spare_chunks == 0) return cut_as_host(a);
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
  // The host's chunks, as if the grid were (sequence, chunk).
  __device__ __forceinline__ int cut_as_host(const DecodeArgs& a) {
    kind = kGrid;
    len.big = a.pages_per_chunk;
    len.small = a.pages_small;
    len.n_big = a.n_big;
    find_chunks();
    others0 = wave_prefix(max(n0 - 1, 0));
    return n_seqs * a.n_chunks;
  }
  // Chunks that are resident together are as long as the longest of the host's; with longer ones, work-groups that come as others go are
  // the better balance (48 x 3K .. 12K tokens in chunks of 68 pages 155 us, by the general rule 143).  Up to kShort pages, a chunk's start
  // and end are worth an empty place.
  static constexpr int kLongest = 64, kShort = 12;
  // Whether more chunks than units, but by less than a third, are above half of the longest one (n0, size0): those few units with two
  // of them end last, at twice the time of the others.  Above kPaired* pages chunks cut without a look at the places are the better ones
  // then; shorter ones, and more units with two, are no slower.  Microseconds, 8 KV heads, as the host or the general rule cuts ->
  // resident together:
  //   fp16 values: 33 x 7700 .. 8200 tokens 127 -> 151;  20 x 8192 + 13 x 600 77 -> 86;  36 x 3700 .. 4100 74 -> 80;  20 x 3584 + 15 x 600
  //     (chunks of 14 pages) 41.5 -> 43.8;  36 x 1350 .. 1500 32.6 -> 33.0;  35 x 900 .. 1800 34 -> 30;  44 x 7700 .. 8200, a third, 166 -> 158
  //   4-bit values: 33 x 7700 .. 8200 75 -> 83;  36 x 3700 .. 4100 47.0 -> 47.0;  36 x 2700 .. 3000 37.9 -> 37.6;  20 x 4096 + 15 x 600 37.5 -> 31.8
  //   grouped quantizer, 4-bit values: 36 x 2170 .. 2300 45 -> 50;  40 x 1920 .. 2048 43.4 -> 41.4
  static constexpr int kPairedFp16 = 12, kPairedGrouped = 16, kPairedQuantized = 28;   // (the two latter: quantized values)
  __device__ __forceinline__ bool pairs_up_few() const {
    const int top = static_cast<int>(wave_max_u32(static_cast<uint32_t>(n0 > 0 ? size0 : 0)));
    const int over = wave_sum(2 * size0 > top ? n0 : 0);
    return over > units && 3 * over < 4 * units;
  }
  // The cut of a launch of at most 64 sequences that leaves places on the compute units when every sequence has one work-group.
  // If all sequences are equally long nothing has to be counted, and if they are as long as the host was told its chunk
  // lengths are the measured ones.  If lengths differ, what matters is that all chunks start at once and that the two work-groups of a compute unit
  // are not both long ones (kFitted): the shortest whole rounds with no more chunks than are resident together, a sequence's
  // chunks alike, and locate_fitted() says who takes which.  Returns the slots that may have a chunk, 0 if neither will do.
  // Measured (8 KV heads, 4 query heads each, microseconds: chunks cut on the host, or here by chunk_lengths() from 48 pages a
  // share on, and dealt out chunk by chunk -> this):
  //   32 x 512 .. 8K tokens 70.9 -> 61.4, 3+3-bit keys and 2-bit values 41.6 -> 35.1 (with fewer instructions a page);  8 x 2K .. 30K, 4-bit values 54.1 -> 41.8
  //   grouped quantizer: 12 x 1K .. 16K 80.8 -> 52.9, 8 heads and 4-bit values 81.2 -> 47.2;  20 x 5K .. 10K, 2-bit values 50.8 -> 39.7
  //   6 x 500 .. 12K 36.4 -> 27.1;  30 x 300 .. 2500 29.3 -> 25.2;  16 x 4K .. 32K 142.8 -> 114.3;  8 x 4K .. 8K, 32 KV heads 82.1 -> 77.0
  //   alike: 16 x 2K with a max_seq_len of 32K 20.7 -> 20.8, 16 x 8K 60.0 -> 59.4, 31 x 3000 43.5 -> 43.5;  8 x 8K, 32 KV heads 109.4 -> 109.0
  __device__ __forceinline__ int cut_resident(const DecodeArgs& a, int paired_long) {
    const int max_pages = pages_of_len(a.max_seq_len);
    const int first_pages = uni(pages0);
    if (__builtin_amdgcn_ballot_w64(lane < n_seqs && pages0 != first_pages) == 0) {
      if (first_pages == max_pages) return cut_as_host(a);
      // Shorter ones: as many chunks as there are places -- unless, with one chunk each, a unit has two sequences and most have one
      // (33 x 8000 tokens with a max_seq_len of 8200: 144 us, the host's 44 pages a chunk 129; 36 x 3000 60 and 55; 44 sequences 1 % the other
      // way, and up to 12 pages 33 x 1500 31.0 and 31.4, with 4-bit values 22.5 and 26.1), or chunks are too long (44 x 12000 227 and 208).
      const int n = a.fit_chunks / n_seqs, c = max(kWaveRound, whole_rounds((first_pages + n - 1) / n));
      if ((n == 1 && c > kShort && 3 * n_seqs < 2 * a.fit_chunks) || c > kLongest) return 0;
      kind = kGrid;
      len.big = len.small = c;
      len.n_big = max_pages;
      find_chunks();
      others0 = (lane + 1) * (n0 - 1);
      return n_seqs * uni(n0);
    }
    // (at most kBalancedFan chunks of the longest sequence there is: by max_seq_len, 8 x 1K .. 8K tokens with one of 128K had chunks of
    // 32 pages where 8 do, 42.5 us instead of 25.5)
    const int total = wave_sum(pages0), longest = static_cast<int>(wave_max_u32(static_cast<uint32_t>(pages0)));
#pragma unroll 1
    for (int c = whole_rounds(max((total + a.fit_chunks - 1) / a.fit_chunks, (longest + kBalancedFan - 1) / kBalancedFan)); c <= kLongest; c += 2 * kWaveRound) {
      // two lengths at a time, their counts in the halves of a word
      const int n = lane < n_seqs ? max(1, div_up(pages0, c, __builtin_amdgcn_rcpf(static_cast<float>(c)))) : 0;
      const int m = lane < n_seqs ? max(1, div_up(pages0, c + kWaveRound, __builtin_amdgcn_rcpf(static_cast<float>(c + kWaveRound)))) : 0;
      const int both = wave_sum(n | (m << 16));
      const bool first = (both & 0xffff) <= a.fit_chunks;
      if (first || (c < kLongest && (both >> 16) <= a.fit_chunks)) {
        n0 = first ? n : m;
        units = kComputeUnits / a.n_kv_heads;
        const int chunks0 = max(n0, 1);                                // (no chunks past the last sequence)
        size0 = div_up(pages0, chunks0, __builtin_amdgcn_rcpf(static_cast<float>(chunks0)));
        // Alike to the page, not in whole rounds: the places are done together (36 x 400 .. 1500 tokens 23.6 us against 25.6, 20 x 11K .. 12K 95.9
        // against 102).  But where no sequence has more than three rounds and no unit two first chunks, rounds of 2 + 1 are three a unit and
        // 6 + 6 pages are four: 28 x 750 .. 1500 tokens 23.6 -> 22.1, with 4-bit values 20.5 -> 18.6, grouped quantizer 29.9 -> 26.7.
        if ((first ? c : c + kWaveRound) == 2 * kWaveRound && longest <= 3 * kWaveRound && n_seqs <= units) size0 = whole_rounds(size0);
        if ((first ? c : c + kWaveRound) > paired_long && pairs_up_few()) return 0;
        kind = kFitted;
        others0 = wave_prefix(max(n0 - 1, 0));
        return 2 * units;
      }
    }
    return 0;
  }
  // Slot u takes its place on compute unit u % units of its KV head, if work-groups are handed out in order (which they are:
  // of 512 work-groups i and i + 256 shared a unit, 256 times of 256; nothing but time hangs on it; with KV heads that do not divide
  // 256 the partner is a neighbour's: 5, 6, 7, 12 and 24 heads, 500 .. 8K tokens, fp16 values 64 -> 56, 67 -> 54, 68 -> 51 us and the like,
  // 6 % faster at least).  The first slots have the sequences' first chunks; of the others, the longest chunk goes to the unit
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
    if (kind == kGrid) {
      chunk = uni(static_cast<int>(static_cast<float>(u) * __builtin_amdgcn_rcpf(static_cast<float>(n_seqs))));   // off by one at most
      chunk += u - chunk * n_seqs >= n_seqs ? 1 : (u - chunk * n_seqs < 0 ? -1 : 0);
      seq = u - chunk * n_seqs;
      return chunk < __builtin_amdgcn_readlane(n0, seq);
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
      chunks_before = seq + __builtin_amdgcn_readlane(others0, seq) - (n_chunks - 1);
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

}  // namespace
}  // namespace pq
