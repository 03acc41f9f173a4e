// Attention kernel on the matrix cores: the uniform angle grid, and the grouped angle quantizer from three query heads per
// KV head on (whose score walk, GroupedWalk, has its own description).
//
// Scores, uniform grid.  A key pair is reconstructed as rho~ (cos theta~, sin theta~), rho~ = s (c + 1/2) + z
// (Section 3.2), and the score is sum over pairs of q . k~.  Written with the four products
//     q_x s, q_y s, q_x z, q_y z          (per pair and page: the query side)
//     c' cos, c' sin, cos, sin, c' = c + 1/2   (a function of the packed symbol alone: the key side)
// it is a contraction over 4 terms a pair.  The key side is a table of 2^(r+t) symbols that does not
// depend on the query, the page or the head: 16 bytes a symbol, each of the four numbers as two
// fp16 (high part, low part: 22 bits and more), and one 128-bit LDS read of it IS an operand of
// v_mfma_f32_16x16x32_f16 -- lane (token, pair block), 8 of the 32 products summed.  The query
// side fills the other operand: 16 columns = 8 query heads x {high, low} fp16 part of the
// products, so a product of an fp16 query and an fp16 parameter (22 bits) enters exactly, and
// any group of 1 to 8 query heads costs the same.  Accumulation is fp32, restarted every 4
// instructions (16 pairs) to keep the partial sums small: measured against float64 the scores
// are as close as those of one fp32 multiply-add per pair.
//
// Values.  The accumulator layout of the scores -- lane (column, four consecutive tokens) -- is
// the operand layout of the next product: probabilities go from score to value product in
// registers, as high and low fp16 parts in the columns that held the query's parts (split_pair; the
// row sums of both parts are added at the end).  fp16 value rows are transposed pairwise with
// v_perm_b32; quantized values need no conversion at all (a masked code is an fp16 denormal).
//
// What bounds it.  Per page (128 tokens of one KV head) a wavefront issues about 1090 vector
// instructions with fp16 values and up to 4 heads, and 196 matrix instructions, 36 of them for the
// values; one multiply-add per (head, pair, token) and (head, dim, token) on the vector unit took 2200.
// With fp16 values a page is 41 KB, 3600 cycles of a compute unit's share of HBM: memory-bound
// (16 x 32K tokens, 4 query heads per KV head: 209 - 210 us, 6.5 TB/s; 217 on the vector unit).  With
// quantized values the page is 11 - 17 KB and its instructions are the longer side, with the clock: a wavefront takes as many cycles a
// page when every page comes from the caches as from memory, but the clock falls from 2.0 GHz to 1.4 - 1.6 -- power.  Read from the
// shader clock in the kernel, 16 x 32K tokens with 4-bit values, 4 heads, cycles a page of a wavefront beside one other:
//   scores   5650   322 vector, 128 matrix and 144 LDS instructions
//   softmax  1730   about 140 vector
//   values   2340   264 vector, 32 matrix (230 of the former bring codes to their fields)
// 9700 in all, 4850 a SIMD; with 10000 at the start of each of four chunks a SIMD, 176000 cycles a launch, 1.37 GHz in that run.  Of
// those, vector and matrix instructions take 69 % of a SIMD's issue slots, the matrix pipe is busy for 46 %, LDS for 51 %: none
// is full, and two wavefronts do not hide one another's chains (alone on its SIMD, a wavefront took 8400 cycles when two took 10700).
// What helped is less to issue: one wait for four operands instead of four, two steps' queries in one LDS read, lane constants kept
// where the registers allow it, denominators and zero-point sums by one multiply-add a token, the next page's scales found among
// the values: 106 vector instructions, 10700 -> 9600 cycles, 124 -> 120 us.  (The values of one page beside the scores of
// the next one, in one instruction stream: the same issue slots, 11200 cycles, +2 %.)
//
// The table is kept 16 times in LDS, copy l in the 16-byte column l of a 256-byte row, and lane l
// reads copy l % 16: reads of 16 lanes touch every bank once whatever the symbols are.  64 KB for
// 8-bit symbols, 16 KB for 6-bit ones: two work-groups per compute unit.
#pragma once
#include "pq_decode_sched.hpp"

namespace pq {

// Launchers (pq_decode_matrix.hip, one per value width).  `w` = r + t; a.n_heads query heads (1 .. 8) from a.head0 on.
// `roles` picks the name the launch runs under.  They return
// false, and launch nothing, for a width without a kernel; launch errors are left to hipGetLastError().
bool launch_attention_matrix_v16(int w, bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st);
bool launch_attention_matrix_v4(int w, bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st);
bool launch_attention_matrix_v2(int w, bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st);
// Grouped angle quantizer (pq_decode_grouped.hip, one per value width), rt = 10 r + t; and its raw scores alone.
bool launch_attention_grouped_v16(int rt, const DecodeArgs& a, dim3 grid, hipStream_t st);
bool launch_attention_grouped_v4(int rt, const DecodeArgs& a, dim3 grid, hipStream_t st);
bool launch_attention_grouped_v2(int rt, const DecodeArgs& a, dim3 grid, hipStream_t st);
bool launch_scores_grouped(int rt, const DecodeArgs& a, dim3 grid, hipStream_t st);

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kMaxHeads = 8;            // query heads of one pass: columns h (high part) and 8 + h (low part)

// ---- key-side table ---------------------------------------------------------------------------
// Entry of symbol (a << r) | c: fp16 {c' cos, c' sin, cos, sin} high parts, then their low parts,
// all scaled by 2^kTableShift (keeps the low parts out of the denormal range; c' <= 31.5).
constexpr int kTableShift = 10;

constexpr uint16_t half_bits(double v) {          // nearest fp16, ties to even; |v| < 65504
  const uint16_t sign = v < 0 ? 0x8000u : 0u;
  if (v < 0) v = -v;
  int e = -14;                                     // quantum 2^(e - 10): fixed below 2^-14
  double quantum = 1.0 / 16777216.0;
  while (v >= quantum * 2048.0) {
    quantum *= 2.0;
    ++e;
  }
  const double n = v / quantum;
  int64_t k = static_cast<int64_t>(n);
  const double rest = n - static_cast<double>(k);
  if (rest > 0.5 || (rest == 0.5 && (k & 1))) ++k;
  // k quanta: 1024 <= k <= 2048 in the normal range (2048 carries into the exponent field by itself)
  return static_cast<uint16_t>(sign | (k < 1024 ? k : ((static_cast<int64_t>(e) + 14) << 10) + k));
}
constexpr double half_value(uint16_t b) {
  const int e = (b >> 10) & 31;
  double v = e == 0 ? (b & 1023) / 1024.0 : 1.0 + (b & 1023) / 1024.0;
  for (int i = e == 0 ? 1 : e; i < 15; ++i) v *= 0.5;
  for (int i = 15; i < e; ++i) v *= 2.0;
  return (b & 0x8000) ? -v : v;
}
constexpr double cos_series(double x) {            // |x| <= pi
  double term = 1.0, sum = 1.0;
  for (int k = 1; k <= 15; ++k) {
    term *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    sum += term;
  }
  return sum;
}
template <int W>
struct KeyTables {
  uint32_t word[3][1 << W][4];
};
// the bit allocations of a width, in table order
constexpr int kTableRadiusBits[2][3] = {{3, 4, 2}, {4, 5, 3}};       // W = 6: (3,3) (4,2) (2,4); W = 8: (4,4) (5,3) (3,5)
template <int W>
constexpr KeyTables<W> make_key_tables() {
  constexpr double kPi = 3.14159265358979323846;
  KeyTables<W> t = {};
  for (int i = 0; i < 3; ++i) {
    const int rb = kTableRadiusBits[W == 8][i], tb = W - rb;
    for (int a = 0; a < (1 << tb); ++a) {
      const double th = -kPi + (a + 0.5) * (2.0 * kPi / (1 << tb));
      // sin from the cosine of the angle a quarter turn back, kept within [-pi, pi]
      const double cs = cos_series(th), sn = th >= -kPi / 2 ? cos_series(th - kPi / 2) : -cos_series(th + kPi / 2);
      for (int c = 0; c < (1 << rb); ++c) {
        const double scale = 1 << kTableShift;
        const double x[4] = {(c + 0.5) * cs * scale, (c + 0.5) * sn * scale, cs * scale, sn * scale};
        uint16_t h[8] = {};
        for (int k = 0; k < 4; ++k) {
          h[k] = half_bits(x[k]);
          h[4 + k] = half_bits(x[k] - half_value(h[k]));
        }
        for (int k = 0; k < 4; ++k) t.word[i][(a << rb) | c][k] = h[2 * k] | (static_cast<uint32_t>(h[2 * k + 1]) << 16);
      }
    }
  }
  return t;
}
__device__ const KeyTables<8> key_tables8 = make_key_tables<8>();
__device__ const KeyTables<6> key_tables6 = make_key_tables<6>();

constexpr int kTableRow = 256;           // bytes of a symbol in LDS: 16 copies of its entry
template <int W>
__device__ __forceinline__ const uint4* key_table(int index) {
  if constexpr (W == 8) return reinterpret_cast<const uint4*>(&key_tables8.word[index][0][0]);
  else return reinterpret_cast<const uint4*>(&key_tables6.word[index][0][0]);
}
// Thread t loads the entry of symbol t % 2^W and stores it to as many of the symbol's copies as fall to it,
// each lane starting at a copy of its own (16 lanes write to all banks).  A work-group barrier must
// follow before the table is read.
template <int W>
__device__ __forceinline__ uint4 fetch_key_entry(const uint4* src, int tid) { return src[tid & ((1 << W) - 1)]; }
template <int W, int NT>
__device__ __forceinline__ void store_key_entry(uint8_t* lut, const uint4& entry, int tid) {
  constexpr int kCopies = 16 * (1 << W) / NT;        // of a thread
  static_assert(kCopies * NT == 16 * (1 << W), "whole copies");
  uint8_t* const row = lut + (tid & ((1 << W) - 1)) * kTableRow;
  const int first = tid + (tid >> W) * kCopies;
#pragma unroll
  for (int i = 0; i < kCopies; ++i) *reinterpret_cast<uint4*>(row + ((first + i) & 15) * 16) = entry;
}

// ---- query side -------------------------------------------------------------------------------
// Columns of the query operand.  NH = 8 (5 to 8 query heads): column = 8 part + head.  NH = 4 (1 to
// 4 heads): column = 8 part + 4 half + head, where half 0 carries the pairs of the first two steps of
// every four and half 1 the others (zeros elsewhere) -- the partial sums of a column are half as long.
template <int NH>
__device__ __forceinline__ int column_head(int col) { return col & (NH - 1); }

// The pass's query in LDS, [pair][column] with 8 bytes an entry: q = (q_x, q_y) as fp16, and
//   fp16 queries: q again in low-part columns, 0 in high-part ones;
//   fp32 queries: what q's rounding to fp16 left over, in low-part columns, 0 in high-part ones.
// Powers of two keep the products inside fp16 and lose nothing: each head is scaled so that its
// largest element is in [2^9, 2^10), then each pair so that this holds for the pair's largest element
// of any head, and the pair's radius parameters are scaled the other way -- what then is below fp16's
// normal range is the parameter of a pair whose products are 2^-18 of the page's largest, or an
// element 2^-23 of what another head has in the same pair.  (With the heads' scale alone a page with
// a radius of 30000 beside ones of 0.3, in a pair where the query is small, had an error of 9.3e-5; so,
// and with fp32 arithmetic, 1.6e-7.)  The 16 pairs of a block are followed by 128 bytes of padding
// (the four lane rows read four blocks at once).
constexpr int kQueryTop = 9, kParamTop = 4;
constexpr int kQueryBlock = 16 * 16 * 8 + 128;
struct QueryShared {
  __attribute__((aligned(16))) uint8_t pairs[kBlocks * kQueryBlock];
};
// As loaded, so that nothing waits for it before store_query_heads(): thread = (head tid / 32, pairs
// 2 (tid % 32), + 1), x coordinates first; heads from n_heads on are zero.
struct QueryFetch {
  uint32_t w[4];
  template <bool Q32>
  __device__ __forceinline__ float value(int comp, int e) const {
    return Q32 ? u2f(w[2 * comp + e]) : static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w[comp] >> (16 * e))));
  }
  __device__ __forceinline__ QueryFetch widened() const {     // fp16 elements as fp32 ones
    return {{f2u(value<false>(0, 0)), f2u(value<false>(0, 1)), f2u(value<false>(1, 0)), f2u(value<false>(1, 1))}};
  }
};
template <bool Q32>
__device__ __forceinline__ QueryFetch fetch_query_heads(const DecodeArgs& a, int64_t q_at, int tid) {
  QueryFetch f = {};
  const int h = tid >> 5;
  if (h < a.n_heads) {
    const int64_t at = q_at + h * kHeadDim + (tid & 31) * 2;
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      if constexpr (Q32) __builtin_memcpy(f.w + 2 * comp, static_cast<const float*>(a.q) + at + comp * kPairs, 8);
      else __builtin_memcpy(f.w + comp, static_cast<const __half*>(a.q) + at + comp * kPairs, 4);
    }
  }
  return f;
}
// A query's elements as a thread has them, and the powers of two they are multiplied with: brings the head's
// largest element, then the pair's largest of any head, into [2^T, 2^(T + 1)).
template <int NH, bool Q32, int T>
struct QueryScale {
  float v[2][2];                                             // [pair][coordinate]
  int shift, up[2];                                          // of the head, of the pair
  // `pair_down`: what the parameters of each pair are to be multiplied with.  `exponents` is scratch.  Holds
  // one work-group barrier; up is set in threads of heads below NH only.
  __device__ __forceinline__ QueryScale(const QueryFetch& f, float* pair_down, uint16_t (*exponents)[NH], int tid) {
    uint32_t high[2];                                        // of the pair's two, as bits
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      v[e][0] = f.value<Q32>(0, e);
      v[e][1] = f.value<Q32>(1, e);
      high[e] = max(f2u(v[e][0]) & 0x7fffffffu, f2u(v[e][1]) & 0x7fffffffu);
    }
    const uint32_t top = half_wave_max_u32(max(high[0], high[1]));
    shift = min(T + 127 - static_cast<int>(top >> 23), 126);
    const int h = tid >> 5, j0 = (tid & 31) * 2;
    // exponents after the head's scale, the largest 64 + T
    if (h < NH) {
#pragma unroll
      for (int e = 0; e < 2; ++e) exponents[j0 + e][h] = static_cast<uint16_t>(max(0, static_cast<int>(high[e] >> 23) + shift - 127 + 64));
    }
    __syncthreads();
    if (h >= NH) return;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      uint32_t of_heads[NH / 2];
      __builtin_memcpy(of_heads, exponents[j0 + e], NH * 2);
      uint32_t most2 = of_heads[0];
#pragma unroll
      for (int o = 1; o < NH / 2; ++o) most2 = max_u16x2(most2, of_heads[o]);
      const int most = static_cast<int>(max(most2 & 0xffffu, most2 >> 16));
      up[e] = most == 0 ? 0 : 64 + T - most;
      if (h == 0) pair_down[j0 + e] = most == 0 ? 0.f : __builtin_ldexpf(1.f, -up[e]);   // (not in any product: no say in the page's scale)
    }
  }
  __device__ __forceinline__ float scaled(int e, int comp, float sign) const { return sign * __builtin_ldexpf(v[e][comp], shift + up[e]); }
};
// `shifts`: the power of two each head was multiplied with.  Holds the barrier of QueryScale.
// (Both coordinates of a pair in one thread: 8 wide stores instead of 48 of 16 bits, and one 16-byte read of
// the other heads' exponents.)
template <int NH, bool Q32>
__device__ __forceinline__ void store_query_heads(QueryShared& q, int* shifts, float* pair_down, uint16_t (*exponents)[NH],
                                                  const QueryFetch& f, float sign, int tid) {
  const QueryScale<NH, Q32, kQueryTop> x(f, pair_down, exponents, tid);
  const int h = tid >> 5, j0 = (tid & 31) * 2;
  if (h >= NH) return;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int j = j0 + e, kk = j & 15;
    f16x2 hi, rest;
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      const float v = x.scaled(e, comp, sign);
      hi[comp] = static_cast<_Float16>(v);
      rest[comp] = Q32 ? static_cast<_Float16>(v - static_cast<float>(hi[comp])) : hi[comp];
    }
    uint8_t* const at = q.pairs + (j >> 4) * kQueryBlock + kk * 128 + h * 8;
#pragma unroll
    for (int half = 0; half < 8 / NH; ++half) {
      const bool here = NH == 8 || ((kk >> 1) & 1) == half;
      const uint32_t hw = here ? __builtin_bit_cast(uint32_t, hi) : 0u, rw = here ? __builtin_bit_cast(uint32_t, rest) : 0u;
      *reinterpret_cast<u32x2*>(at + half * NH * 8) = u32x2{hw, 0u};
      *reinterpret_cast<u32x2*>(at + half * NH * 8 + 64) = u32x2{hw, rw};
    }
  }
  if ((tid & 31) == 0) shifts[h] = x.shift;
}

__device__ __forceinline__ f16x2 to_half2(float x, float y) { return __builtin_convertvector((f32x2{x, y}), f16x2); }
__device__ __forceinline__ uint32_t h2u(f16x2 h) {
  uint32_t u;
  __builtin_memcpy(&u, &h, 4);
  return u;
}
__device__ __forceinline__ f16x2 u2h(uint32_t u) {
  f16x2 h;
  __builtin_memcpy(&h, &u, 4);
  return h;
}
// A probability's fp16 parts, of x in [0, 2^(15 - S)]: the nearest fp16 to 2^S x in the lanes of
// high-part columns (part = {0, 2^S}), 2^kLowShift times what that leaves over -- 2^3 at most -- in
// those of low-part ones (part = {-2^-S, 2^(S + kLowShift)}).  Accumulator rows are scaled back when a
// chunk ends.  The two carry 22 bits until the high part is below fp16's normal range, a bit less for
// every power of two below that: with S = 15 a token keeps 22 bits of its weight down to 2^-29 of the
// largest, and vanishes at 2^-51.  (Where the output hangs on weights of 2^-25 beside an attention sink
// its error is 4e-7 so, 5e-7 with fp32 weights, and was 3.3e-3 with both parts on one scale and the
// largest at 2^4.)  2^S is not in the exponential's argument, which would be rounded at that size:
// flat softmaxes 1.6e-7 with 2^7 there, 1.3e-7 so (fp32 throughout: 1.4e-7).
constexpr int kLowShift = 12;
template <int S>
__device__ __forceinline__ f32x2 split_part(bool low) {
  constexpr float kUp = static_cast<float>(1 << S);
  return low ? f32x2{-1.f / kUp, kUp * (1 << kLowShift)} : f32x2{0.f, kUp};
}
template <int S>
__device__ __forceinline__ uint32_t split_pair(float x0, float x1, f32x2 part) {
  constexpr float kUp = static_cast<float>(1 << S);
  const f16x2 h = {static_cast<_Float16>(fmaf(x0, kUp, 0.f)), static_cast<_Float16>(fmaf(x1, kUp, 0.f))};
  const f16x2 r = {static_cast<_Float16>(fmaf(fmaf(static_cast<float>(h.x), part.x, x0), part.y, 0.f)),
                   static_cast<_Float16>(fmaf(fmaf(static_cast<float>(h.y), part.x, x1), part.y, 0.f))};
  return h2u(r);
}
// Sums of two accumulators' parts, the high ones in lanes 0 - 31, the low ones (already scaled back) in lanes
// 32 - 63: of x in lanes 0 - 31, of y in the others.  Where a value is infinite the high part is what the product is; a low
// part may be zero or negative there.
__device__ __forceinline__ float sum_parts(float x, float y) {
  auto r = __builtin_amdgcn_permlane32_swap(f2u(x), f2u(y), false, false);
  const float high = u2f(r[0]), low = u2f(r[1]);
  return __builtin_isinf(high) ? high : high + low;
}
constexpr int kScaleTop = 3;
__device__ __forceinline__ f16x8 as_operand(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const u32x4 v = {a, b, c, d};
  f16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}
// {a, b, a, b}, the second half as one 64-bit move
__device__ __forceinline__ f16x8 twice(uint32_t a, uint32_t b) {
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  const uint64_t ab = __builtin_bit_cast(uint64_t, (u32x2{a, b}));
  uint64_t again = ab;
  asm("" : "+v"(again));                          // (or the halves are copied one by one)
  return __builtin_bit_cast(f16x8, (u64x2{ab, again}));
}
__device__ __forceinline__ f16x8 as_operand(const uint4& v) { return as_operand(v.x, v.y, v.z, v.w); }

// A page's radius parameters, one pair a lane, times `down` (of the pair) and the power of two 2^k that
// brings the largest into [2^4, 2^5); sets k.
__device__ __forceinline__ uint32_t scale_page_params(uint32_t par, float down, int& k) {
  const f16x2 p = u2h(par);
  const float s = static_cast<float>(p.x) * down, z = static_cast<float>(p.y) * down;
  const uint32_t e = wave_max_u32(max(f2u(s) & 0x7fffffffu, f2u(z) & 0x7fffffffu)) >> 23;
  k = min(100, kParamTop + 127 - static_cast<int>(e));               // (a page of zeros: anything)
  return h2u(to_half2(__builtin_ldexpf(s, k), __builtin_ldexpf(z, k)));
}

__device__ __forceinline__ float max2(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// ---- scores of a page ---------------------------------------------------------------------------
// Which tokens of a page are batch t of 16, matrix row m (a result lane of row r holds m = 4 r .. 4 r + 3):
// the order the values of the same lane come in.
enum class TokenOrder {
  kRows,       // fp16 values, four consecutive rows a load: token 16 ((t + rot) % 8) + 4 (m % 4) + m / 4
  kPlain,      // 4-bit values (units of 4 tokens): token 16 ((t + rot) % 8) + m
  kUnits8      // 2-bit values (units of 8 tokens): token 32 (t / 2) + 8 (m / 4) + 4 (t % 2) + m % 4
};
constexpr TokenOrder token_order(int v_bits) {
  return v_bits == 16 ? TokenOrder::kRows : (v_bits == 4 ? TokenOrder::kPlain : TokenOrder::kUnits8);
}
template <TokenOrder O>
__device__ __forceinline__ int batch_token(int t, int rot) {     // wavefront-uniform part
  return O == TokenOrder::kUnits8 ? 32 * (t >> 1) + 4 * (t & 1) : 16 * ((t + rot) & 7);
}
template <TokenOrder O>
__device__ __forceinline__ int row_token(int m) {                // part of the matrix row
  return O == TokenOrder::kRows ? 4 * (m & 3) + (m >> 2) : (O == TokenOrder::kPlain ? m : 8 * (m >> 2) + (m & 3));
}

// Sums of a head's columns.  NH = 8: s[t] of all batches in both columns of a head.  NH = 4: the columns of half 0
// keep batches 0 .. 3, those of half 1 batches 4 .. 7, in s[0] .. s[3].
template <int NH>
__device__ __forceinline__ void fold_columns(f32x4 (&s)[8], bool half) {
  if constexpr (NH == 4) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) s[t][i] += dpp_of<0x124>(s[t][i]);     // row_ror:4: the neighbour in (part, half)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[j][i] = half ? s[4 + j][i] : s[j][i];
        s[j][i] += dpp_of<0x128>(s[j][i]);                               // row_ror:8: the other two
        asm volatile("" : "+v"(s[j][i]));                                // (here, as one instruction, not behind the next branch)
      }
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[t][i] += dpp_of<0x128>(s[t][i]);
        asm volatile("" : "+v"(s[t][i]));
      }
  }
}
// Scores of the residual group (un-quantized fp16 keys, rows past nv_res read as zero), not yet folded: a key row
// is an operand as it lies in memory, 32 dims per instruction.  query(kd, j0, e): the column's query of dims
// 32 kd + 8 row + 2 e, + 1 -- one coordinate of pairs j0 + 2 e, + 1 -- as an fp16 pair.
template <TokenOrder O, typename Query>
__device__ __forceinline__ void residual_products(f32x4 (&s)[8], const __half* rows, int nv_res, int rot, int lane, Query query) {
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(rows, static_cast<uint32_t>(nv_res) * (kHeadDim * 2));
  const int row = lane >> 4, col = lane & 15;
  f16x8 q8[4];
#pragma unroll
  for (int kd = 0; kd < 4; ++kd) {
    const int j0 = 32 * (kd & 1) + 8 * row;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = query(kd, j0, e);
    q8[kd] = as_operand(w[0], w[1], w[2], w[3]);
  }
  const uint32_t voff = row_token<O>(col) * (kHeadDim * 2) + row * 16;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const uint32_t soff = static_cast<uint32_t>(batch_token<O>(t, rot)) * (kHeadDim * 2);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 lo = zero, hi = zero;
#pragma unroll
    for (int kd = 0; kd < 4; ++kd) {
      const f16x8 k_op = as_operand(buf_load16<kAuxCached>(rs, voff, soff + kd * 64));
      if (kd < 2) lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(k_op, q8[kd], lo, 0, 0, 0);
      else hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(k_op, q8[kd], hi, 0, 0, 0);
    }
    s[t] = lo + hi;
    if (t & 1) __builtin_amdgcn_sched_barrier(0);
  }
}

// One wavefront's key codes and parameters of a page, and the walk over them.  Operand lane =
// (token row l % 16, pair block l / 16), pair 16 (l / 16) + kk in step kk; result lane = (column
// l % 16, tokens 4 (l / 16) .. + 3).  The table reads run 4 or 8 instructions ahead (8 where there are registers for it); as a unit is used
// for the last time it is refilled with the next page's.
//
// kChain: steps after which the accumulators restart (16: never).  The instruction rounds once per
// pair, at the size of the running sum.  Error of a score against float64, 8 x 32K keys with
// outlier channels, as part of the scores' 2-norm (one fp32 multiply-add per pair: 9.3e-8):
// NH = 4 (whose columns carry half of the pairs each) with chains of 4: 9.5e-8, NH = 8 with 4:
// 1.05e-7, with 2: 9.5e-8.  The kernel takes 4 (its output's error, 4e-7 - 7e-7, is that of the
// exponentials) and none with quantized values (1e-5).  Raw scores that are handed out come from the
// token-lane kernel: fp32 queries and 5 to 8 heads would have 1.2e-7 from here where it has 9.2e-8.
// kAhead: half-steps (4 table reads each) between a read and its use.
template <int W, TokenOrder O, int NH, bool Q32, int kAhead, int kChain>
struct ScoreWalk {
  static constexpr int UB = 2 * W;
  static_assert(16 % kChain == 0, "steps of a chain");
  Unit<W / 2> cu[8];
  uint32_t par;                                 // {fp16 s, fp16 z} of pair `lane`
  f32x4 s[8], d[4], done[4];                    // sums, the chain under way, the chain before it
  f32x4 entry[kAhead + 1][4];
  // query and scaled parameters of the next steps: fetched early enough that waiting for them does not wait for the
  // table reads under way; step by step, or (kPairFetch) two steps at a time, half as many LDS operations
  static constexpr bool kPairFetch = kChain == 16;
  static constexpr int kFetched = kPairFetch ? 4 : 2;
  u32x2 qv[kFetched];
  uint32_t sz[kFetched];
  // Order of the half-steps: a chain's steps first for one half of the batches, then for the other, so
  // that four accumulators serve a chain; without restarts simply step by step.
  static constexpr int kOps = kChain == 16 ? 1 : kChain;   // query operands kept
  uint32_t q_op[kOps][2];
  f16x8 q_twice;                                // kOps = 1: the operand as a whole, made a half-step ahead
  uint32_t lane_lut, q_addr, par_put, par_get, voff_codes, low_mask, down_addr, table;

  __device__ __forceinline__ void init(const uint8_t* lut, const QueryShared& q, const float* pair_down, const uint32_t* params, int lane) {
    const int row = lane >> 4, col = lane & 15;
    table = lds_addr(lut);
    lane_lut = W == 8 ? col * 16 : table + col * 16;
    q_addr = lds_addr(q.pairs) + row * kQueryBlock + col * 8;
    down_addr = lds_addr(pair_down);
    par_put = lds_addr(params) + lane * 4;
    par_get = lds_addr(params) + row * 64;
    voff_codes = (row * kGroup + row_token<O>(col)) * UB;
    low_mask = col >= 8 ? 0xffffffffu : 0u;
  }
  __device__ __forceinline__ void load_unit_of(int t, __amdgpu_buffer_rsrc_t rc, int rot) {
    cu[t] = load_unit<W>(rc, voff_codes, static_cast<uint32_t>(batch_token<O>(t, rot)) * UB);
  }
  __device__ __forceinline__ void load_params(__amdgpu_buffer_rsrc_t rp, int lane) { par = buf_load4<kAuxCached>(rp, lane * 4, 0); }

  template <int KK>
  __device__ __forceinline__ f32x4 lookup(const Unit<W / 2>& u) const {
    uint32_t addr;
    if constexpr (W == 8) {
      // byte 0 from the lane's column, byte 1 from the symbol; where the table starts is the read's offset
      addr = __builtin_amdgcn_perm(u.d[KK >> 2], lane_lut, 0x0c0c0000u | ((4u + (KK & 3)) << 8)) + table;
    } else {
      constexpr int bit = KK * W, wi = bit >> 5, sh = bit & 31;
      uint32_t src = u.d[wi];
      int off = sh;
      if constexpr (sh + W > 32) {
        src = __builtin_amdgcn_alignbit(u.d[wi + 1], u.d[wi], sh);
        off = 0;
      }
      uint32_t sym;
      asm("v_bfe_u32 %0, %1, %2, %3" : "=v"(sym) : "v"(src), "n"(off), "n"(W));
      asm("v_lshl_add_u32 %0, %1, 8, %2" : "=v"(addr) : "v"(sym), "v"(lane_lut));
    }
    return *(const PQ_LDS f32x4*)static_cast<uintptr_t>(addr);
  }
  // after the operand of step `made` has been made: what is fetched into the place its query had
  static constexpr bool fetches_after(int made) { return kPairFetch ? (made & 1) && made + 3 < 16 : made + 2 < 16; }
  __device__ __forceinline__ void fetch_q(int kk) {
    constexpr int kMask = kFetched - 1;
    if constexpr (kPairFetch) {
      const u32x2 two = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(par_get + kk * 4);
      qv[kk & kMask] = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(q_addr + kk * 128);
      qv[(kk + 1) & kMask] = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(q_addr + (kk + 1) * 128);
      sz[kk & kMask] = two.x;
      sz[(kk + 1) & kMask] = two.y;
    } else {
      qv[kk & kMask] = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(q_addr + kk * 128);
      sz[kk & kMask] = *(const PQ_LDS uint32_t*)static_cast<uintptr_t>(par_get + kk * 4);
    }
  }
  __device__ __forceinline__ void fetch_after(int made) { fetch_q(kPairFetch ? made + 3 : made + 2); }
  // The step's query operand: q s and q z rounded to fp16 in high-part columns, what the rounding
  // left over -- exact for fp16 queries -- in low-part ones.
  __device__ __forceinline__ void make_query_operand(int kk) {
    const f16x2 p = u2h(sz[kk & (kFetched - 1)]);
    const f16x2 s_ = {p.x, p.x}, z_ = {p.y, p.y};
    const u32x2 v = qv[kk & (kFetched - 1)];
    const f16x2 q = u2h(v.x), ql = Q32 ? u2h(v.x & low_mask) : u2h(v.y);
    f16x2 ys = __builtin_elementwise_fma(q, s_, -(ql * s_));
    f16x2 yz = __builtin_elementwise_fma(q, z_, -(ql * z_));
    if constexpr (Q32) {
      ys = __builtin_elementwise_fma(u2h(v.y), s_, ys);
      yz = __builtin_elementwise_fma(u2h(v.y), z_, yz);
    }
    q_op[kk % kOps][0] = h2u(ys);
    q_op[kk % kOps][1] = h2u(yz);
    if constexpr (kOps == 1) q_twice = twice(q_op[0][0], q_op[0][1]);
  }
  // Half-step H: batches 4 half ..+3 of pair step kk.
  static constexpr int step_of(int H) { return H / (2 * kOps) * kOps + H % kOps; }
  static constexpr int half_of(int H) { return H / kOps % 2; }
  static constexpr bool ends_chain(int H) { return H >= 0 && step_of(H) >= kChain && step_of(H) % kChain == kChain - 1; }
  template <int H>
  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rc_nxt, int rot_nxt) {
    if constexpr (H < 32) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = half_of(H) * 4 + j;
        entry[H % (kAhead + 1)][j] = lookup<step_of(H)>(cu[t]);
        if constexpr (step_of(H) == 15) load_unit_of(t, rc_nxt, rot_nxt);
      }
    }
  }
  // LDS operations issued after the table reads of half-step H when that half-step begins: its matrix instructions wait
  // once, for their four operands together (a wait each took issue slots: a walk alone on its SIMD 4309 -> 3880 cycles,
  // two together 6364 -> 6115).
  static constexpr int younger(int H) {
    int n = 4 * (kAhead - 1);
    for (int h = H - kAhead; h < H; ++h)
      if (makes_operand(h) && fetches_after(step_of(h) + kOps)) n += 2;
    return n;
  }
  static constexpr bool makes_operand(int H) { return half_of(H) == 1 && step_of(H) + kOps < 16; }
  template <int H>
  __device__ __forceinline__ void steps(__amdgpu_buffer_rsrc_t rc_nxt, int rot_nxt) {
    if constexpr (H < 32) {
      constexpr int kk = step_of(H), half = half_of(H);
      if constexpr (kAhead > 1 && H >= kAhead) __builtin_amdgcn_s_waitcnt(0xc07f | younger(H) << 8);   // lgkmcnt alone
      issue<H + kAhead>(rc_nxt, rot_nxt);
      const f16x8 q8 = kOps == 1 ? q_twice : twice(q_op[kk % kOps][0], q_op[kk % kOps][1]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = half * 4 + j;
        f16x8 k_op;
        __builtin_memcpy(&k_op, &entry[H % (kAhead + 1)][j], 16);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        if constexpr (kk < kChain) {
          s[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k_op, q8, kk == 0 ? zero : s[t], 0, 0, 0);
        } else {
          d[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k_op, q8, kk % kChain == 0 ? zero : d[j], 0, 0, 0);
        }
      }
      // a finished chain is added a half-step later, when its results are there
      if constexpr (ends_chain(H - 1)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) s[half_of(H - 1) * 4 + j] += done[j];
      }
      if constexpr (ends_chain(H)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) done[j] = d[j];
      }
      // the step's operand has been used for the last time: make that of the same step of the next chain
      if constexpr (makes_operand(H)) {
        make_query_operand(kk + kOps);
        if constexpr (fetches_after(kk + kOps)) fetch_after(kk + kOps);
      }
      __builtin_amdgcn_sched_barrier(0);
      steps<H + 1>(rc_nxt, rot_nxt);
    }
  }
  // Puts the parameters in par, scaled by 2^k, where the walk reads them (and must have ended); returns k.  Without chains that
  // restart (quantized values) the caller does so before run(), otherwise run() does (fp16 values: one sequence of
  // 1000 tokens 13.3 us so, 13.45 with it before).
  static constexpr bool kPrepared = kChain == 16;
  __device__ __forceinline__ int prepare(int lane) {
    int k;
    *(PQ_LDS uint32_t*)static_cast<uintptr_t>(par_put) =
        scale_page_params(par, *(const PQ_LDS float*)static_cast<uintptr_t>(down_addr + lane * 4), k);
    return k;
  }
  // Scores of the page in cu, summed over the columns of a head and left as fold_columns() says, scaled by 2^(k of prepare(),
  // if run() calls it what is returned, + the head's query shift + kTableShift).  cu and par then hold the next page.
  __device__ __forceinline__ int run(__amdgpu_buffer_rsrc_t rc_nxt, __amdgpu_buffer_rsrc_t rp_nxt, int rot_nxt, int lane) {
    int k = 0;
    if constexpr (!kPrepared) {
      issue<0>(rc_nxt, rot_nxt);
      k = prepare(lane);
    }
    load_params(rp_nxt, lane);
    wave_lds_sync();
    if constexpr (kPrepared) issue<0>(rc_nxt, rot_nxt);
    fetch_q(0);
    fetch_q(kFetched / 2);
#pragma unroll
    for (int kk = 0; kk < kOps; ++kk) {
      make_query_operand(kk);
      if (fetches_after(kk)) fetch_after(kk);
    }
    if constexpr (kAhead == 2) issue<1>(rc_nxt, rot_nxt);
    static_assert(kAhead == 1 || kAhead == 2, "reads issued before the first half-step");
    __builtin_amdgcn_sched_barrier(0);
    steps<0>(rc_nxt, rot_nxt);
    if constexpr (kChain < 16) {
#pragma unroll
      for (int j = 0; j < 4; ++j) s[4 + j] += done[j];
    }
    fold_columns<NH>(s, lane & 4);
    wave_lds_sync();
    return k;
  }
  // Scaled with k = 0, table shift 0.
  __device__ __forceinline__ void residual(const __half* rows, int nv_res, int rot, int lane) {
    const uint32_t q0 = q_addr - (static_cast<uint32_t>(lane) >> 4) * kQueryBlock;
    residual_products<O>(s, rows, nv_res, rot, lane, [&](int kd, int j0, int e) {
      // the query in high-part columns, what its rounding to fp16 left over in low-part ones
      const uint32_t at = q0 + (j0 >> 4) * kQueryBlock + (j0 & 15) * 128;
      uint32_t x[2];
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const u32x2 v = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(at + (2 * e + o) * 128);
        const uint32_t pick = (v.x & ~low_mask) | (Q32 ? v.y : 0u);
        // without the pair's scale: no parameter carries the other half of it here
        const float down = *(const PQ_LDS float*)static_cast<uintptr_t>(down_addr + (j0 + 2 * e + o) * 4);
        const f16x2 picked = u2h(pick);
        x[o] = h2u(to_half2(static_cast<float>((kd >> 1) ? picked.y : picked.x) * down, 0.f));
      }
      return x[0] | (x[1] << 16);
    });
    fold_columns<NH>(s, lane & 4);
  }
};

// ---- scores of a page, grouped angle quantizer ------------------------------------------------------
// The angle levels belong to the page, so that the key side cannot be a table of symbols: every wavefront keeps
// the (cos, sin) of its page's 64 x 2^t angle states in LDS (built anew for each page) and makes the key's
// coordinates rho~ cos theta~, rho~ sin theta~ themselves, in fp32, each handed to the matrix unit as two fp16
// parts (24 bits).  The query side {q_x, q_y} is constant: high part in columns 0 - 7, what its rounding
// left over in columns 8 - 15.  One instruction takes two pairs of each of the four blocks; any group of 1 to 8 query
// heads costs the same.  About 11 vector instructions a symbol (1440 a page, table and fold included); with a table of the heads'
// products and fp32 multiply-adds (pq_decode_partials_kernel) it is 3 + heads, and values cost heads times as much as here.
//
// Scales: as on the uniform grid (QueryShared), each head's and then each pair's largest query element goes to the top and
// the pair's radius parameters are multiplied the other way, so that a key coordinate keeps its 24 bits until its products
// are 2^-15 of the page's largest of any head, whatever the radius is.  (With one scale a page a radius of 15000 beside ones
// of 2^-9, where the query is small in that pair, left the scores an error of 1.2e-5; 1.4e-7 so, as with fp32 multiply-adds.)
//
// Table entry of (pair j, state a): 8 bytes at (j / 2) 2^t 16 + 16 a + 8 ((j + j / 16) % 2): a block's two pairs of an
// instruction share a row, and neighbouring blocks, which are read together, use the other half of the banks.
constexpr int kGroupedTop = 13;                  // the page's radii, times their pairs' scales, are brought below 2^(kGroupedTop + 2)
constexpr int kGroupedQueryTop = 14;
constexpr int kGroupedQueryBlock = 8 * 16 * 8 + 128;
struct GroupedQuery {                            // [block][pair / 2 of the block][column]{x, y of the even pair, of the odd one}
  __attribute__((aligned(16))) uint8_t pairs[kBlocks * kGroupedQueryBlock];
};
// Scaled like the uniform grid's query (QueryScale); `shifts` says by which power of two a head was.
template <int NH>
__device__ __forceinline__ void store_grouped_query(GroupedQuery& q, int* shifts, float* pair_down, uint16_t (*exponents)[NH],
                                                    const QueryFetch& f, float sign, int tid) {
  const QueryScale<NH, true, kGroupedQueryTop> scale(f, pair_down, exponents, tid);
  const int h = tid >> 5, j0 = (tid & 31) * 2;
  if (h >= NH) return;
  uint32_t hi[2], lo[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float x = scale.scaled(e, 0, sign), y = scale.scaled(e, 1, sign);
    const f16x2 high = {static_cast<_Float16>(x), static_cast<_Float16>(y)};
    const f16x2 low = {static_cast<_Float16>(x - static_cast<float>(high.x)), static_cast<_Float16>(y - static_cast<float>(high.y))};
    hi[e] = __builtin_bit_cast(uint32_t, high);
    lo[e] = __builtin_bit_cast(uint32_t, low);
  }
  const int step = (j0 & 15) >> 1;
  uint8_t* const at = q.pairs + (j0 >> 4) * kGroupedQueryBlock + step * 128 + h * 8;
#pragma unroll
  for (int half = 0; half < 8 / NH; ++half) {
    const bool here = NH == 8 || (step >> 2) == half;
    *reinterpret_cast<u32x2*>(at + half * NH * 8) = here ? u32x2{hi[0], hi[1]} : u32x2{0u, 0u};
    *reinterpret_cast<u32x2*>(at + half * NH * 8 + 64) = here ? u32x2{lo[0], lo[1]} : u32x2{0u, 0u};
  }
  if ((tid & 31) == 0) shifts[h] = scale.shift;
}

template <int RB, int TB, TokenOrder O, int NH>
struct GroupedWalk {
  static constexpr int W = RB + TB, UB = 2 * W, NA = 1 << TB;
  static constexpr int kTableBytes = kPairs * NA * 8;
  static constexpr int kAhead = 3;                // steps (two table reads each) between a read and its use
  static constexpr int kRing = kAhead + 1;
  Unit<W / 2> cu[8];
  uint32_t par, tpar;                             // {fp16 s, fp16 z} of pair `lane`: radius, angle
  f32x4 s[8], d[4], done[4];
  f32x2 trig[kRing][2];                           // (cos, sin)
  float code[kRing][2];
  f32x4 rad;                                      // {s, z + s / 2} of a step's two pairs, scaled
  u32x2 qv;
  uint32_t row_even, row_odd, rad_put, rad_get, q_addr, voff_codes, build_even, build_odd, down_addr;

  __device__ __forceinline__ void init(const uint8_t* table, const GroupedQuery& q, const float* pair_down, const f32x2* radii, int lane) {
    down_addr = lds_addr(pair_down);
    const int row = lane >> 4, col = lane & 15;
    row_even = lds_addr(table) + row * (8 * NA * 16) + (row & 1) * 8;
    row_odd = row_even ^ 8u;
    rad_put = lds_addr(radii) + lane * 8;
    rad_get = lds_addr(radii) + row * 128;
    q_addr = lds_addr(q.pairs) + row * kGroupedQueryBlock + col * 8;
    voff_codes = (row * kGroup + row_token<O>(col)) * UB;
    const int pair = lane >> TB, state = lane & (NA - 1);
    build_even = lds_addr(table) + (pair >> 1) * (NA * 16) + state * 16 + (pair & 1) * 8;
    build_odd = build_even ^ 8u;
  }
  __device__ __forceinline__ void load_unit_of(int t, __amdgpu_buffer_rsrc_t rc, int rot) {
    cu[t] = load_unit<W>(rc, voff_codes, static_cast<uint32_t>(batch_token<O>(t, rot)) * UB);
  }
  __device__ __forceinline__ void load_params(__amdgpu_buffer_rsrc_t rp, int lane) {
    par = buf_load4<kAuxCached>(rp, lane * 4, 0);
    tpar = buf_load4<kAuxCached>(rp, lane * 4, kPairs * 4);
  }
  // (cos, sin) of the page's angle states theta~ = (a + 1/2) s_t + z_t
  __device__ __forceinline__ void build_table(int lane) {
    const float level = static_cast<float>(lane & (NA - 1)) + 0.5f;
    constexpr int kPairsAtOnce = 64 >> TB;
#pragma unroll
    for (int it = 0; it < NA; ++it) {
      const uint32_t p = static_cast<uint32_t>(__shfl(static_cast<int>(tpar), it * kPairsAtOnce + (lane >> TB)));
      const f16x2 sz = u2h(p);
      const float rev = fmaf(level, static_cast<float>(sz.x), static_cast<float>(sz.y)) * 0.15915494309189535f;   // turns
      const uint32_t at = ((it * kPairsAtOnce) >> 4) & 1 ? build_odd : build_even;
      *(PQ_LDS f32x2*)static_cast<uintptr_t>(at + it * (kPairsAtOnce / 2) * (NA * 16)) = f32x2{__builtin_amdgcn_cosf(rev), __builtin_amdgcn_sinf(rev)};
    }
  }
  // Step S: pairs 2 pair_step, + 1 of the lane's block, one batch; half of the batches after the other.  The
  // instruction rounds at the size of the running sum, which is restarted after two (16 pairs).  With NH = 4 two
  // accumulators do: a column has zeros in the first or in the last four pair steps.
  static constexpr int pair_step(int S) { return S % 32 / 4; }
  static constexpr int batch_of(int S) { return S / 32 * 4 + S % 4; }
  static constexpr bool to_sum(int j) { return NH == 4 ? j % 4 < 2 : j < 2; }            // (else to d)
  static constexpr bool starts(int j) { return NH == 4 ? j == 2 : j % 2 == 0; }          // d, from zero
  static constexpr bool ends(int j) { return NH == 4 ? j == 7 : j > 2 && j % 2 == 1; }   // d is added to the sum, four steps later
  template <int S>
  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rc_nxt, int rot_nxt) {
    if constexpr (S < 64) {
      constexpr int j = pair_step(S), t = batch_of(S);
      uint32_t at;
      pair_fields<RB, TB, 2 * j>(cu[t], row_even, code[S % kRing][0], at);
      trig[S % kRing][0] = *(const PQ_LDS f32x2*)static_cast<uintptr_t>(at + j * (NA * 16));
      pair_fields<RB, TB, 2 * j + 1>(cu[t], row_odd, code[S % kRing][1], at);
      trig[S % kRing][1] = *(const PQ_LDS f32x2*)static_cast<uintptr_t>(at + j * (NA * 16));
      if constexpr (j == 7) load_unit_of(t, rc_nxt, rot_nxt);
    }
  }
  template <int S>
  __device__ __forceinline__ void steps(__amdgpu_buffer_rsrc_t rc_nxt, int rot_nxt) {
    if constexpr (S < 64) {
      constexpr int j = pair_step(S), t = batch_of(S);
      if constexpr (t % 4 == 0) {
        rad = *(const PQ_LDS f32x4*)static_cast<uintptr_t>(rad_get + j * 16);
        qv = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(q_addr + j * 128);
      }
      issue<S + kAhead>(rc_nxt, rot_nxt);
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float rho = fmaf(code[S % kRing][e], rad[2 * e], rad[2 * e + 1]);
        const float cs = trig[S % kRing][e].x, sn = trig[S % kRing][e].y;
        w[2 * e] = h2u(to_half2(rho * cs, rho * sn));
        asm("" : "+v"(w[2 * e]));                 // (read back from the pair, not converted once more)
        const f16x2 high = u2h(w[2 * e]);
        // of the product, not of its rounding to fp32; one conversion for both (v_fma_mixlo / mixhi, two fewer: 118.4 against 116.5 us)
        float lx = fmaf(rho, cs, -static_cast<float>(high.x)), ly = fmaf(rho, sn, -static_cast<float>(high.y));
        asm("" : "+v"(lx), "+v"(ly));
        const f16x2 low = to_half2(lx, ly);
        w[2 * e + 1] = h2u(low);
      }
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const f16x8 k_op = as_operand(w[0], w[1], w[2], w[3]), q_op = as_operand(qv.x, qv.x, qv.y, qv.y);
      if constexpr (to_sum(j)) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k_op, q_op, j == 0 ? zero : s[t], 0, 0, 0);
      else d[t % 4] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k_op, q_op, starts(j) ? zero : d[t % 4], 0, 0, 0);
      if constexpr (S >= 4) {
        if constexpr (ends(pair_step(S - 4))) s[batch_of(S - 4)] += done[t % 4];
      }
      if constexpr (ends(j)) done[t % 4] = d[t % 4];
      __builtin_amdgcn_sched_barrier(0);
      steps<S + 1>(rc_nxt, rot_nxt);
    }
  }
  static constexpr bool kPrepared = false;
  // As ScoreWalk::run, the scores scaled by 2^(what is returned + the head's query shift).
  __device__ __forceinline__ int run(__amdgpu_buffer_rsrc_t rc_nxt, __amdgpu_buffer_rsrc_t rp_nxt, int rot_nxt, int lane) {
    const f16x2 p = u2h(par);
    const float pair = *(const PQ_LDS float*)static_cast<uintptr_t>(down_addr + lane * 4);
    const float sc = static_cast<float>(p.x) * pair, z = static_cast<float>(p.y) * pair;
    const uint32_t bound = wave_max_u32(max(f2u(sc * static_cast<float>(1 << RB)) & 0x7fffffffu, f2u(z) & 0x7fffffffu));
    const int k = min(100, kGroupedTop + 127 - static_cast<int>(bound >> 23));   // (a page of zeros: anything)
    *(PQ_LDS f32x2*)static_cast<uintptr_t>(rad_put) = f32x2{__builtin_ldexpf(sc, k), __builtin_ldexpf(fmaf(0.5f, sc, z), k)};
    build_table(lane);
    load_params(rp_nxt, lane);
    wave_lds_sync();
    issue<0>(rc_nxt, rot_nxt);
    issue<1>(rc_nxt, rot_nxt);
    issue<2>(rc_nxt, rot_nxt);
    static_assert(kAhead == 3, "reads issued before the first step");
    __builtin_amdgcn_sched_barrier(0);
    steps<0>(rc_nxt, rot_nxt);
#pragma unroll
    for (int i = 0; i < 4; ++i) s[4 + i] += done[i];
    fold_columns<NH>(s, lane & 4);
    wave_lds_sync();
    return k;
  }
  __device__ __forceinline__ void residual(const __half* rows, int nv_res, int rot, int lane) {
    const uint32_t row = static_cast<uint32_t>(lane) >> 4;
    const uint32_t q0 = q_addr - row * kGroupedQueryBlock;
    residual_products<O>(s, rows, nv_res, rot, lane, [&](int kd, int j0, int e) {
      // dims of pairs j0 + 2 e, + 1: one coordinate of each
      const int j = j0 + 2 * e;
      const u32x2 v = *(const PQ_LDS u32x2*)static_cast<uintptr_t>(q0 + (j >> 4) * kGroupedQueryBlock + ((j & 15) >> 1) * 128);
      const f16x2 two = u2h(__builtin_amdgcn_perm(v.y, v.x, kd >> 1 ? 0x07060302u : 0x05040100u));
      // without the pairs' scales: no parameter carries the other half of them here
      const f32x2 pairs = *(const PQ_LDS f32x2*)static_cast<uintptr_t>(down_addr + j * 4);
      return h2u(to_half2(static_cast<float>(two.x) * pairs.x, static_cast<float>(two.y) * pairs.y));
    });
    fold_columns<NH>(s, lane & 4);
  }
};

// Pool pages of the pages a wavefront handles in a chunk (chunk pages wave, wave + NW, ...), read one by
// one through the scalar cache, a page ahead of their use.  Entries of the table row are read
// without knowing the sequence's length; `get` masks the pages past the wavefront's last one, and
// block-table entries outside the pool.
template <int NW>
struct PageIds {
  const PQ_CONST int32_t* table;   // block-table row of the sequence, at the wavefront's first page
  int64_t n_pool_pages;
  int n_row;                       // entries of the row that belong to the wavefront from there on
  int n_p;                         // pages of the wavefront in this chunk
  int ahead;                       // entry of the page that get() is asked for next
  __device__ __forceinline__ void fetch(int k) { ahead = k < n_row ? table[NW * k] : -1; }
  __device__ __forceinline__ void start(const DecodeArgs& a, int seq, int first_page) {
    table = reinterpret_cast<const PQ_CONST int32_t*>(
        reinterpret_cast<uintptr_t>(a.block_table + static_cast<int64_t>(seq) * a.max_pages_per_seq + first_page));
    n_pool_pages = a.n_pool_pages;
    n_row = first_page < a.max_pages_per_seq ? (a.max_pages_per_seq - first_page + NW - 1) / NW : 0;
    fetch(0);
  }
  // id of the wavefront's k-th page, k = 0, 1, 2, ...; -1 if masked or past its last page
  __device__ __forceinline__ int get(int k) {
    const int id = ahead;
    fetch(k + 1);
    return k < n_p && id >= 0 && id < n_pool_pages ? id : -1;
  }
};
// Lane number, computed where it is asked for (two instructions): cheaper than a register through
// the page loop.
__device__ __forceinline__ int lane_id() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
  return l;
}

// Two work-groups share a compute unit, a wavefront of each a SIMD: with quantized values they take the higher issue
// priority in turns, page by page, so that one's matrix instructions meet the other's vector work.
__device__ __forceinline__ int priority_turn() {
  return static_cast<int>(((blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) / 256u) & 1u);
}
__device__ __forceinline__ void alternate_priority(int turn) {
  if (turn & 1) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// With fp16 values the priority falls with the part of the chunk that is left, so that the work-groups of a compute
// unit get on alike.  Among equals the SIMD favours the older wavefront: of two work-groups that had started
// together with four pages a wavefront each, one was done at 38 us, the other, by then alone with half of the loads
// in flight, at 48.  One 128K sequence at 3+3 bits 63.0 -> 57.4 us (on a device where it takes 56.5 without, 55.6), 64 ragged ones 241 -> 229, 31 x 3000 tokens
// 40.4 -> 39.6; 16 x 32K 208.1 -> 208.9, one head per KV head 110.3 -> 110.8.  (The later work-group always first: 61 / 225 / 40.9 /
// 210.4 / 112; by pages left, not by their part: 57 - 61 / 230 / 40.4 / 209.  With quantized values no difference from turns.)
__device__ __forceinline__ void priority_of_rest(int left, int all) {
  if (left == all) __builtin_amdgcn_s_setprio(3);
  else if (4 * left >= 3 * all) __builtin_amdgcn_s_setprio(2);
  else if (2 * left >= all) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// What an accumulator of dim k (of the lane's 8) is multiplied with at the end with quantized values: a
// code was masked in place as an fp16 denormal, code * 2^(position - 24).  Fields are moved up to
// bits 4 .. 9 first: the matrix unit aligns products by their operands' exponent fields, and the
// low bits of products with denormals further down are lost (measured: 2e-4 of the output with
// fields at bit 0, 1e-6 at bits 4 and up).
template <int VB>
__device__ __forceinline__ constexpr float code_unscale(int k) {
  constexpr int kAt2[8] = {4, 6, 8, 6, 8, 4, 6, 8};
  const int at = VB == 4 ? ((k & 3) == 1 ? 4 : 6) : kAt2[k];
  return static_cast<float>(1 << (24 - at));
}

// Stores a page's raw scores, left by a walk in plain token order and folded, for the heads from row `first_head` of a.scores
// on: the lane's tokens 4 row .. + 3 of its batches, of one head.  Tokens from nv on are not stored.
template <int NH>
__device__ __forceinline__ void store_scores(const DecodeArgs& a, const f32x4 (&s)[8], int down, int64_t first_head, int page, int nv, int lane) {
  const int row = lane >> 4, col = lane & 15, head = column_head<NH>(col);
  if (col >= 8 || head >= a.n_heads) return;
  const int other = NH == 4 && (col & 4) ? 64 : 0;                     // batch 4 + j: the token's bit 6 the other way
  float* const out = a.scores + (first_head + head) * a.scores_stride + static_cast<int64_t>(page) * kGroup;
#pragma unroll
  for (int t = 0; t < NH; ++t) {
    const int token = (16 * t + 4 * row) ^ other;
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __builtin_ldexpf(s[t][i], -down);
    if (uni(nv) == kGroup) {                                           // a whole page: four neighbours at a time
      __builtin_memcpy(out + token, v, 16);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (token + i < nv) out[token + i] = v[i];
    }
  }
}

// Raw scores alone, grouped angle quantizer: the walk of the attention kernel, page by page.
template <int RB, int TB, int NH>
__device__ __forceinline__ void grouped_scores_body(const DecodeArgs& a) {
  constexpr int kWaves4 = 4;
  using Walk = GroupedWalk<RB, TB, TokenOrder::kPlain, NH>;
  constexpr uint32_t kCodesBytes = kBlocks * kGroup * Walk::UB;
  __shared__ __attribute__((aligned(16))) uint8_t table[kWaves4][Walk::kTableBytes];
  __shared__ GroupedQuery query;
  __shared__ __attribute__((aligned(16))) f32x2 radii[kWaves4][kPairs];
  __shared__ int q_shift[kMaxHeads];
  __shared__ __attribute__((aligned(16))) float pair_down[kPairs];
  __shared__ __attribute__((aligned(16))) uint16_t exponents[kPairs][NH];
  const int kvh = blockIdx.x, seq = blockIdx.y, chunk = blockIdx.z;
  const int L = uni(clamped_len(a, seq)), n_pages = pages_of_len(L);
  const int page0 = chunk * a.pages_per_chunk;
  if (page0 >= n_pages) return;
  const int npg = min(a.pages_per_chunk, n_pages - page0);
  const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63;
  const int64_t first_head = static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0;
  const QueryFetch qf = a.q_is_f32 ? fetch_query_heads<true>(a, first_head * kHeadDim, tid) : fetch_query_heads<false>(a, first_head * kHeadDim, tid).widened();
  const int n_w = npg > wave ? (npg - wave + kWaves4 - 1) / kWaves4 : 0;
  const int res_page = (a.residual != nullptr && (L % kGroup) != 0) ? L / kGroup : -1;
  PageIds<kWaves4> pids;
  pids.start(a, seq, page0 + wave);
  pids.n_p = n_w;
  auto page_setup = [&](int k, __amdgpu_buffer_rsrc_t& rc, __amdgpu_buffer_rsrc_t& rp, int& nv) {
    const int pid = pids.get(k);
    const bool ok = pid >= 0;
    const int64_t ph = ok ? static_cast<int64_t>(pid) * a.n_kv_heads + kvh : 0;
    const int page = page0 + wave + kWaves4 * k;
    nv = ok ? min(kGroup, L - page * kGroup) : 0;
    const bool packed = ok && page != res_page;
    rc = make_rsrc(a.codes + ph * kCodesBytes, packed ? kCodesBytes : 0u);
    rp = make_rsrc(a.params + ph * (kPairs * 2), packed ? kPairs * 8u : 0u);
  };
  Walk w;
  w.init(table[wave], query, pair_down, radii[wave], lane);
  __amdgpu_buffer_rsrc_t rc_cur, rp_cur, rc_nxt, rp_nxt;
  int nv_cur, nv_nxt;
  page_setup(0, rc_cur, rp_cur, nv_cur);
  w.load_params(rp_cur, lane);
#pragma unroll
  for (int t = 0; t < 8; ++t) w.load_unit_of(t, rc_cur, 0);
  store_grouped_query<NH>(query, q_shift, pair_down, exponents, qf, 1.f, tid);
  __syncthreads();
  const int shift = q_shift[column_head<NH>(lane & 15)];
  for (int it = 0; it < n_w; ++it) {
    const int page = page0 + wave + kWaves4 * it;
    page_setup(it + 1, rc_nxt, rp_nxt, nv_nxt);
    int down = w.run(rc_nxt, rp_nxt, 0, lane) + shift;
    int nv = nv_cur;
    if (page == res_page) {                                            // its keys are here, whatever the block table says
      nv = L - res_page * kGroup;
      w.residual(a.residual + (static_cast<int64_t>(seq) * a.n_kv_heads + kvh) * (kGroup * kHeadDim), nv, 0, lane);
      down = shift;
    }
    store_scores<NH>(a, w.s, down, first_head, page, nv, lane);
    nv_cur = nv_nxt;
  }
}

// ---- attention ----------------------------------------------------------------------------------
// kCut: the chunks are cut on the device (a.cut_places > 0).  kMatWaves: wavefronts of the work-group, 4 or 8.
// kGroupedRadius: 0 on the uniform grid; with the grouped angle quantizer the radius bits (queries of either type are
// taken as fp32 there, so that Q32 is true).
template <int W, int VB, int NH, bool Q32, bool kCut, int kMatWaves, int kGroupedRadius = 0>
__device__ __forceinline__ void attention_body(const DecodeArgs& a) {
  constexpr int UB = 2 * W;
  constexpr int kMatThreads = kMatWaves * 64;
  constexpr bool kQuantV = VB != 16;
  constexpr bool kGrouped = kGroupedRadius != 0;
  static_assert(!kGrouped || (Q32 && kMatWaves == 4), "what the grouped quantizer's kernels are");
  constexpr TokenOrder kOrder = token_order(VB);
  constexpr int kChain = kQuantV ? 16 : 4;
  constexpr uint32_t kCodesBytes = kBlocks * kGroup * UB;
  // Probabilities are exp2(score - m) with m the running maximum rounded up to a whole number
  // (rescaling factors are then exact powers of two).  With quantized values they meet the token's
  // scale before they are split; scales are taken times 2^s_exp, which brings the largest that
  // the wavefront has seen into [2^3, 2^4), so that what is split stays below 2^4 and keeps its bits
  // whatever the values' size (it is 2^-10: error 3e-6 so, 4e-3 with the scales as they are).
  constexpr int kUp = kQuantV ? 15 - (kScaleTop + 1) : 15;               // the split's S
  // The softmax of a token is the work of one lane in each part: with 4 heads the columns of the two
  // halves take half of the batches each (kOwn) and hand their operand words to each other.
  constexpr int kOwn = NH;
  constexpr int kVLoads = kQuantV ? kGroup * kHeadDim * VB / 8 / 1024 : 32;   // 1 KB wavefront loads per page of values

  using Grouped = GroupedWalk<kGrouped ? kGroupedRadius : 4, kGrouped ? W - kGroupedRadius : 4, kOrder, NH>;
  struct Shared {
    union {
      __attribute__((aligned(16))) uint8_t lut[kGrouped ? kMatWaves * Grouped::kTableBytes : (1 << W) * kTableRow];
      __attribute__((aligned(16))) float red[kMatWaves][NH][kHeadDim];   // end of the chunk
    };
    union {
      std::conditional_t<kGrouped, GroupedQuery, QueryShared> q;
      __attribute__((aligned(16))) float lent[kFinishLdsFloats];         // end of the chunk: to the merge
      int32_t pages[kCut ? kBalancedSeqs : 1];                           // of the sequences, while the chunks are cut
    };
    __attribute__((aligned(16))) std::conditional_t<kGrouped, f32x2, uint32_t> params[kMatWaves][kPairs];
    // {scale, zero} of the page's values; the same with 1 in the zero's place
    __attribute__((aligned(16))) uint32_t vpar[kQuantV ? kMatWaves : 1][2][kQuantV ? kGroup : 1];
    __attribute__((aligned(16))) float red_ml[3][NH][kMatWaves];          // m, l, sum of p * zero-point; a head's read together
    int q_shift[kMaxHeads];
    __attribute__((aligned(16))) float pair_down[kPairs];
    __attribute__((aligned(16))) uint16_t exponents[kPairs][NH];
    int stage;
  };
  __shared__ Shared sh;
  static_assert(sizeof(Shared) <= (kMatWaves == 4 ? 80 : 160) * 1024, "eight wavefronts per compute unit");

  const int tid = threadIdx.x;
  const int wave = uni(tid >> 6);
  const int lane = tid & 63;
  const int kvh = blockIdx.x;
  int seq = blockIdx.y, chunk = blockIdx.z;
  int L, n_pages, page0 = 0, n_chunks = 1, npg = 0;
  int64_t row0 = 0;
  // A launch cut on the device: what the sequences' lengths make of this work-group's slot.  False: nothing.
  const int slot = seq;
  BalancedPlan plan;
  auto take_cut = [&] {
    plan.store_others(a, sh.pages, tid);
    const int chunks = plan.cut(a, VB == 16, kGrouped);
    if (slot >= chunks) return false;
    if (slot >= a.n_seqs && !plan.locate(slot, seq, chunk)) return false;
    int before;
    plan.sequence(seq, n_pages, n_chunks, before);
    int most;
    plan.pages_of_chunk(seq, chunk, page0, most);
    npg = min(most, n_pages - page0);
    row0 = (static_cast<int64_t>(before) * a.n_kv_heads + kvh * n_chunks) * a.group_total + static_cast<int64_t>(a.head0) * n_chunks;
    if (a.n_seqs > 64) __syncthreads();                                // the lengths make room for what shares their memory
    return true;
  };
  // The key table's entry, and the query below, are asked for before the page's loads: whoever waits for them
  // does not wait for the page as well (loads return in order).
  uint4 entry;
  if constexpr (!kGrouped) entry = fetch_key_entry<W>(key_table<W>(a.table_index), tid);
  // A first chunk, of sequence number `slot`: its pages are under way before the cut is made.
  const bool cut_later = kCut && slot < a.n_seqs;
  if constexpr (kCut) {
    plan.load(a, lane);
    if (!cut_later && !take_cut()) return;
  } else {
    const int big = min(chunk, a.n_big);
    page0 = big * a.pages_per_chunk + (chunk - big) * a.pages_small;
  }
  // (the same in every lane; said once more where paths have joined, or these go to vector registers)
  seq = uni(seq);
  chunk = uni(chunk);
  page0 = uni(page0);
  // the query and the page numbers are asked for without waiting for the sequence's length
  const int64_t q_at = (static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0) * kHeadDim;
  QueryFetch qf;
  if constexpr (kGrouped) qf = a.q_is_f32 ? fetch_query_heads<true>(a, q_at, tid) : fetch_query_heads<false>(a, q_at, tid).widened();
  else qf = fetch_query_heads<Q32>(a, q_at, tid);
  PageIds<kMatWaves> pids;
  pids.start(a, seq, page0 + wave);
  L = uni(clamped_len(a, seq));
  n_pages = pages_of_len(L);
  if (cut_later) {
    npg = min(kMatWaves, n_pages);                                     // at least
  } else if (!kCut) {
    n_chunks = chunks_of_pages(n_pages, a.pages_per_chunk, a.n_big, a.pages_small);
    npg = min(chunk < a.n_big ? a.pages_per_chunk : a.pages_small, n_pages - page0);
    row0 = (static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0) * a.n_chunks;
  }
  const int64_t first_head = static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0;
  if (page0 >= n_pages) {
    // nothing here; a sequence without pages gets its zero rows from its first work-group
    if (a.merge_in_kernel && chunk == 0 && tid < a.n_heads * 32)
      reinterpret_cast<float4*>(a.out + first_head * kHeadDim)[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const float sign = a.scale_log2 < 0.f ? -1.f : 1.f, scale_abs = fabsf(a.scale_log2);
  npg = uni(npg);
  int n_w = npg > wave ? (npg - wave + kMatWaves - 1) / kMatWaves : 0;   // chunk pages wave, wave + 4, ...
  const int res_page = (a.residual != nullptr && (L % kGroup) != 0) ? L / kGroup : -1;
  pids.n_p = n_w;

  const uint32_t voff_values = lane * 16;     // 16 lanes a token row (fp16) or a block of units (quantized)
  auto page_setup = [&](int k, __amdgpu_buffer_rsrc_t& rc, __amdgpu_buffer_rsrc_t& rp, __amdgpu_buffer_rsrc_t& rv,
                        __amdgpu_buffer_rsrc_t& rvp, int& nv, int& rot) {
    const int pid = pids.get(k);
    const bool ok = pid >= 0;
    const int64_t ph = ok ? static_cast<int64_t>(pid) * a.n_kv_heads + kvh : 0;
    const int page = page0 + wave + kMatWaves * k;
    nv = ok ? min(kGroup, L - page * kGroup) : 0;
    // pages and heads are a power-of-two number of bytes apart: wavefronts that walk them in the
    // same order keep hitting the same memory channels together, so the order is rotated
    rot = (ok && !kQuantV) ? (pid * 13 + kvh * 5) & 7 : 0;
    const bool packed = ok && page != res_page;                        // the residual group has no codes yet
    rc = make_rsrc(a.codes + ph * kCodesBytes, packed ? kCodesBytes : 0u);
    constexpr uint32_t kParamWords = kPairs * (kGrouped ? 2 : 1);
    rp = make_rsrc(a.params + ph * kParamWords, packed ? kParamWords * 4u : 0u);
    if constexpr (kQuantV) {
      // whole units are read; codes of slots past the sequence end are finite by construction
      // and meet a zero probability.  Their parameters could be anything: bounded by nv.
      rv = make_rsrc(reinterpret_cast<const uint8_t*>(a.values) + ph * (kGroup * kHeadDim * VB / 8),
                     nv > 0 ? kGroup * kHeadDim * VB / 8 : 0u);
      rvp = make_rsrc(a.v_params + ph * kGroup, static_cast<uint32_t>(nv) * 4u);
    } else {
      rv = make_rsrc(a.values + ph * (kGroup * kHeadDim), static_cast<uint32_t>(nv) * (kHeadDim * 2));
      rvp = rv;
    }
  };
  __amdgpu_buffer_rsrc_t rc_cur, rp_cur, rv_cur, rvp_cur, rc_nxt, rp_nxt, rv_nxt, rvp_nxt;
  int nv_cur, nv_nxt, rot_cur, rot_nxt;
  std::conditional_t<kGrouped, Grouped, ScoreWalk<W, kOrder, NH, Q32, kQuantV ? 2 : 1, kChain>> w;
  auto init_walk = [&](int lane) {
    if constexpr (kGrouped) w.init(sh.lut + wave * Grouped::kTableBytes, sh.q, sh.pair_down, sh.params[wave], lane);
    else w.init(sh.lut, sh.q, sh.pair_down, sh.params[wave], lane);
  };
  init_walk(lane);
  uint4 vr[kQuantV ? 1 : 4][8];                                        // fp16 values: four groups of 8 rows (32 tokens)
  uint4 vq[kQuantV ? kVLoads : 1];                                     // quantized values: the page's units
  u32x2 vpar = {0u, 0u};                                               // (scale, zero) of tokens 2 lane, 2 lane + 1
  // rows of value group g: batches 2g, 2g + 1, tokens 4 i + row of each
  auto load_rows = [&](uint4 (&dst)[8], __amdgpu_buffer_rsrc_t rv, int g, int rot_of_page) {
    int rot = uni(rot_of_page);
    asm volatile("" : "+s"(rot));      // offsets stay scalar, whatever else is derived from the rotation (else a loop per load)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dst[4 * b + i] = buf_load16<kAuxStream>(rv, voff_values, static_cast<uint32_t>((2 * g + b + rot) & 7) * 4096u + i * 1024u);
  };
  page_setup(0, rc_cur, rp_cur, rv_cur, rvp_cur, nv_cur, rot_cur);
  w.load_params(rp_cur, lane);
#pragma unroll
  for (int t = 0; t < 8; ++t) w.load_unit_of(t, rc_cur, rot_cur);
  if constexpr (kQuantV) {
    vpar = __builtin_amdgcn_raw_buffer_load_b64(rvp_cur, lane * 8, 0, kAuxCached);
#pragma unroll
    for (int k = 0; k < kVLoads; ++k) vq[k] = buf_load16<kAuxStream>(rv_cur, voff_values, k * 1024);
  } else {
    load_rows(vr[0], rv_cur, 0, rot_cur);
    load_rows(vr[1], rv_cur, 1, rot_cur);
  }
  if constexpr (kCut) {
    if (cut_later) {
      take_cut();                                                      // (a first chunk always exists)
      npg = uni(npg);
      n_w = npg > wave ? (npg - wave + kMatWaves - 1) / kMatWaves : 0;
      pids.n_p = n_w;
    }
    n_chunks = uni(n_chunks);
  }
  const int stride = kCut ? n_chunks : a.n_chunks;
  if constexpr (kGrouped) {
    store_grouped_query<NH>(sh.q, sh.q_shift, sh.pair_down, sh.exponents, qf, sign, tid);
  } else {
    store_key_entry<W, kMatThreads>(sh.lut, entry, tid);                              // while the first page is under way
    store_query_heads<NH, Q32>(sh.q, sh.q_shift, sh.pair_down, sh.exponents, qf, sign, tid);
  }
  __syncthreads();

  // per lane: column (head, part), running maximum, sums over the lane's tokens
  // (fp16 values: the sums of p come from the matrix unit like one more dim, l_acc)
  // (quantized values: sums of p in high-part columns, of p * zero-point in low-part ones, lz_run)
  float m_run = kNegInf, lz_run = 0.f;
  int s_exp = 15;                                                      // (as far as fp16 goes)
  f32x4 l_acc = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[8];                                                        // dim 8 col + e; columns 4 row .. + 3
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int lane0 = lane;
  int q_shift = kQuantV ? sh.q_shift[column_head<NH>(lane & 15)] : 0;
  const uint32_t vpar_put = lds_addr(sh.vpar[kQuantV ? wave : 0]) + lane * 8;
  const uint32_t vpar_get = lds_addr(sh.vpar[kQuantV ? wave : 0]) +
                            (row_token<kOrder>(4 * (lane >> 4)) + (NH == 4 && (lane & 4) ? 64 : 0) + (lane & 8 ? 0 : kGroup)) * 4;
  // Quantized values: a page's parameters brought to their scales and put in LDS -- of the first page here, of the others among the
  // values of the page before, where nobody waits for the reductions one behind the other.
  static_assert(std::remove_reference_t<decltype(w)>::kPrepared == (kQuantV && !kGrouped), "who prepares the parameters");
  int page_shift = 0, s_exp_page = s_exp;
  auto prepare_page = [&](int lane) {
    if constexpr (kQuantV) {
      const int e = static_cast<int>(wave_max_u32(max(vpar.x & 0xffffu, vpar.y & 0xffffu)) >> 10);   // of the page's largest scale
      s_exp_page = max(-12, min(s_exp, kScaleTop + 15 - e));
      const f16x2 factor = u2h(static_cast<uint32_t>((s_exp_page + 15) << 10) | 0x3c000000u);         // {2^s_exp, 1}
      const u32x2 sz = {h2u(u2h(vpar.x) * factor), h2u(u2h(vpar.y) * factor)};
      *(PQ_LDS u32x2*)static_cast<uintptr_t>(vpar_put) = sz;
      *(PQ_LDS u32x2*)static_cast<uintptr_t>(vpar_put + kGroup * 4) = u32x2{(sz.x & 0xffffu) | 0x3c000000u, (sz.y & 0xffffu) | 0x3c000000u};
    }
    if constexpr (kQuantV && !kGrouped) page_shift = w.prepare(lane);
  };
  prepare_page(lane);
  const int turn = priority_turn();
  for (int it = 0; it < n_w; ++it) {
    const int pi = page0 + wave + kMatWaves * it;
    if constexpr (kQuantV) alternate_priority(turn + it);             // (costs 1 % where memory is the bound)
    else priority_of_rest(n_w - it, n_w);
    page_setup(it + 1, rc_nxt, rp_nxt, rv_nxt, rvp_nxt, nv_nxt, rot_nxt);
    // lane constants of the score walk, with fp16 values derived anew for each page: the value phase needs their registers
    auto lane_now = [&] { return kQuantV ? lane0 : lane_id(); };
    const int lane = lane_now();
    if constexpr (!kQuantV) {
      init_walk(lane);
      q_shift = sh.q_shift[column_head<NH>(lane & 15)];
    }
    const int s_exp_before = s_exp;
    s_exp = s_exp_page;
    if constexpr (kQuantV) vpar = __builtin_amdgcn_raw_buffer_load_b64(rvp_nxt, lane * 8, 0, kAuxCached);
    int down = w.run(rc_nxt, rp_nxt, rot_nxt, lane) + page_shift + (kGrouped ? 0 : kTableShift) + q_shift;
    if (pi == res_page) {
      w.residual(a.residual + (static_cast<int64_t>(seq) * a.n_kv_heads + kvh) * (kGroup * kHeadDim), L - res_page * kGroup,
                 rot_cur, lane_now());
      down = q_shift;
    }
    // the groups the score walk had no registers for
    if constexpr (!kQuantV) load_rows(vr[2], rv_cur, 2, rot_cur);
    __builtin_amdgcn_sched_barrier(0);

    // ---- online softmax (log2 domain) over the lane's tokens: 4 row .. + 3 of kOwn batches ----
    // above zero, so that masked scores (-inf) stay masked whatever the scale is
    const float mult = fmaxf(__builtin_ldexpf(scale_abs, -down), 1.17549435e-38f);
    if (nv_cur < kGroup) {
      const int row = lane_now() >> 4, other = NH == 4 && (lane_now() & 4) ? 64 : 0;   // batch 4 + j: the token's bit 6 the other way
      int nv = uni(nv_cur);
      asm volatile("" : "+s"(nv));                                     // 32 conditions: not worth keeping in registers
#pragma unroll
      for (int t = 0; t < kOwn; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (((batch_token<kOrder>(t, rot_cur) + row_token<kOrder>(4 * row + i)) ^ other) >= nv) w.s[t][i] = kNegInf;
    }
    float pm = max2(w.s[0][0], w.s[0][1]);
    pm = max3(pm, w.s[0][2], w.s[0][3]);
#pragma unroll
    for (int t = 1; t < kOwn; ++t) {
      pm = max3(pm, w.s[t][0], w.s[t][1]);
      pm = max3(pm, w.s[t][2], w.s[t][3]);
    }
    {
      if constexpr (NH == 4) pm = max2(pm, dpp_of<0x124>(pm));
      auto r = __builtin_amdgcn_permlane16_swap(f2u(pm), f2u(pm), false, false);
      pm = max2(u2f(r[0]), u2f(r[1]));
      auto q = __builtin_amdgcn_permlane32_swap(f2u(pm), f2u(pm), false, false);
      pm = max2(u2f(q[0]), u2f(q[1]));
    }
    const float m_new = max2(m_run, __builtin_ceilf(pm * mult));
    const bool dead = !(m_new > kNegInf);                              // nothing valid seen so far
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0 || s_exp != s_exp_before) {
      const float alpha = dead ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first page
      if constexpr (kQuantV) lz_run *= alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float al = __shfl(alpha, (NH == 8 ? 4 * ((lane_now() >> 4) & 1) : 0) + i);   // head of accumulator row i
        if constexpr (!kQuantV) l_acc[i] *= al;
        else al = __builtin_ldexpf(al, s_exp - s_exp_before);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e][i] *= al;
      }
      m_run = m_new;
    }
    const float off = dead ? 0.f : -m_run;
    const f32x2 part = split_part<kUp>(lane_now() & 8);
    uint32_t p_op[8][2];                                               // batch t: fp16 pairs of tokens 4 row + (0, 1), (2, 3)
#pragma unroll
    for (int t = 0; t < kOwn; ++t) {
      float p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(w.s[t][i], mult, off));
      if constexpr (kQuantV) {
        // V~ = code * s + z (Section 2): fold s (times 2^s_exp) into the probability, collect p * z (low-part columns; p in the others)
        const u32x4 vp = *(const PQ_LDS u32x4*)static_cast<uintptr_t>(vpar_get + batch_token<kOrder>(t, 0) * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f16x2 sz = u2h(vp[i]);
          lz_run = fmaf(p[i], static_cast<float>(sz.y), lz_run);
          p[i] = fmaf(p[i], static_cast<float>(sz.x), 0.f);
        }
      }
      if constexpr (!kQuantV) {
        // (not all at once, nor behind the exponentials: 1 - 2 % with one head per KV head)
        if (t == kOwn / 4) load_rows(vr[3], rv_cur, 3, rot_cur);
      }
      p_op[t][0] = split_pair<kUp>(p[0], p[1], part);
      p_op[t][1] = split_pair<kUp>(p[2], p[3], part);
      if constexpr (NH == 4) {
        // columns of half 1 take batch t from half 0 (row_ror:4), those of half 0 batch 4 + t from half 1 (row_ror:12)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int own = static_cast<int>(p_op[t][e]);
          p_op[t][e] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(own, own, 0x124, 0xf, 0xa, false));
          p_op[4 + t][e] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(own, own, 0x12c, 0xf, 0x5, false));
        }
      }
    }

    // ---- values: acc += P^T V, 32 tokens (batches 2g, 2g + 1) per instruction ----
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (g == 1) prepare_page(lane_now());
      const f16x8 pa = as_operand(p_op[2 * g][0], p_op[2 * g][1], p_op[2 * g + 1][0], p_op[2 * g + 1][1]);
      if constexpr (VB == 16) {
        constexpr uint32_t kOnes = 0x3c003c00u;
        l_acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, as_operand(kOnes, kOnes, kOnes, kOnes), l_acc, 0, 0, 0);
        uint4(&v)[8] = vr[g];
        const uint32_t wv[4][8] = {{v[0].x, v[1].x, v[2].x, v[3].x, v[4].x, v[5].x, v[6].x, v[7].x},
                                   {v[0].y, v[1].y, v[2].y, v[3].y, v[4].y, v[5].y, v[6].y, v[7].y},
                                   {v[0].z, v[1].z, v[2].z, v[3].z, v[4].z, v[5].z, v[6].z, v[7].z},
                                   {v[0].w, v[1].w, v[2].w, v[3].w, v[4].w, v[5].w, v[6].w, v[7].w}};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t lo[4], hi[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            lo[k] = __builtin_amdgcn_perm(wv[e][2 * k + 1], wv[e][2 * k], 0x05040100u);   // dim 2e of a token pair
            hi[k] = __builtin_amdgcn_perm(wv[e][2 * k + 1], wv[e][2 * k], 0x07060302u);   // dim 2e + 1
          }
          acc[2 * e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, as_operand(lo[0], lo[1], lo[2], lo[3]), acc[2 * e], 0, 0, 0);
          acc[2 * e + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, as_operand(hi[0], hi[1], hi[2], hi[3]), acc[2 * e + 1], 0, 0, 0);
        }
        if (g < 2) load_rows(vr[g], rv_nxt, g, rot_nxt);
        __builtin_amdgcn_sched_barrier(0);
      } else if constexpr (VB == 4) {
        // units 2g, 2g + 1 = the tokens of batches 2g, 2g + 1: words (token pair, dim half)
        const uint32_t u[2][4] = {{vq[2 * g].x, vq[2 * g].y, vq[2 * g].z, vq[2 * g].w},
                                  {vq[2 * g + 1].x, vq[2 * g + 1].y, vq[2 * g + 1].z, vq[2 * g + 1].w}};
#pragma unroll
        for (int dh = 0; dh < 2; ++dh) {
          const uint32_t x[4] = {u[0][dh], u[0][2 + dh], u[1][dh], u[1][2 + dh]};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            uint32_t f[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
              f[j] = (k == 0 ? x[j] << 6 : (k == 1 ? x[j] : x[j] >> (4 * k - 6))) & (k == 1 ? 0x00f000f0u : 0x03c003c0u);
            acc[4 * dh + k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, as_operand(f[0], f[1], f[2], f[3]), acc[4 * dh + k], 0, 0, 0);
          }
        }
        vq[2 * g] = buf_load16<kAuxStream>(rv_nxt, voff_values, (2 * g) * 1024);
        vq[2 * g + 1] = buf_load16<kAuxStream>(rv_nxt, voff_values, (2 * g + 1) * 1024);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        static_assert(VB == 2, "value bits");
        // unit g = 32 tokens: words are token pairs with all 8 dims
        const uint32_t x[4] = {vq[g].x, vq[g].y, vq[g].z, vq[g].w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          constexpr uint32_t kMask[8] = {0x00300030u, 0x00c000c0u, 0x03000300u, 0x00c000c0u,
                                         0x03000300u, 0x00300030u, 0x00c000c0u, 0x03000300u};
          uint32_t f[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) f[j] = (k < 3 ? x[j] << 4 : (k < 5 ? x[j] : x[j] >> 6)) & kMask[k];
          acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, as_operand(f[0], f[1], f[2], f[3]), acc[k], 0, 0, 0);
        }
        vq[g] = buf_load16<kAuxStream>(rv_nxt, voff_values, g * 1024);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    rc_cur = rc_nxt; rp_cur = rp_nxt; rv_cur = rv_nxt; rvp_cur = rvp_nxt; nv_cur = nv_nxt; rot_cur = rot_nxt;
  }

  auto top_of = [&](int h) {                                           // the wavefronts' largest maximum
    float m = sh.red_ml[0][h][0];
#pragma unroll
    for (int v = 1; v < kMatWaves; ++v) m = fmaxf(m, sh.red_ml[0][h][v]);
    return m;
  };
  // ---- fold the wavefronts: maxima and sums through LDS, then the accumulators, where the key table was ----
  // (Two accumulators' parts at a time, each in half of the lanes: with a value a time, in lanes that half of the time held
  // nothing, the fold was 224 instructions instead of 112 and one sequence of 777 tokens 12.3 us instead of 11.6.)
  {
    const int lane = lane_id(), row = lane >> 4, col = lane & 15;
    const int acc_head = NH == 8 ? 4 * (row & 1) : 0;                  // head of accumulator row i: acc_head + i
    const float back = __builtin_ldexpf(1.f, row >= 2 ? -kUp - kLowShift : -kUp);   // rows 2, 3 are low parts
    // columns 0 .. NH - 1 are the heads' high parts; accumulator rows: high part + low part
    float l_tot = kQuantV ? sum_rows(lz_run) : 0.f;
    if constexpr (kQuantV && NH == 4) l_tot += dpp_of<0x12c>(l_tot);   // the other half's batches (row_ror:12, of the same part)
    const float z_tot = kQuantV ? dpp_of<0x128>(l_tot) : 0.f;          // of the head's low-part column
    if (lane < NH) {
      sh.red_ml[0][lane][wave] = m_run;
      if constexpr (kQuantV) sh.red_ml[1][lane][wave] = l_tot;
      sh.red_ml[2][lane][wave] = z_tot;
    }
    if constexpr (!kQuantV) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float l = tsum32(l_acc[i] * back, l_acc[i] * back);
        if (col == 0 && row < NH / 4) sh.red_ml[1][4 * row + i][wave] = l;
      }
    }
    __syncthreads();
    float wgt[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = acc_head + i;
      const float M = top_of(h);
      wgt[i] = M > kNegInf ? __builtin_amdgcn_exp2f(sh.red_ml[0][h][wave] - M) : 0.f;
      if constexpr (kQuantV) wgt[i] = __builtin_ldexpf(wgt[i], -s_exp);
    }
    // dims 8 col .. + 3 in lanes 0 - 31, 8 col + 4 .. + 7 in lanes 32 - 63
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[e][i] = sum_parts(acc[e][i] * back, acc[4 + e][i] * back) * wgt[i];
        if constexpr (kQuantV) acc[e][i] *= row < 2 ? code_unscale<VB>(e) : code_unscale<VB>(4 + e);
      }
    if ((row & 1) < NH / 4) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(&sh.red[wave][4 * (row & 1) + i][col * 8 + 4 * (row >> 1)]) = f32x4{acc[0][i], acc[1][i], acc[2][i], acc[3][i]};
    }
    __syncthreads();
  }

  finish_chunk<NH>(a, seq, kvh, chunk, n_chunks, row0, stride, wave * 64 + lane_id(), [&](int h, int quad, float& M, float& l) {
    M = top_of(h);
    auto part = [&](int v) { return *reinterpret_cast<const f32x4*>(&sh.red[v][h][quad * 4]); };
    f32x4 o = (part(0) + part(2)) + (part(1) + part(3));
    if constexpr (kMatWaves == 8) o += (part(4) + part(6)) + (part(5) + part(7));
    l = 0.f;
    if (M > kNegInf) {
      float zp = 0.f;                                                  // zero-point term: the same for every dim
#pragma unroll
      for (int v = 0; v < kMatWaves; ++v) {
        const float wg = __builtin_amdgcn_exp2f(sh.red_ml[0][h][v] - M);
        l = fmaf(wg, sh.red_ml[1][h][v], l);
        zp = fmaf(wg, sh.red_ml[2][h][v], zp);
      }
      if constexpr (kQuantV) o += zp;
    }
    return o;
  }, sh.lent, &sh.stage);
}

}  // namespace
}  // namespace pq
