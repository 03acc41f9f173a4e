// Angle bin of the uniform t-bit grid over [-pi, pi) (paper Section 3.2 with a uniform grid):
// the code is floor((atan2(y, x) + pi) * 2^t / (2 pi)) evaluated as in exact arithmetic, without
// an arc tangent.  Plain C++ (host and device) so that the rule can also be checked on the CPU.
//
// The grid is cut into eight octants that start on an axis or a diagonal.  The octant follows
// from sign and magnitude comparisons, which are exact, so a point exactly on an octant boundary
// lands in the octant that STARTS there (bins are half-open arcs; these are the only directions
// where a float pair can sit exactly on a bin edge, because the other edges have irrational
// slopes).  Inside an octant the 2^t / 8 bins are separated by the slopes tan(k D), D = 2 pi / 2^t:
// the bin is a count of float64 comparisons against mx * tan(k D) (mn, mx = the smaller / larger
// of |x|, |y|), whose rounding moves an edge by ~1e-16 rad.  In odd octants the angle runs against
// the ratio mn / mx, so the count is taken from the other side.
// Conventions: x = y = 0 -> bin 2^(t-1) (theta = 0); y = +0, x < 0 (theta = +pi) -> last bin;
// y = -0, x < 0 (theta = -pi) -> bin 0.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#ifndef PQ_HD
#define PQ_HD
#endif

namespace pq {

// tan_edge[k] = tan(k * 2 pi / 2^t) for 1 <= k < 2^t / 8 (unused entries are ignored)
template <int TB>
PQ_HD inline uint32_t angle_bin(float x, float y, const double* tan_edge) {
  constexpr int NB = 1 << TB;
  constexpr int S = NB >= 8 ? NB / 8 : 1;           // bins per octant
  // Everything about the octant is integer arithmetic on the IEEE bit patterns (finite inputs):
  // magnitudes compare like unsigned integers, and 0/1 flags are combined without branches.
  uint32_t bx, by;
  __builtin_memcpy(&bx, &x, 4);
  __builtin_memcpy(&by, &y, 4);
  const uint32_t ax = bx & 0x7fffffffu, ay = by & 0x7fffffffu;
  const uint32_t xnz = (ax + 0x7fffffffu) >> 31, ynz = (ay + 0x7fffffffu) >> 31;   // 1 if non-zero
  const uint32_t xn = (bx >> 31) & xnz;                      // x < 0
  const uint32_t yn = (by >> 31) & (ynz | xn);               // y < 0, or y = -0 with x < 0 (theta = -pi)
  const uint32_t lt = (ay - ax) >> 31, gt = (ax - ay) >> 31; // |y| < |x|, |y| > |x|
  // octant:
  //   lower half plane (yn): x < 0 -> 0 | 1 (the diagonal starts 1); x = 0 -> 2; x > 0 -> 2 | 3
  //   upper half plane     : x > 0 -> 4 | 5;                         x = 0 -> 6; x < 0 -> 6 | 7
  const uint32_t same = 1u ^ xn ^ yn;
  const uint32_t within_nz = same * (1u - lt) + (1u ^ same) * (3u - gt);
  const uint32_t within = xnz * within_nz + (1u ^ xnz) * 2u;
  const uint32_t o = (1u ^ yn) * 4u + within;
  uint32_t code;
  if (TB == 2) {
    code = o >> 1;                                  // bins are quadrants
  } else {
    uint32_t sub = 0;
    if (S > 1) {
      const uint32_t mnb = ax < ay ? ax : ay, mxb = ax < ay ? ay : ax;
      float mnf, mxf;
      __builtin_memcpy(&mnf, &mnb, 4);
      __builtin_memcpy(&mxf, &mxb, 4);
      const double mn = mnf, mx = mxf;
      const uint32_t odd = o & 1u;
      for (int k = 1; k < S; ++k) {
        const double edge = mx * tan_edge[k];
        const uint32_t past_odd = mn <= edge, past_even = edge <= mn;
        sub += odd * past_odd + (1u ^ odd) * past_even;
      }
    }
    code = o * S + sub;
  }
  const uint32_t origin = 1u ^ (xnz | ynz);
  return origin * (NB / 2) + (1u ^ origin) * code;
}

// The same bin for a pair strictly inside an octant (x != 0, y != 0, |x| != |y|; `interior` says
// whether that holds -- if not, the result is meaningless and angle_bin decides).  There the
// octant is a table look-up on (x < 0, y < 0, |y| > |x|): entry = first bin of the octant, plus
// S - 1 in odd octants, where the angle runs against the ratio mn / mx and the count of passed
// edges is subtracted; since the count is below S, both cases are one XOR with the entry.  (A
// float64 product that equals mn exactly is counted as passed in both directions; angle_bin
// counts it as passed towards the upper bin.  Edges have irrational slopes, so this is a
// statement about rounding noise, not about points on an edge.)
namespace detail {
constexpr uint32_t octant_of(int idx) {          // idx = (x < 0) + 2 (y < 0) + 4 (|y| > |x|)
  constexpr uint32_t o[8] = {4, 7, 3, 0, 5, 6, 2, 1};
  return o[idx];
}
template <int TB>
constexpr uint32_t octant_entries(int gt) {      // 4 entries of 8 bits, for idx = 4 gt .. 4 gt + 3
  constexpr int NB = 1 << TB;
  constexpr int S = NB >= 8 ? NB / 8 : 1;
  uint32_t w = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t o = octant_of(4 * gt + i);
    const uint32_t e = TB == 2 ? (o >> 1) : o * S + (o & 1u) * (S - 1);
    w |= e << (8 * i);
  }
  return w;
}
}  // namespace detail

template <int TB>
PQ_HD inline uint32_t angle_bin_interior(float x, float y, const double* tan_edge, bool& interior) {
  constexpr int NB = 1 << TB;
  constexpr int S = NB >= 8 ? NB / 8 : 1;
  constexpr uint32_t lo = detail::octant_entries<TB>(0), hi = detail::octant_entries<TB>(1);
  uint32_t bx, by;
  __builtin_memcpy(&bx, &x, 4);
  __builtin_memcpy(&by, &y, 4);
  const float ax = __builtin_fabsf(x), ay = __builtin_fabsf(y);
  const float mnf = ax < ay ? ax : ay, mxf = ax < ay ? ay : ax;
  interior = mnf != 0.f && mnf != mxf;
  const uint32_t shift = ((bx >> 28) & 8u) | ((by >> 27) & 16u);      // 8 * ((x < 0) + 2 (y < 0))
  uint32_t code = ((ay > ax ? hi : lo) >> shift) & 0xffu;
  if (S > 1) {
    const double mn = mnf, mx = mxf;
    uint32_t passed = 0;
    for (int k = 1; k < S; ++k) passed += mx * tan_edge[k] <= mn;
    code ^= passed;
  }
  return code;
}

// ---- four fp16 pairs at a time ---------------------------------------------------------------
// The same bins for four fp16 pairs with the octant found by byte look-ups.  A pair's octant number is
// (x < 0) + 2 (y < 0) + 4 (past the diagonal), as in octant_of(): the three bits of four pairs are
// gathered into the bytes of one word, which selects four bytes of the octant table.  Where the signs
// are equal a pair ON the diagonal counts as past it, otherwise not: the octant that starts there.
// Bin edges inside the octant are compared in fp32, sign(mx * tan - mn) by one fused multiply-add:
// with 11-bit significands mn / mx is never nearer to an edge than the rounding of tan
// (checked for every pair of significands in the tests).
// The result does not hold where x = 0 or y = 0, unless settle_zeros() has been over the pairs; `smallest` collects
// min(|x|, |y|) as fp16 bits in its two halves, so that the caller can tell.
namespace detail {
#if defined(__HIP_DEVICE_COMPILE__)
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u16x2(uint32_t w) { return __builtin_bit_cast(u16x2, w); }
__device__ __forceinline__ uint32_t as_word(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ uint32_t min_u16x2(uint32_t a, uint32_t b) { return as_word(__builtin_elementwise_min(as_u16x2(a), as_u16x2(b))); }
__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) { return as_word(__builtin_elementwise_max(as_u16x2(a), as_u16x2(b))); }
__device__ __forceinline__ uint32_t sub_u16x2(uint32_t a, uint32_t b) { return as_word(as_u16x2(a) - as_u16x2(b)); }
__device__ __forceinline__ uint32_t top_bits_u16x2(uint32_t a) { return as_word(as_u16x2(a) >> static_cast<uint16_t>(15)); }
__device__ __forceinline__ uint32_t pick_bytes(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }
// bits of mx * tan - mn, of half HI of the words
template <int HI>
__device__ __forceinline__ uint32_t edge_bits(uint32_t mx, uint32_t mn, float tan_edge) {
  uint32_t r;
  if constexpr (HI == 0) asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(mx), "s"(tan_edge), "v"(mn));
  else asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(mx), "s"(tan_edge), "v"(mn));
  return r;
}
#else
inline uint32_t lanes(uint32_t a, uint32_t b, uint32_t (*f)(uint32_t, uint32_t)) {
  return (f(a & 0xffffu, b & 0xffffu) & 0xffffu) | (f(a >> 16, b >> 16) << 16);
}
inline uint32_t min_u16x2(uint32_t a, uint32_t b) { return lanes(a, b, [](uint32_t p, uint32_t q) { return p < q ? p : q; }); }
inline uint32_t max_u16x2(uint32_t a, uint32_t b) { return lanes(a, b, [](uint32_t p, uint32_t q) { return p < q ? q : p; }); }
inline uint32_t sub_u16x2(uint32_t a, uint32_t b) { return lanes(a, b, [](uint32_t p, uint32_t q) { return p - q; }); }
inline uint32_t top_bits_u16x2(uint32_t a) { return (a >> 15) & 0x00010001u; }
inline uint32_t pick_bytes(uint32_t hi, uint32_t lo, uint32_t sel) {       // selectors 0 .. 7 only
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = (sel >> (8 * i)) & 7u;
    r |= (((s < 4 ? lo : hi) >> (8 * (s & 3))) & 0xffu) << (8 * i);
  }
  return r;
}
inline float half_to_float(uint32_t h) {                                    // finite, not negative
  const int e = static_cast<int>(h >> 10);
  return static_cast<float>(e == 0 ? ldexp(h & 1023u, -24) : ldexp(1024u + (h & 1023u), e - 25));
}
template <int HI>
inline uint32_t edge_bits(uint32_t mx, uint32_t mn, float tan_edge) {
  const float f = fmaf(half_to_float((mx >> (16 * HI)) & 0xffffu), tan_edge, -half_to_float((mn >> (16 * HI)) & 0xffffu));
  uint32_t b;
  memcpy(&b, &f, 4);
  return b;
}
#endif
// top bits of the four halves of (w0, w1), each in bit 7 of a byte (the other bits are anything)
PQ_HD inline uint32_t top_bytes(uint32_t w1, uint32_t w0) { return pick_bytes(w1, w0, 0x07050301u); }
}  // namespace detail

// x, y: two words each, pairs 0, 1 and 2, 3; returns the bins in the four bytes.
template <int TB>
PQ_HD inline uint32_t angle_bins_of_four(const uint32_t (&x)[2], const uint32_t (&y)[2], const float* tan_edge, uint32_t& smallest) {
  using namespace detail;
  constexpr int NB = 1 << TB;
  constexpr int S = NB >= 8 ? NB / 8 : 1;
  constexpr uint32_t lo = octant_entries<TB>(0), hi = octant_entries<TB>(1);
  uint32_t mn[2], mx[2], past[2];
  for (int i = 0; i < 2; ++i) {
    const uint32_t ax = x[i] & 0x7fff7fffu, ay = y[i] & 0x7fff7fffu;
    mn[i] = min_u16x2(ax, ay);
    mx[i] = max_u16x2(ax, ay);
    // sign of |x| - |y| - (1 where the signs are equal)
    past[i] = sub_u16x2(sub_u16x2(ax, ay), top_bits_u16x2(~(x[i] ^ y[i])));
    smallest = min_u16x2(smallest, mn[i]);
  }
  const uint32_t idx = ((top_bytes(x[1], x[0]) >> 7) & 0x01010101u) | ((top_bytes(y[1], y[0]) >> 6) & 0x02020202u) |
                       ((top_bytes(past[1], past[0]) >> 5) & 0x04040404u);
  uint32_t code = pick_bytes(hi, lo, idx);
  if (S > 1) {
    uint32_t passed = 0;
    for (int k = 1; k < S; ++k) {
      const uint32_t e01 = pick_bytes(edge_bits<1>(mx[0], mn[0], tan_edge[k]), edge_bits<0>(mx[0], mn[0], tan_edge[k]), 0x07030703u);
      const uint32_t e23 = pick_bytes(edge_bits<1>(mx[1], mn[1], tan_edge[k]), edge_bits<0>(mx[1], mn[1], tan_edge[k]), 0x07030703u);
      passed += (pick_bytes(e23, e01, 0x05040100u) >> 7) & 0x01010101u;
    }
    code ^= passed;
  }
  return code;
}

// Two fp16 pairs a word: gives zero coordinates the sign of the octant that the pair's axis belongs to (the one that
// starts there; theta = +pi stays in the last), and the origin the direction theta = 0, so that
// angle_bins_of_four holds for them.  Other pairs stay as they are.
PQ_HD inline void settle_zeros(uint32_t& x, uint32_t& y) {
  using namespace detail;
  constexpr uint32_t kOne = 0x00010001u;
  const uint32_t ax = x & 0x7fff7fffu, ay = y & 0x7fff7fffu;
  const uint32_t zx = top_bits_u16x2(sub_u16x2(ax, kOne)), zy = top_bits_u16x2(sub_u16x2(ay, kOne));   // 1 if zero
  const uint32_t xn = top_bits_u16x2(x) & ~zx, yn = top_bits_u16x2(y);
  const uint32_t yneg = yn & (~zy | xn);                     // y = -0 counts as negative beside x < 0 only (theta = -pi)
  const uint32_t xneg = xn | (zx & ~(zy | yn));              // x = 0: left of the upper half axis, right of the lower one
  x = ax | (xneg << 15) | (zx & zy);
  y = ay | (yneg << 15);
}

// v rounded to the nearest fp16 value, ties to even, returned as a double (|v| < 65504).  One
// rounding, straight from float64: the quantum is 2^(e - 10) for |v| in [2^e, 2^(e+1)), and 2^-24
// below the smallest normal fp16.  Used for the 16-bit parameters of the grouped angle quantizer,
// whose statistics are float64.
PQ_HD inline double round_to_half(double v) {
  uint64_t b;
  __builtin_memcpy(&b, &v, 8);
  int e = static_cast<int>((b >> 52) & 0x7ffu) - 1023;
  if (e < -14) e = -14;
  const uint64_t qb = static_cast<uint64_t>(e - 10 + 1023) << 52, ib = static_cast<uint64_t>(10 - e + 1023) << 52;
  double q, iq;
  __builtin_memcpy(&q, &qb, 8);
  __builtin_memcpy(&iq, &ib, 8);
  return rint(v * iq) * q;         // both scalings are exact (powers of two)
}

}  // namespace pq
