// CPU build of the library's angle-bin rule (csrc/pq_angle.hpp) for tests: fills codes[i] for
// n pairs; t_bits in 2..5.  Returns 0, or -1 for an unsupported t_bits.
#include <math.h>
#include <stdint.h>

#include "pq_angle.hpp"

extern "C" int angle_bins_host(const float* x, const float* y, int64_t n, int t_bits, int32_t* codes) {
  double tan_edge[4] = {0, 0, 0, 0};
  const int nb = 1 << t_bits;
  for (int k = 1; k < nb / 8 && k < 4; ++k) tan_edge[k] = tan(k * (2.0 * M_PI / nb));
  for (int64_t i = 0; i < n; ++i) {
    switch (t_bits) {
      case 2: codes[i] = (int32_t)pq::angle_bin<2>(x[i], y[i], tan_edge); break;
      case 3: codes[i] = (int32_t)pq::angle_bin<3>(x[i], y[i], tan_edge); break;
      case 4: codes[i] = (int32_t)pq::angle_bin<4>(x[i], y[i], tan_edge); break;
      case 5: codes[i] = (int32_t)pq::angle_bin<5>(x[i], y[i], tan_edge); break;
      default: return -1;
    }
  }
  return 0;
}

// The rule for pairs strictly inside an octant: codes[i] where it applies, -1 where the pair sits
// on an axis, a diagonal or the origin (the library then uses angle_bin).
extern "C" int angle_bins_interior_host(const float* x, const float* y, int64_t n, int t_bits, int32_t* codes) {
  double tan_edge[4] = {0, 0, 0, 0};
  const int nb = 1 << t_bits;
  for (int k = 1; k < nb / 8 && k < 4; ++k) tan_edge[k] = tan(k * (2.0 * M_PI / nb));
  for (int64_t i = 0; i < n; ++i) {
    bool interior = false;
    uint32_t c;
    switch (t_bits) {
      case 2: c = pq::angle_bin_interior<2>(x[i], y[i], tan_edge, interior); break;
      case 3: c = pq::angle_bin_interior<3>(x[i], y[i], tan_edge, interior); break;
      case 4: c = pq::angle_bin_interior<4>(x[i], y[i], tan_edge, interior); break;
      case 5: c = pq::angle_bin_interior<5>(x[i], y[i], tan_edge, interior); break;
      default: return -1;
    }
    codes[i] = interior ? (int32_t)c : -1;
  }
  return 0;
}

// The rule for four fp16 pairs at a time: x, y are fp16 bit patterns, n a multiple of 4.  codes[i] where
// it applies, -1 in all four where one of the four has a zero coordinate.
extern "C" int angle_bins_of_four_host(const uint16_t* x, const uint16_t* y, int64_t n, int t_bits, int32_t* codes) {
  float tan_edge[4] = {0, 0, 0, 0};
  const int nb = 1 << t_bits;
  for (int k = 1; k < nb / 8 && k < 4; ++k) tan_edge[k] = (float)tan(k * (2.0 * M_PI / nb));
  for (int64_t i = 0; i < n; i += 4) {
    uint32_t xw[2], yw[2], smallest = 0xffffffffu, c;
    for (int j = 0; j < 2; ++j) {
      xw[j] = x[i + 2 * j] | ((uint32_t)x[i + 2 * j + 1] << 16);
      yw[j] = y[i + 2 * j] | ((uint32_t)y[i + 2 * j + 1] << 16);
    }
    switch (t_bits) {
      case 2: c = pq::angle_bins_of_four<2>(xw, yw, tan_edge, smallest); break;
      case 3: c = pq::angle_bins_of_four<3>(xw, yw, tan_edge, smallest); break;
      case 4: c = pq::angle_bins_of_four<4>(xw, yw, tan_edge, smallest); break;
      case 5: c = pq::angle_bins_of_four<5>(xw, yw, tan_edge, smallest); break;
      default: return -1;
    }
    const bool holds = (smallest & 0xffffu) && (smallest >> 16);
    for (int j = 0; j < 4; ++j) codes[i + j] = holds ? (int32_t)((c >> (8 * j)) & 0xffu) : -1;
  }
  return 0;
}

// The same after settle_zeros(): holds for every pair.
extern "C" int angle_bins_of_four_settled_host(const uint16_t* x, const uint16_t* y, int64_t n, int t_bits, int32_t* codes) {
  float tan_edge[4] = {0, 0, 0, 0};
  const int nb = 1 << t_bits;
  for (int k = 1; k < nb / 8 && k < 4; ++k) tan_edge[k] = (float)tan(k * (2.0 * M_PI / nb));
  for (int64_t i = 0; i < n; i += 4) {
    uint32_t xw[2], yw[2], smallest = 0xffffffffu, c;
    for (int j = 0; j < 2; ++j) {
      xw[j] = x[i + 2 * j] | ((uint32_t)x[i + 2 * j + 1] << 16);
      yw[j] = y[i + 2 * j] | ((uint32_t)y[i + 2 * j + 1] << 16);
      pq::settle_zeros(xw[j], yw[j]);
    }
    switch (t_bits) {
      case 2: c = pq::angle_bins_of_four<2>(xw, yw, tan_edge, smallest); break;
      case 3: c = pq::angle_bins_of_four<3>(xw, yw, tan_edge, smallest); break;
      case 4: c = pq::angle_bins_of_four<4>(xw, yw, tan_edge, smallest); break;
      case 5: c = pq::angle_bins_of_four<5>(xw, yw, tan_edge, smallest); break;
      default: return -1;
    }
    for (int j = 0; j < 4; ++j) codes[i + j] = (int32_t)((c >> (8 * j)) & 0xffu);
  }
  return 0;
}

// Number of pairs (mn, mx) of fp16 significands and exponent differences for which sign(mx * tan - mn) in
// fp32, with tan rounded to fp32, is not that of float64.  Every ratio of two fp16 numbers in (2^-3, 1] is one of them.
extern "C" int64_t edge_mismatches_host(int t_bits) {
  int64_t bad = 0;
  const int nb = 1 << t_bits;
  for (int k = 1; k < nb / 8; ++k) {
    const double edge = tan(k * (2.0 * M_PI / nb));
    for (int mx = 1; mx < 2048; ++mx)
      for (int mn = 1; mn < 2048; ++mn)
        for (int shift = 0; shift < 4; ++shift) {
          const float p = (float)mn, q = (float)(mx << shift);
          if (p > q) continue;
          bad += (fmaf(q, (float)edge, -p) < 0.f) != (q * edge <= (double)p);
        }
  }
  return bad;
}

// The library's float64 -> fp16-grid rounding (parameters of the grouped angle quantizer).
extern "C" void round_to_half_host(const double* v, int64_t n, double* out) {
  for (int64_t i = 0; i < n; ++i) out[i] = pq::round_to_half(v[i]);
}
