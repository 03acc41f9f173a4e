// Prefill-time encoder of the polar-quantized key cache (gfx950).
//
// Per pair (x, y) = (K[j], K[j + d/2]) (Section 3.2; pairing of footnote 2 in
// Section 3.1):   rho = sqrt(x^2 + y^2),  theta = atan2(y, x),
//   angle code  a = floor((theta + pi) 2^t / 2 pi)    uniform grid over [-pi, pi)
//   radius code c = Clamp(floor((rho - z) / s), 0, 2^r - 1)
// with z = min, s = (max - min) / 2^r of rho over the tokens of the group,
// both rounded to fp16 and used as rounded.  Codes are integer decisions, so
// the arithmetic that leads to them is pinned:
//   * rho, (rho - z) / s: as IEEE fp32 with one rounding per operation and no fused
//     multiply-add gives them (this file is compiled with floating-point contraction off).
//   * the angle bin is decided by exact sign/magnitude comparisons (octant)
//     and slope comparisons against the bin edges inside the octant that are as good as
//     exact (float64, or fp32 where fp16 keys make it enough), so it equals the floor of the real-number quotient; a point exactly on
//     an edge (only possible on an axis or a diagonal) belongs to the upper
//     bin, theta = +pi is clamped into the last bin, and x = y = 0 goes to
//     bin 2^(t-1).
// With the grouped angle quantizer (Section 3.2 as printed) the angle is instead
//   theta = atan2(y, x) in float64,  a = Clamp(floor((theta - z_t) / s_t), 0, 2^t - 1)
// with z_t = min, s_t = (max - min) / 2^t of theta over the group, rounded once from
// float64 to fp16 and used as rounded (a = 0 when s_t == 0); the page's parameter block
// then holds the 64 radius entries followed by the 64 angle entries.
//
// One work-group encodes one page (128 tokens) of one KV head: thread =
// (pair octet o = tid % 8, token slot tid / 8), four tokens per thread.
#pragma clang fp contract(off)

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <math.h>

#define PQ_HD __host__ __device__
#include "pq_angle.hpp"
#include "pq_internal.hpp"

namespace pq {
namespace {

constexpr int kEncThreads = 256;
constexpr int kItems = 4;   // tokens per thread

struct EncodeArgs {
  const void* keys;
  const int32_t* page_ids;
  uint8_t* codes;
  uint32_t* params;
  int64_t token_stride;
  int64_t head_stride;
  int64_t n_tokens;
  int64_t n_pool_pages;
  int32_t n_kv_heads;
  double tan_edge[kMaxAngleBins / 8];    // tan(k * 2 pi / 2^t) for the edges inside an octant
  float tan_edge_f[kMaxAngleBins / 8];   // ... rounded to fp32
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// A thread's 8 pairs of one token as they lie in memory: 8 x coordinates, 8 y coordinates.
template <typename KT>
struct RawPairs {
  static constexpr int kQuads = sizeof(KT) / 2;      // 16-byte words a coordinate
  u32x4 x[kQuads], y[kQuads];
  __device__ __forceinline__ void load(const KT* p) {
#pragma unroll
    for (int i = 0; i < kQuads; ++i) {
      x[i] = reinterpret_cast<const u32x4*>(p)[i];
      y[i] = reinterpret_cast<const u32x4*>(p + kPairs)[i];
    }
  }
  static __device__ __forceinline__ float element(const u32x4 (&v)[kQuads], int e) {
    if constexpr (sizeof(KT) == 4) return __uint_as_float(v[e >> 2][e & 3]);
    else return static_cast<float>(__builtin_bit_cast(f16x2, static_cast<uint32_t>(v[0][e >> 1]))[e & 1]);
  }
  __device__ __forceinline__ float x_of(int e) const { return element(x, e); }
  __device__ __forceinline__ float y_of(int e) const { return element(y, e); }
  // x^2 + y^2, each operation rounded to fp32.  (The squares of fp16 numbers are exact, so that fused
  // multiply-adds, which read the halves as they are, round where the sum does.)
  __device__ __forceinline__ float squared(int e) const {
    const float a = x_of(e), b = y_of(e);
    if constexpr (sizeof(KT) == 4) {
      const float aa = a * a, bb = b * b;
      return aa + bb;
    } else {
      return __builtin_fmaf(a, a, __builtin_fmaf(b, b, 0.f));
    }
  }
};

__device__ __forceinline__ void load8(const __half* p, float (&v)[8]) {
  const uint4 r = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const __half2 h = *reinterpret_cast<const __half2*>(&w[e]);
    v[2 * e] = __low2float(h);
    v[2 * e + 1] = __high2float(h);
  }
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Correctly rounded fp32 square root.  For fp32 inputs this is the compiler's sequence (it also
// covers denormal and infinite arguments).  A sum of two squares of fp16 values is either 0 or at
// least 2^-48 and at most 2^33, so the hardware approximation (1 ulp) only needs the final
// rounding fix: step to the neighbour whose exact residual has the right sign.
template <typename KT>
__device__ __forceinline__ float sqrt_rn(float s) {
  if constexpr (sizeof(KT) == 4) {
    return sqrtf(s);
  } else {
    const float r = __builtin_amdgcn_sqrtf(s);
    const float dn = __uint_as_float(__float_as_uint(r) - 1u), up = __uint_as_float(__float_as_uint(r) + 1u);
    const float e_dn = __builtin_fmaf(-dn, r, s), e_up = __builtin_fmaf(-up, r, s);
    float out = e_dn <= 0.f ? dn : r;
    out = e_up > 0.f ? up : out;
    return s == 0.f ? 0.f : out;
  }
}

__device__ __forceinline__ uint32_t pack_half2(float lo, float hi) {
  return static_cast<uint32_t>(__half_as_ushort(__float2half_rn(lo))) |
         (static_cast<uint32_t>(__half_as_ushort(__float2half_rn(hi))) << 16);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_of(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, true));
}
constexpr int kDppSwapNeighbours = 0xB1, kDppRotate8 = 0x128;   // lane ^ 1; lane ^ 8 within a row of 16

// Folds v[0 .. 7] over the wavefront's 8 token slots (lane / 8) with f; lane l gets the result of v[l / 8].
// Each step halves the values along with the slots.
template <typename F>
__device__ __forceinline__ uint32_t fold_slots(const uint32_t (&v)[8], int lane, F f) {
  uint32_t a[4], b[2];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    auto r = __builtin_amdgcn_permlane32_swap(v[e], v[e + 4], false, false);
    a[e] = f(r[0], r[1]);
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    auto r = __builtin_amdgcn_permlane16_swap(a[e], a[e + 2], false, false);
    b[e] = f(r[0], r[1]);
  }
  b[0] = f(b[0], dpp_of<kDppRotate8>(b[0]));
  b[1] = f(b[1], dpp_of<kDppRotate8>(b[1]));
  return lane & 8 ? b[1] : b[0];
}
__device__ __forceinline__ double shuffle_fold(double v, bool smallest) {
#pragma unroll
  for (int m = 8; m < 64; m <<= 1) {
    const double o = __shfl_xor(v, m);
    v = smallest ? fmin(v, o) : fmax(v, o);
  }
  return v;
}

// Encodes one group (page) of one KV head with the 256 threads of the calling work-group.
// `keys` points at the head's d elements of the group's first token; rows are token_stride
// elements apart; nv <= 128 tokens are valid.  codes_ph / params_ph are the (page, head) slices
// of the pools.  Contains work-group barriers: all threads must call it.
//
// Radius codes.  rho = sqrt of n = x^2 + y^2 grows with n, rounding included, so the group's minimum and
// maximum are taken of n, and only they get the correctly rounded root.  A code is the floor of
// (rho - z) / s (equal to that of the rounded quotient: k s has 16 bits, so the fp32 quotient of a number
// below it stays below k).  Almost always that is settled by approximations -- the hardware's root, a
// product with 1 / s -- whose error, in units of s, is below 2^-21 of the group's maximum over s
// (root 2^-23, reciprocal and the three roundings 2^-24 each, z <= rho <= maximum); only where
// such a quotient is that near to a whole number (2 10^-5 of the pairs at 4 bits) is the wavefront's
// step done again with the exact operations.
// Angle codes: four pairs at a time for fp16 keys (pq_angle.hpp), a second time where a lane has a zero coordinate; pair by pair
// for fp32.
//
// Bound: neither the vector unit (25 instructions a pair, 44 % of the issue slots) nor HBM (52 %) alone, but one behind the
// other: work-groups that start together load, compute and store at the same time.  With 72 registers seven of a compute
// unit's possible eight are resident (64 registers for the eighth: spills, 25.4 us), 1792 of the 2048 of 32768 tokens x 8 heads;
// the others follow.  That is 84 MB, fp16 keys at 4+4 bits: 33.2 -> 20.1 us, fp32 keys 42.7 -> 32.7,
// grouped angles (whose float64 arc tangents remain) 80.5 -> 62.  Before: 69 instructions a pair -- rounded roots and IEEE
// divisions for all pairs, 20 for the angle -- and one token's loads at a time.  Two tokens a thread in work-groups of 512,
// which all fit: 21.0 us; one in 1024: 22.6.  Zero coordinates in every step (a dead channel; the same input again and again): 16.8 us
// without, 20.4 with them at 4+4 bits, 18.4 and 23.3 at 3+5; with the integer rule for those steps 28.3 and 35.6.
template <bool GA>
struct EncodeShared {                                        // LDS of encode_group
  uint32_t mn[kEncThreads / 64][kPairs];                     // per-wavefront minima / maxima of n (bits: n >= 0)
  uint32_t mx[kEncThreads / 64][kPairs];
  double tmn[GA ? kEncThreads / 64 : 1][GA ? kPairs : 1];    // of the angles
  double tmx[GA ? kEncThreads / 64 : 1][GA ? kPairs : 1];
  // of the group: 1 / s, -z / s - 1/2, and how far from a half-way point the code's approximation has to be at least
  __attribute__((aligned(16))) float inverse[kPairs];
  __attribute__((aligned(16))) float offset[kPairs];
  __attribute__((aligned(16))) float doubt[kPairs];
  __attribute__((aligned(16))) float scale[kPairs], zero[kPairs];      // s and z as stored
};

constexpr float kRounder = 12582912.f;       // 1.5 * 2^23: a sum with it is a whole number, in the low bits

template <int RB, int TB, typename KT, bool GA>
__device__ __forceinline__ void encode_group(const KT* keys, int64_t token_stride, int nv, uint8_t* codes_ph,
                                             uint32_t* params_ph, const double* tan_edge, const float* tan_edge_f, EncodeShared<GA>& sh) {
  constexpr int W = RB + TB;
  constexpr int UB = 2 * W;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int o = tid & 7;          // pairs 8o .. 8o+7
  const int slot = tid >> 3;      // tokens slot, slot+32, slot+64, slot+96
  const int wave = tid >> 6;

  // all loads of the thread under way together; past the end the last token again, which no minimum or maximum minds
  RawPairs<KT> raw[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it) raw[it].load(keys + min(slot + 32 * it, nv - 1) * token_stride + o * 8);

  float n[kItems][8];
  uint32_t ang[kItems][2];        // 8 angle codes, one byte each
  double th[GA ? kItems : 1][8];  // grouped angle quantizer: theta of every pair
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
#pragma unroll
    for (int e = 0; e < 8; ++e) n[it][e] = raw[it].squared(e);
    if constexpr (GA) {
      if (it > 0 && __builtin_amdgcn_readfirstlane(wave) * 8 + 32 * it >= nv) {   // all tokens of the step past the end: any token of the group will do
#pragma unroll
        for (int e = 0; e < 8; ++e) th[it][e] = th[it > 0 ? it - 1 : 0][e];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) th[it][e] = atan2(static_cast<double>(raw[it].y_of(e)), static_cast<double>(raw[it].x_of(e)));
      }
    } else if constexpr (sizeof(KT) == 4) {
      ang[it][0] = ang[it][1] = 0u;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // the short rule; the full one only when some lane's pair sits on an axis, a diagonal or the origin
        bool interior;
        const float x = raw[it].x_of(e), y = raw[it].y_of(e);
        uint32_t bin = angle_bin_interior<TB>(x, y, tan_edge, interior);
        if (__builtin_amdgcn_ballot_w64(!interior) != 0) bin = interior ? bin : angle_bin<TB>(x, y, tan_edge);
        ang[it][e >> 2] |= bin << (8 * (e & 3));
      }
    } else {
      uint32_t smallest = 0xffffffffu;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const uint32_t xw[2] = {raw[it].x[0][2 * g], raw[it].x[0][2 * g + 1]}, yw[2] = {raw[it].y[0][2 * g], raw[it].y[0][2 * g + 1]};
        ang[it][g] = angle_bins_of_four<TB>(xw, yw, tan_edge_f, smallest);
      }
      // a coordinate is zero in some lane
      if (__builtin_expect(__builtin_amdgcn_ballot_w64((smallest & 0xffffu) == 0 || (smallest >> 16) == 0) != 0, 0)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(raw[it].x[0][i]), "+v"(raw[it].y[0][i]));   // (nothing of it is prepared outside)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          uint32_t xw[2] = {raw[it].x[0][2 * g], raw[it].x[0][2 * g + 1]}, yw[2] = {raw[it].y[0][2 * g], raw[it].y[0][2 * g + 1]};
          settle_zeros(xw[0], yw[0]);
          settle_zeros(xw[1], yw[1]);
          ang[it][g] = angle_bins_of_four<TB>(xw, yw, tan_edge_f, smallest);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);           // one token after the other: registers
  }

  // group statistics: over this thread's tokens, the wavefront's 8 token slots, then the 4 wavefronts
  {
    uint32_t mn[8], mx[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mn[e] = mx[e] = __float_as_uint(n[0][e]);
#pragma unroll
      for (int it = 1; it < kItems; ++it) {
        mn[e] = min(mn[e], __float_as_uint(n[it][e]));
        mx[e] = max(mx[e], __float_as_uint(n[it][e]));
      }
    }
    const int pair = o * 8 + (lane >> 3);
    sh.mn[wave][pair] = fold_slots(mn, lane, [](uint32_t p, uint32_t q) { return min(p, q); });
    sh.mx[wave][pair] = fold_slots(mx, lane, [](uint32_t p, uint32_t q) { return max(p, q); });
    if constexpr (GA) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        double tmn = th[0][e], tmx = th[0][e];
#pragma unroll
        for (int it = 1; it < kItems; ++it) {
          tmn = fmin(tmn, th[it][e]);
          tmx = fmax(tmx, th[it][e]);
        }
        tmn = shuffle_fold(tmn, true);
        tmx = shuffle_fold(tmx, false);
        if (lane < 8) {
          sh.tmn[wave][o * 8 + e] = tmn;
          sh.tmx[wave][o * 8 + e] = tmx;
        }
      }
    }
  }
  __syncthreads();
  if (tid < kPairs) {
    // a pair a lane of the first wavefront: its parameters, stored in 16 bits (Appendix B.1) and used as stored
    uint32_t lo_n = sh.mn[0][tid], hi_n = sh.mx[0][tid];
#pragma unroll
    for (int w = 1; w < kEncThreads / 64; ++w) {
      lo_n = min(lo_n, sh.mn[w][tid]);
      hi_n = max(hi_n, sh.mx[w][tid]);
    }
    const float lo = sqrt_rn<KT>(__uint_as_float(lo_n)), hi = sqrt_rn<KT>(__uint_as_float(hi_n));
    const float s32 = (hi - lo) * (1.0f / static_cast<float>(1 << RB));   // exact scaling by 2^-r
    const uint32_t sz = pack_half2(s32, lo);
    const f16x2 szh = __builtin_bit_cast(f16x2, sz);
    const float s = static_cast<float>(szh.x), z = static_cast<float>(szh.y);
    const float inv = s != 0.f ? __builtin_amdgcn_rcpf(s) : 0.f;          // constant group: code 0
    params_ph[tid] = sz;
    sh.scale[tid] = s;
    sh.zero[tid] = z;
    sh.inverse[tid] = inv;
    sh.offset[tid] = __builtin_fmaf(-z, inv, -0.5f);
    sh.doubt[tid] = hi * inv * 0x1p-21f;
  }
  // grouped angle quantizer: (s_t, z_t) of this thread's 8 pairs, as stored
  double ts[8], tz[8];
  if constexpr (GA) {
    uint32_t packed_t[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      double lo = sh.tmn[0][o * 8 + e], hi = sh.tmx[0][o * 8 + e];
#pragma unroll
      for (int w = 1; w < kEncThreads / 64; ++w) {
        lo = fmin(lo, sh.tmn[w][o * 8 + e]);
        hi = fmax(hi, sh.tmx[w][o * 8 + e]);
      }
      ts[e] = round_to_half((hi - lo) * (1.0 / static_cast<double>(1 << TB)));   // exact scaling by 2^-t
      tz[e] = round_to_half(lo);
      packed_t[e] = pack_half2(static_cast<float>(ts[e]), static_cast<float>(tz[e]));   // exact conversions
    }
    if (slot == 0) {
      uint4* dst = reinterpret_cast<uint4*>(params_ph + kPairs + o * 8);
      dst[0] = make_uint4(packed_t[0], packed_t[1], packed_t[2], packed_t[3]);
      dst[1] = make_uint4(packed_t[4], packed_t[5], packed_t[6], packed_t[7]);
    }
  }
  __syncthreads();

  // radius codes and symbols, four pairs of all tokens after the other four
  constexpr float kTop = static_cast<float>((1 << RB) - 1);
  uint32_t sym[kItems][2];        // one symbol a byte
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int first = o * 8 + 4 * g;
    const f32x4 inv = *reinterpret_cast<const f32x4*>(&sh.inverse[first]), off = *reinterpret_cast<const f32x4*>(&sh.offset[first]);
    const f32x4 doubt = *reinterpret_cast<const f32x4*>(&sh.doubt[first]);
    const float sure = 0.5f - fmaxf(fmaxf(doubt[0], doubt[1]), fmaxf(doubt[2], doubt[3]));
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
      uint32_t u[4];                                       // the code in the low byte
      float worst = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // the quotient less a half, rounded to the nearest whole number; below 0 and above the top code nothing is in doubt
        const float t = __builtin_amdgcn_fmed3f(__builtin_fmaf(__builtin_amdgcn_sqrtf(n[it][4 * g + e]), inv[e], off[e]), 0.f, kTop);
        const float rounded = t + kRounder;
        u[e] = __float_as_uint(rounded);
        worst = fmaxf(worst, __builtin_fabsf(t - (rounded - kRounder)));
      }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(worst < sure)) != 0, 0)) {
        const f32x4 s = *reinterpret_cast<const f32x4*>(&sh.scale[first]), z = *reinterpret_cast<const f32x4*>(&sh.zero[first]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float qf = floorf((sqrt_rn<KT>(n[it][4 * g + e]) - z[e]) / s[e]);   // IEEE division
          qf = fminf(fmaxf(qf, 0.f), kTop);
          qf = s[e] != 0.f ? qf : 0.f;                                        // constant group: code 0 (also drops the NaN of 0/0)
          u[e] = __float_as_uint(qf + kRounder);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      const uint32_t c01 = __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400u), c23 = __builtin_amdgcn_perm(u[3], u[2], 0x0c0c0400u);
      uint32_t a;
      if constexpr (GA) {
        a = 0;
#pragma unroll
        for (int e = 4 * g; e < 4 * g + 4; ++e) {
          double q = floor((th[it][e] - tz[e]) / ts[e]);   // IEEE division
          q = fmin(fmax(q, 0.0), static_cast<double>((1 << TB) - 1));
          a |= (ts[e] != 0.0 ? static_cast<uint32_t>(q) : 0u) << (8 * (e & 3));   // constant group: code 0
        }
      } else {
        a = ang[it][g];
      }
      const uint32_t both = (a << RB) | __builtin_amdgcn_perm(c23, c01, 0x05040100u);
      sym[it][g] = slot + 32 * it < nv ? both : 0u;
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // the even lane of each (o, o^1) pair stores a token's whole 16-pair unit
  uint8_t* const cbase = codes_ph + (o >> 1) * kGroup * UB;
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int tok = slot + 32 * it;
    const uint32_t mine[2] = {sym[it][0], sym[it][1]};
    const uint32_t other[2] = {dpp_of<kDppSwapNeighbours>(mine[0]), dpp_of<kDppSwapNeighbours>(mine[1])};
    if ((o & 1) == 0) {
      uint8_t* dst = cbase + tok * UB;
      if constexpr (W == 8) {
        *reinterpret_cast<u32x4*>(dst) = u32x4{mine[0], mine[1], other[0], other[1]};
      } else {
        static_assert(W == 6, "unit width");
        // four symbols of 6 bits, a byte each, to 24 bits
        auto squeeze = [](uint32_t w) {
          const uint32_t t = (w & 0x003f003fu) | ((w >> 2) & 0x0fc00fc0u);
          return (t & 0xfffu) | ((t >> 4) & 0xfff000u);
        };
        const uint32_t q[4] = {squeeze(mine[0]), squeeze(mine[1]), squeeze(other[0]), squeeze(other[1])};
        uint32_t* d32 = reinterpret_cast<uint32_t*>(dst);
        d32[0] = q[0] | (q[1] << 24);
        d32[1] = (q[1] >> 8) | (q[2] << 16);
        d32[2] = (q[2] >> 16) | (q[3] << 8);
      }
    }
  }
}

template <int RB, int TB, typename KT, bool GA>
__global__ __launch_bounds__(kEncThreads) void pq_encode_kernel(const EncodeArgs a) {
  __shared__ EncodeShared<GA> stats;
  // the KV heads of a page are neighbours in memory and run together
  const int kvh = blockIdx.x % a.n_kv_heads, grp = blockIdx.x / a.n_kv_heads;
  const int64_t page = a.page_ids[grp];
  if (page < 0 || page >= a.n_pool_pages) return;
  const int64_t tok0 = static_cast<int64_t>(grp) * kGroup;
  const int nv = static_cast<int>(min<int64_t>(kGroup, a.n_tokens - tok0));
  const int64_t ph = page * a.n_kv_heads + kvh;
  encode_group<RB, TB, KT, GA>(static_cast<const KT*>(a.keys) + tok0 * a.token_stride + kvh * a.head_stride,
                               a.token_stride, nv, a.codes + ph * (kBlocks * kGroup * 2 * (RB + TB)),
                               a.params + ph * (kPairs * (GA ? 2 : 1)), a.tan_edge, a.tan_edge_f, stats);
}

// Appends one decode step's key per sequence to the fp16 residual buffer and, when that fills a
// group of 128 tokens, encodes the group into its page (the residual mechanism the paper's
// Appendix B.1 refers to: recent keys stay un-quantized until a full group exists).
struct AppendArgs {
  const void* new_keys;        // [seq][kv_head][d]
  __half* residual;            // [seq][kv_head][g][d]
  const int32_t* seq_lens;     // lengths BEFORE the append
  const int32_t* block_table;
  uint8_t* codes;
  uint32_t* params;
  int64_t n_pool_pages;
  int32_t n_kv_heads;
  int32_t max_pages_per_seq;
  double tan_edge[kMaxAngleBins / 8];
  float tan_edge_f[kMaxAngleBins / 8];
};

template <int RB, int TB, typename KT, bool GA>
__global__ __launch_bounds__(kEncThreads) void pq_append_kernel(const AppendArgs a) {
  __shared__ EncodeShared<GA> stats;
  const int kvh = blockIdx.x, seq = blockIdx.y, tid = threadIdx.x;
  const int L = a.seq_lens[seq];
  if (L < 0) return;
  const int slot = L % kGroup, grp = L / kGroup;
  const int64_t sh = static_cast<int64_t>(seq) * a.n_kv_heads + kvh;
  __half* const res = a.residual + sh * (kGroup * kHeadDim);
  if (tid < kHeadDim / 8) {
    float v[8];
    load8(static_cast<const KT*>(a.new_keys) + sh * kHeadDim + tid * 8, v);
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = static_cast<uint32_t>(__half_as_ushort(__float2half_rn(v[2 * e]))) |
             (static_cast<uint32_t>(__half_as_ushort(__float2half_rn(v[2 * e + 1]))) << 16);
    *reinterpret_cast<uint4*>(res + slot * kHeadDim + tid * 8) = make_uint4(w[0], w[1], w[2], w[3]);
  }
  if (slot != kGroup - 1) return;                 // the group is not complete yet (uniform)
  if (grp >= a.max_pages_per_seq) return;
  const int64_t page = a.block_table[static_cast<int64_t>(seq) * a.max_pages_per_seq + grp];
  if (page < 0 || page >= a.n_pool_pages) return;
  __syncthreads();                                // the new row is visible to the whole work-group
  const int64_t ph = page * a.n_kv_heads + kvh;
  encode_group<RB, TB, __half, GA>(res, kHeadDim, kGroup, a.codes + ph * (kBlocks * kGroup * 2 * (RB + TB)),
                                   a.params + ph * (kPairs * (GA ? 2 : 1)), a.tan_edge, a.tan_edge_f, stats);
}

template <typename Args>
void fill_edges(Args& a, int t_bits) {
  const int nb = 1 << t_bits;
  for (int k = 0; k < kMaxAngleBins / 8; ++k) {
    a.tan_edge[k] = (k >= 1 && k < nb / 8) ? tan(k * (2.0 * M_PI / nb)) : 0.0;
    a.tan_edge_f[k] = static_cast<float>(a.tan_edge[k]);
  }
}

template <int RB, int TB, bool GA = false>
hipError_t launch_encode(const EncodeArgs& a, pq_dtype dt, dim3 grid, hipStream_t st) {
  if (dt == PQ_F16) hipLaunchKernelGGL((pq_encode_kernel<RB, TB, __half, GA>), grid, dim3(kEncThreads), 0, st, a);
  else              hipLaunchKernelGGL((pq_encode_kernel<RB, TB, float, GA>), grid, dim3(kEncThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace
}  // namespace pq

using namespace pq;

extern "C" int pq_encode_keys(const pq_layout* layout, const void* keys, pq_dtype key_dtype,
                              int64_t token_stride, int64_t head_stride, int64_t n_tokens,
                              const int32_t* page_ids, void* codes_pool, void* params_pool,
                              int64_t n_pool_pages, void* hip_stream) {
  if (!layout) return PQ_ERR_INVALID_ARG;
  if (!layout_supported(layout)) return PQ_ERR_UNSUPPORTED;
  if (n_tokens < 0 || n_pool_pages <= 0) return PQ_ERR_INVALID_ARG;
  if (key_dtype != PQ_F16 && key_dtype != PQ_F32) return PQ_ERR_INVALID_ARG;
  if (n_tokens == 0) return PQ_OK;
  if (!keys || !page_ids || !codes_pool || !params_pool) return PQ_ERR_INVALID_ARG;
  // 128-bit loads: rows of a head must start on 16-byte boundaries
  const int64_t vec = key_dtype == PQ_F16 ? 8 : 4;
  if ((reinterpret_cast<uintptr_t>(keys) & 15u) || token_stride % vec || head_stride % vec ||
      token_stride < kHeadDim || head_stride < 0)
    return PQ_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(codes_pool) & 15u) || (reinterpret_cast<uintptr_t>(params_pool) & 15u))
    return PQ_ERR_INVALID_ARG;
  const int64_t n_groups = (n_tokens + kGroup - 1) / kGroup;
  if (n_groups >= (int64_t{1} << 24) || layout->n_kv_heads > 65535) return PQ_ERR_UNSUPPORTED;

  EncodeArgs a;
  a.keys = keys;
  a.page_ids = page_ids;
  a.codes = static_cast<uint8_t*>(codes_pool);
  a.params = static_cast<uint32_t*>(params_pool);
  a.token_stride = token_stride;
  a.head_stride = head_stride;
  a.n_tokens = n_tokens;
  a.n_pool_pages = n_pool_pages;
  a.n_kv_heads = layout->n_kv_heads;
  fill_edges(a, layout->t_bits);

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int kind = layout->r_bits * 10 + layout->t_bits + (layout->angle_quantizer == PQ_ANGLE_GROUPED ? 100 : 0);
  const hipError_t e = for_group_ranges(n_groups, layout->n_kv_heads, [&](int64_t first, int64_t groups) {
    EncodeArgs part = a;
    part.keys = static_cast<const char*>(keys) + first * kGroup * token_stride * (key_dtype == PQ_F16 ? 2 : 4);
    part.page_ids += first;
    part.n_tokens -= first * kGroup;
    const dim3 grid(static_cast<uint32_t>(groups * layout->n_kv_heads));
    switch (kind) {
      case 144: return launch_encode<4, 4, true>(part, key_dtype, grid, st);
      case 133: return launch_encode<3, 3, true>(part, key_dtype, grid, st);
      case 153: return launch_encode<5, 3, true>(part, key_dtype, grid, st);
      case 135: return launch_encode<3, 5, true>(part, key_dtype, grid, st);
      case 142: return launch_encode<4, 2, true>(part, key_dtype, grid, st);
      case 124: return launch_encode<2, 4, true>(part, key_dtype, grid, st);
      case 44: return launch_encode<4, 4>(part, key_dtype, grid, st);
      case 33: return launch_encode<3, 3>(part, key_dtype, grid, st);
      case 53: return launch_encode<5, 3>(part, key_dtype, grid, st);
      case 35: return launch_encode<3, 5>(part, key_dtype, grid, st);
      case 42: return launch_encode<4, 2>(part, key_dtype, grid, st);
      default: return launch_encode<2, 4>(part, key_dtype, grid, st);     // layout_supported() admits no other
    }
  });
  if (e != hipSuccess) return record_hip_error(e);
  return PQ_OK;
}

namespace pq {
namespace {
template <int RB, int TB, bool GA = false>
hipError_t launch_append(const AppendArgs& a, pq_dtype dt, dim3 grid, hipStream_t st) {
  if (dt == PQ_F16) hipLaunchKernelGGL((pq_append_kernel<RB, TB, __half, GA>), grid, dim3(kEncThreads), 0, st, a);
  else              hipLaunchKernelGGL((pq_append_kernel<RB, TB, float, GA>), grid, dim3(kEncThreads), 0, st, a);
  return hipGetLastError();
}
}  // namespace
}  // namespace pq

extern "C" int pq_append_keys(const pq_layout* layout, const void* new_keys, pq_dtype key_dtype, int32_t n_seqs,
                              void* residual, const int32_t* seq_lens, const int32_t* block_table,
                              int32_t max_pages_per_seq, void* codes_pool, void* params_pool,
                              int64_t n_pool_pages, void* hip_stream) {
  if (!layout) return PQ_ERR_INVALID_ARG;
  if (!layout_supported(layout)) return PQ_ERR_UNSUPPORTED;
  if (n_seqs < 0 || n_pool_pages <= 0 || max_pages_per_seq <= 0) return PQ_ERR_INVALID_ARG;
  if (key_dtype != PQ_F16 && key_dtype != PQ_F32) return PQ_ERR_INVALID_ARG;
  if (n_seqs == 0) return PQ_OK;
  if (!new_keys || !residual || !seq_lens || !block_table || !codes_pool || !params_pool) return PQ_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(new_keys) & 15u) || (reinterpret_cast<uintptr_t>(residual) & 15u) ||
      (reinterpret_cast<uintptr_t>(codes_pool) & 15u) || (reinterpret_cast<uintptr_t>(params_pool) & 15u))
    return PQ_ERR_INVALID_ARG;
  if (n_seqs > 65535) return PQ_ERR_UNSUPPORTED;
  AppendArgs a;
  a.new_keys = new_keys;
  a.residual = static_cast<__half*>(residual);
  a.seq_lens = seq_lens;
  a.block_table = block_table;
  a.codes = static_cast<uint8_t*>(codes_pool);
  a.params = static_cast<uint32_t*>(params_pool);
  a.n_pool_pages = n_pool_pages;
  a.n_kv_heads = layout->n_kv_heads;
  a.max_pages_per_seq = max_pages_per_seq;
  fill_edges(a, layout->t_bits);
  const dim3 grid(layout->n_kv_heads, n_seqs);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  hipError_t e = hipSuccess;
  switch (layout->r_bits * 10 + layout->t_bits + (layout->angle_quantizer == PQ_ANGLE_GROUPED ? 100 : 0)) {
    case 144: e = launch_append<4, 4, true>(a, key_dtype, grid, st); break;
    case 133: e = launch_append<3, 3, true>(a, key_dtype, grid, st); break;
    case 153: e = launch_append<5, 3, true>(a, key_dtype, grid, st); break;
    case 135: e = launch_append<3, 5, true>(a, key_dtype, grid, st); break;
    case 142: e = launch_append<4, 2, true>(a, key_dtype, grid, st); break;
    case 124: e = launch_append<2, 4, true>(a, key_dtype, grid, st); break;
    case 44: e = launch_append<4, 4>(a, key_dtype, grid, st); break;
    case 33: e = launch_append<3, 3>(a, key_dtype, grid, st); break;
    case 53: e = launch_append<5, 3>(a, key_dtype, grid, st); break;
    case 35: e = launch_append<3, 5>(a, key_dtype, grid, st); break;
    case 42: e = launch_append<4, 2>(a, key_dtype, grid, st); break;
    case 24: e = launch_append<2, 4>(a, key_dtype, grid, st); break;
    default: return PQ_ERR_UNSUPPORTED;
  }
  if (e != hipSuccess) return record_hip_error(e);
  return PQ_OK;
}
