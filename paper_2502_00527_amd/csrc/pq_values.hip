// Token-wise value quantization (paper Section 2, the formula for Q(V_n[j]); used by the paper in
// Section 6.3 "+ value quantization" and the dagger rows of its throughput table):
//   code = Clamp(round((v - z) / s), 0, 2^b - 1),  z = min of the token's d values, s = (max - min) / (2^b - 1),
// round-half-to-even, s and z stored as fp16 and used as stored, codes as fp32 arithmetic with IEEE
// division gives them; a constant row (s == 0) and a NaN get code 0.  Dequantized value: code * s + z.
//
// One work-group quantizes one page (128 tokens) of one KV head: thread = (dim slices sl and sl + 8 of
// 8 dims each, sl = tid % 8; 4 consecutive tokens), all eight 16-byte loads of it under way together; a
// token's minimum and maximum are folded over its 8 lanes by DPP moves.
//
// The code is the exact quotient d / s, d = (v - z) rounded to fp32, rounded half to even: s and the
// half-way points (k + 1/2) s have so few bits that the nearest fp32 number to d / s lies on the same side of
// k + 1/2 as d / s itself, and is k + 1/2 only if d / s is.  So the product with 1 / s, rounded by the addition of
// 1.5 * 2^23, is the code unless d - k s, which one multiply-add gives exactly, is
// half of s to within 2^-17 s; then (every third wavefront step, for tokens on the fp16 grid hit half-way points) the
// remainder decides.  No division, and a clamp only where s is denormal: a normal s makes (max - z) / s < 2^b - 1/2.
//
// Bound: HBM, with vector issue close (about 11 instructions a value; 56 registers: all eight work-groups of a
// compute unit are resident).  32768 tokens x 8 heads, 4 bits, 85 MB: 25.2 -> 15.0 us (5.7 TB/s).  Before: 29
// instructions a value, a division where a quotient was near a half, one token's 8 values a thread.
#pragma clang fp contract(off)

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <math.h>

#include "pq_internal.hpp"

namespace pq {
namespace {

struct ValueArgs {
  const __half* values;
  const int32_t* page_ids;
  uint8_t* vq;
  uint32_t* vparams;
  int64_t token_stride;
  int64_t head_stride;
  int64_t n_tokens;
  int64_t n_pool_pages;
  int32_t n_kv_heads;
};

// fp16 pairs: element-wise minimum, and that of the negated operands' -- so that {min, -max} of a
// token is one word and one instruction folds both.
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t pk_min_neg(uint32_t a, uint32_t b) {       // min(-a, -b)
  uint32_t r;
  asm("v_pk_min_f16 %0, %1, %2 neg_lo:[1,1] neg_hi:[1,1]" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_of(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, true));
}
// {min, -max} over a token's 128 values: the thread's 16 (eight words), then the token's 8 lanes
// (lane ^ 1, lane ^ 2, mirror within 8), result in all of them
__device__ __forceinline__ uint32_t min_and_negated_max(const uint32_t (&w)[8]) {
  const uint32_t lo = pk_min(pk_min(pk_min(w[0], w[1]), pk_min(w[2], w[3])), pk_min(pk_min(w[4], w[5]), pk_min(w[6], w[7])));
  const uint32_t neg = pk_min(pk_min(pk_min_neg(w[0], w[1]), pk_min_neg(w[2], w[3])), pk_min(pk_min_neg(w[4], w[5]), pk_min_neg(w[6], w[7])));
  uint32_t m = pk_min(__builtin_amdgcn_perm(neg, lo, 0x05040100u), __builtin_amdgcn_perm(neg, lo, 0x07060302u));
  m = pk_min(m, dpp_of<0xB1>(m));
  m = pk_min(m, dpp_of<0x4E>(m));
  return pk_min(m, dpp_of<0x141>(m));
}

// fp16 half HI of a word, minus z, rounded to fp32
template <int HI>
__device__ __forceinline__ float half_minus(uint32_t w, float z) {
  float d;
  if constexpr (HI == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(z));
  else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(z));
  return d;
}
__device__ __forceinline__ float max3_abs(float a, float b, float c) {          // max(a, |b|, |c|), NaN if one of them is
  float r;
  asm("v_maximum3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// x / (2^VB - 1) correctly rounded, for x = 0, a difference of two fp16 values or infinity: one residual step
// after the product with the rounded reciprocal, equal to the division for every significand.  (Not to be
// merged with the rounding to fp16 that follows, which would then be the only one.)
template <int VB>
__device__ __forceinline__ float over_levels(float x) {
  constexpr float kLevels = static_cast<float>((1 << VB) - 1), kInverse = 1.f / kLevels;
  float q = x * kInverse;
  q = __builtin_fmaf(__builtin_fmaf(-kLevels, q, x), kInverse, q);
  asm("" : "+v"(q));
  return x < INFINITY ? q : x;
}

constexpr float kRounder = 12582912.f;           // 1.5 * 2^23: a sum with it is a whole number, in the low bits
constexpr uint32_t kRounderBits = 0x4b400000u;

// Codes of 8 values (four words) of a token as one field of 8 VB bits, the first value lowest.
template <int VB>
__device__ __forceinline__ uint32_t quantize8(const uint32_t (&w)[4], float s, float z, float inv, float half, bool clamp) {
  float t[8], off = 0.f;
  auto rest = [&](int e) {
    const float d = e & 1 ? half_minus<1>(w[e / 2], z) : half_minus<0>(w[e / 2], z);
    return __builtin_fmaf(kRounder - t[e], s, d);
  };
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    t[e] = __builtin_fmaf(half_minus<0>(w[e / 2], z), inv, kRounder);
    t[e + 1] = __builtin_fmaf(half_minus<1>(w[e / 2], z), inv, kRounder);
    off = max3_abs(off, rest(e), rest(e + 1));
  }
  if (__builtin_amdgcn_ballot_w64(!(off <= half * (1.f - 0x1p-16f))) != 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      asm volatile("" : "+v"(t[e]));             // remainders are made again: eight registers less, which is a wavefront more
      const float r = rest(e);
      // past half of s by the bit pattern: from half on if the code is odd, above half if it is even
      const uint32_t limit = __float_as_uint(half) - (__float_as_uint(t[e]) & 1u);
      t[e] += (__float_as_uint(r) & 0x7fffffffu) > limit ? __builtin_copysignf(1.f, r) : 0.f;
    }
    if (__builtin_amdgcn_ballot_w64(off != off) != 0) {     // NaN: code 0, and nothing of its bit pattern beside it
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = __builtin_fmaxf(t[e], kRounder);
    }
  }
  if (__builtin_amdgcn_ballot_w64(clamp) != 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = __uint_as_float(min(__float_as_uint(t[e]), kRounderBits + (1u << VB) - 1u));
  }
  uint32_t bits = 0, base = 0;
#pragma unroll
  for (int e = 7; e >= 0; --e) {
    bits = (bits << VB) + __float_as_uint(t[e]);
    base = (base << VB) + kRounderBits;
  }
  return bits - base;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kValueThreads = 256;
constexpr int kTokens = 4;                       // of a thread

__device__ const uint4 zero_row[16] = {};

template <int VB>
__global__ __launch_bounds__(kValueThreads, 8) void pq_encode_values_kernel(const ValueArgs a) {
  // the KV heads of a page are neighbours in memory and run together
  const int kvh = blockIdx.x % a.n_kv_heads, grp = blockIdx.x / a.n_kv_heads;
  const int64_t page = a.page_ids[grp];
  if (page < 0 || page >= a.n_pool_pages) return;
  const int64_t tok0 = static_cast<int64_t>(grp) * kGroup;
  const int nv = static_cast<int>(min<int64_t>(kGroup, a.n_tokens - tok0));
  const int64_t ph = page * a.n_kv_heads + kvh;
  const int sl = threadIdx.x & 7, block = threadIdx.x >> 3, first = block * kTokens;
  const __half* const base = a.values + kvh * a.head_stride + (tok0 + first) * a.token_stride + sl * 8;

  // (tokens past the end are rows of zeros: code 0, parameters 0)
  u32x4 raw[kTokens][2];
#pragma unroll
  for (int k = 0; k < kTokens; ++k) {
    // (as global memory, which a choice of two pointers hides)
    typedef const __attribute__((address_space(1))) u32x4 Quad;
    const Quad* const row = first + k < nv ? (Quad*)reinterpret_cast<uintptr_t>(base + k * a.token_stride) : (Quad*)reinterpret_cast<uintptr_t>(zero_row + sl);
    raw[k][0] = row[0];
    raw[k][1] = row[8];
  }

  uint32_t field[2][kTokens], par[kTokens];
#pragma unroll
  for (int k = 0; k < kTokens; ++k) {
    const uint32_t w[2][4] = {{raw[k][0].x, raw[k][0].y, raw[k][0].z, raw[k][0].w}, {raw[k][1].x, raw[k][1].y, raw[k][1].z, raw[k][1].w}};
    const uint32_t m = min_and_negated_max({w[0][0], w[0][1], w[0][2], w[0][3], w[1][0], w[1][1], w[1][2], w[1][3]});
    const __half2 mh = *reinterpret_cast<const __half2*>(&m);
    const float mn = __low2float(mh), mx = -__high2float(mh);
    const uint32_t sb = __half_as_ushort(__float2half_rn(over_levels<VB>(mx - mn)));
    const float sf = __half2float(__ushort_as_half(static_cast<unsigned short>(sb)));
    par[k] = sb | (m << 16);                     // the minimum is stored as it is
    const bool flat = sb == 0, finite = sb < 0x7c00u, denormal = sb - 1u < 0x3ffu;
    const float inv = flat ? 0.f : __builtin_amdgcn_rcpf(sf), half = flat ? INFINITY : 0.5f * sf;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const uint32_t codes = quantize8<VB>(w[p], sf, mn, inv, half, denormal);
      field[p][k] = finite ? codes : 0u;
      asm volatile("" : "+v"(field[p][k]));    // packed here, not when all tokens are done
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // A unit's 32-bit words hold two consecutive tokens each, the even one in the low half: 4-bit codes word
  // 2 * pair + (dims 0-3 | dims 4-7), 2-bit codes word pair (all 8 dims; the unit is two threads').
  uint8_t* const dst = a.vq + ph * (kGroup * kHeadDim * VB / 8);
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const uint32_t(&f)[kTokens] = field[p];
    const int slice = sl + 8 * p;
    if constexpr (VB == 4) {
      *reinterpret_cast<uint4*>(dst + (block * 16 + slice) * 16) =
          make_uint4(__builtin_amdgcn_perm(f[1], f[0], 0x05040100u), __builtin_amdgcn_perm(f[1], f[0], 0x07060302u),
                     __builtin_amdgcn_perm(f[3], f[2], 0x05040100u), __builtin_amdgcn_perm(f[3], f[2], 0x07060302u));
    } else {
      static_assert(VB == 2, "value bits");
      *reinterpret_cast<uint2*>(dst + ((block >> 1) * 16 + slice) * 16 + (block & 1) * 8) = make_uint2(f[0] | (f[1] << 16), f[2] | (f[3] << 16));
    }
  }
  if (sl == 0) {
    uint32_t* const vp = a.vparams + ph * kGroup + first;
#pragma unroll
    for (int k = 0; k < kTokens; ++k) vp[k] = par[k];
  }
}

bool value_bits_ok(int v_bits) { return v_bits == 4 || v_bits == 2; }

}  // namespace
}  // namespace pq

using namespace pq;

extern "C" size_t pq_vq_bytes_per_page(const pq_layout* l, int32_t v_bits) {
  if (!layout_supported(l) || !value_bits_ok(v_bits)) return 0;
  return static_cast<size_t>(l->n_kv_heads) * kGroup * kHeadDim * v_bits / 8;
}

extern "C" size_t pq_vq_params_bytes_per_page(const pq_layout* l) {
  if (!layout_supported(l)) return 0;
  return static_cast<size_t>(l->n_kv_heads) * kGroup * 4;
}

extern "C" int pq_encode_values(const pq_layout* layout, int32_t v_bits, const void* values, int64_t token_stride,
                                int64_t head_stride, int64_t n_tokens, const int32_t* page_ids, void* vq_pool,
                                void* vq_params_pool, int64_t n_pool_pages, void* hip_stream) {
  if (!layout) return PQ_ERR_INVALID_ARG;
  if (!layout_supported(layout) || !value_bits_ok(v_bits)) return PQ_ERR_UNSUPPORTED;
  if (n_tokens < 0 || n_pool_pages <= 0) return PQ_ERR_INVALID_ARG;
  if (n_tokens == 0) return PQ_OK;
  if (!values || !page_ids || !vq_pool || !vq_params_pool) return PQ_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(values) & 15u) || token_stride % 8 || head_stride % 8 || token_stride < kHeadDim ||
      head_stride < 0 || (reinterpret_cast<uintptr_t>(vq_pool) & 15u) || (reinterpret_cast<uintptr_t>(vq_params_pool) & 3u))
    return PQ_ERR_INVALID_ARG;
  const int64_t n_groups = (n_tokens + kGroup - 1) / kGroup;
  if (n_groups >= (int64_t{1} << 24) || layout->n_kv_heads > 65535) return PQ_ERR_UNSUPPORTED;
  ValueArgs a;
  a.values = static_cast<const __half*>(values);
  a.page_ids = page_ids;
  a.vq = static_cast<uint8_t*>(vq_pool);
  a.vparams = static_cast<uint32_t*>(vq_params_pool);
  a.token_stride = token_stride;
  a.head_stride = head_stride;
  a.n_tokens = n_tokens;
  a.n_pool_pages = n_pool_pages;
  a.n_kv_heads = layout->n_kv_heads;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const hipError_t e = for_group_ranges(n_groups, layout->n_kv_heads, [&](int64_t first, int64_t groups) {
    ValueArgs part = a;
    part.values += first * kGroup * token_stride;
    part.page_ids += first;
    part.n_tokens -= first * kGroup;
    const dim3 grid(static_cast<uint32_t>(groups * layout->n_kv_heads));
    if (v_bits == 4) hipLaunchKernelGGL(pq_encode_values_kernel<4>, grid, dim3(kValueThreads), 0, st, part);
    else hipLaunchKernelGGL(pq_encode_values_kernel<2>, grid, dim3(kValueThreads), 0, st, part);
    return hipGetLastError();
  });
  if (e != hipSuccess) return record_hip_error(e);
  return PQ_OK;
}
