// Token-wise value quantization (paper Section 2, the formula for Q(V_n[j]); used by the paper in
// Section 6.3 "+ value quantization" and the dagger rows of its throughput table):
//   code = Clamp(round((v - z) / s), 0, 2^b - 1),  z = min of the token's d values, s = (max - min) / (2^b - 1),
// round-half-to-even, s and z stored as fp16 and used as stored, fp32 arithmetic with IEEE
// division; a constant row (s == 0) gets code 0.  Dequantized value: code * s + z.
//
// One work-group quantizes one page (128 tokens) of one KV head: thread = (dim slice tid % 16 of
// 8 dims, a unit's 4 or 8 consecutive tokens), so that a thread has the whole 16-byte unit when it
// has quantized its tokens and stores it at once; a token's minimum and maximum are folded over
// its 16 lanes by DPP moves.  Bound: vector issue (with an IEEE division per value those would be
// most of it).  32768 tokens x 8 heads, 4 bits: 28.8 us with one token a thread, divisions throughout, 2-byte stores
// and LDS shuffles; 25.1 us so.
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
// {min, -max} over a token's 128 values: the thread's 8 (four words), then the 16 lanes of the row
// (lane ^ 1, lane ^ 2, mirror within 8, mirror within 16), result in all of them
__device__ __forceinline__ uint32_t min_and_negated_max(const uint32_t (&w)[4]) {
  const uint32_t lo = pk_min(pk_min(w[0], w[1]), pk_min(w[2], w[3]));
  const uint32_t neg = pk_min(pk_min_neg(w[0], w[1]), pk_min_neg(w[2], w[3]));
  uint32_t m = pk_min(__builtin_amdgcn_perm(neg, lo, 0x05040100u), __builtin_amdgcn_perm(neg, lo, 0x07060302u));
  m = pk_min(m, dpp_of<0xB1>(m));
  m = pk_min(m, dpp_of<0x4E>(m));
  m = pk_min(m, dpp_of<0x141>(m));
  return pk_min(m, dpp_of<0x140>(m));
}

constexpr int kValueThreads = 256;

template <int VB>
__global__ __launch_bounds__(kValueThreads) void pq_encode_values_kernel(const ValueArgs a) {
  constexpr int T = 16 / VB;                     // tokens per 16-byte unit
  constexpr int kUnits = kGroup / T * 16;        // units of a page
  constexpr float kLevels = static_cast<float>((1 << VB) - 1);
  const int grp = blockIdx.x, kvh = blockIdx.y;
  const int64_t page = a.page_ids[grp];
  if (page < 0 || page >= a.n_pool_pages) return;
  const int64_t tok0 = static_cast<int64_t>(grp) * kGroup;
  const int nv = static_cast<int>(min<int64_t>(kGroup, a.n_tokens - tok0));
  const int64_t ph = page * a.n_kv_heads + kvh;
  const int sl = threadIdx.x & 15;
  const __half* base = a.values + kvh * a.head_stride + sl * 8;
  uint8_t* const dst = a.vq + ph * (kGroup * kHeadDim * VB / 8);
#pragma unroll
  for (int u = 0; u < kUnits / kValueThreads; ++u) {
    const int unit = u * kValueThreads + threadIdx.x;      // (token block unit / 16, slice unit % 16)
    const int first = unit / 16 * T;
    uint4 raw[T];
#pragma unroll
    for (int k = 0; k < T; ++k)
      raw[k] = first + k < nv ? *reinterpret_cast<const uint4*>(base + (tok0 + first + k) * a.token_stride) : make_uint4(0, 0, 0, 0);
    uint32_t field[T], par[T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
      const uint32_t w[4] = {raw[k].x, raw[k].y, raw[k].z, raw[k].w};
      float v[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const __half2 h = *reinterpret_cast<const __half2*>(&w[e]);
        v[2 * e] = __low2float(h);
        v[2 * e + 1] = __high2float(h);
      }
      const uint32_t m = min_and_negated_max(w);
      const __half2 mh = *reinterpret_cast<const __half2*>(&m);
      const float mn = __low2float(mh), mx = -__high2float(mh);
      const __half sh = __float2half_rn((mx - mn) / kLevels), zh = __float2half_rn(mn);
      const float sf = __half2float(sh), zf = __half2float(zh);
      // The code is rint of the IEEE quotient (v - z) / s, half to even.  The product with 1 / s is within
      // 2^-22 of it (relatively), so it rounds to the same whole number unless it lies within 2^-17 of
      // a half (codes beyond 2^5 are clamped whatever they are); only then the division is carried out.
      const float inv = 1.f / sf;
      float q[8], off = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float p = (v[e] - zf) * inv;
        q[e] = rintf(p);
        off = fmaxf(off, fabsf(p - q[e]));
      }
      if (__builtin_amdgcn_ballot_w64(off > 0.5f - 0x1p-17f) != 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = rintf((v[e] - zf) / sf);
      }
      uint32_t bits = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float c = fminf(fmaxf(q[e], 0.f), kLevels);
        bits |= static_cast<uint32_t>(sf != 0.f ? c : 0.f) << (VB * e);
      }
      const bool valid = first + k < nv;
      field[k] = valid ? bits : 0u;
      par[k] = valid ? (static_cast<uint32_t>(__half_as_ushort(sh)) | (static_cast<uint32_t>(__half_as_ushort(zh)) << 16)) : 0u;
    }
    // A unit's 32-bit words hold two consecutive tokens each, the even one in the low half:
    // 4-bit codes word 2 * pair + (dims 0-3 | dims 4-7), 2-bit codes word pair (all 8 dims).
    uint4 out;
    if constexpr (VB == 4) {
      out = make_uint4((field[0] & 0xffffu) | (field[1] << 16), (field[0] >> 16) | (field[1] & 0xffff0000u),
                       (field[2] & 0xffffu) | (field[3] << 16), (field[2] >> 16) | (field[3] & 0xffff0000u));
    } else {
      out = make_uint4(field[0] | (field[1] << 16), field[2] | (field[3] << 16), field[4] | (field[5] << 16),
                       field[6] | (field[7] << 16));
    }
    *reinterpret_cast<uint4*>(dst + unit * 16) = out;
    if (sl == 0) {
#pragma unroll
      for (int k = 0; k < T; ++k) a.vparams[ph * kGroup + first + k] = par[k];
    }
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
  if (n_groups > 0x7fffffff || layout->n_kv_heads > 65535) return PQ_ERR_UNSUPPORTED;
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
  const dim3 grid(static_cast<uint32_t>(n_groups), layout->n_kv_heads);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (v_bits == 4) hipLaunchKernelGGL(pq_encode_values_kernel<4>, grid, dim3(kValueThreads), 0, st, a);
  else hipLaunchKernelGGL(pq_encode_values_kernel<2>, grid, dim3(kValueThreads), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return record_hip_error(e);
  return PQ_OK;
}
