// Attention kernel of the uniform angle grid (pq_decode_matrix.hpp) and its launch ladder.  The
// kernel runs under two names, which pq_decode_kernel_name() reports: pq_decode_roles_kernel for
// launches of 256 work-groups or more, pq_decode_partials_kernel for the others (and for
// quantized values with more than two query heads per KV head).
//
// This file is the fp16-value kernels; pq_decode_matrix_v4.hip and pq_decode_matrix_v2.hip compile
// it again for 4-bit and 2-bit values.
#include "pq_decode_matrix.hpp"

#ifndef PQ_MATRIX_VB
#define PQ_MATRIX_VB 16
#define PQ_MATRIX_LAUNCH launch_attention_matrix_v16
#endif

namespace pq {
namespace {
namespace matrix {

#define PQ_MATRIX_ATTR(waves) __launch_bounds__(waves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))

template <int W, int VB, int NH, bool Q32, bool kCut>
__global__ PQ_MATRIX_ATTR(4) void pq_decode_roles_kernel(const DecodeArgs a) { attention_body<W, VB, NH, Q32, kCut, 4>(a); }
template <int W, int VB, int NH, bool Q32, bool kCut, int kWaves>
__global__ PQ_MATRIX_ATTR(kWaves) void pq_decode_partials_kernel(const DecodeArgs a) { attention_body<W, VB, NH, Q32, kCut, kWaves>(a); }

template <int W, int VB, int NH, bool Q32, bool kCut>
void launch_named(bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (roles) hipLaunchKernelGGL((pq_decode_roles_kernel<W, VB, NH, Q32, kCut>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((pq_decode_partials_kernel<W, VB, NH, Q32, kCut, 4>), grid, dim3(256), 0, st, a);
}
template <int W, int VB, int NH, bool Q32>
void launch_one(bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (a.cut_places > 0) launch_named<W, VB, NH, Q32, true>(roles, a, grid, st);
  else if (a.wide_groups && !roles) hipLaunchKernelGGL((pq_decode_partials_kernel<W, VB, NH, Q32, false, 8>), grid, dim3(512), 0, st, a);
  else launch_named<W, VB, NH, Q32, false>(roles, a, grid, st);
}
template <int W, int VB>
void launch_q(bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (a.n_heads <= 4) a.q_is_f32 ? launch_one<W, VB, 4, true>(roles, a, grid, st) : launch_one<W, VB, 4, false>(roles, a, grid, st);
  else a.q_is_f32 ? launch_one<W, VB, 8, true>(roles, a, grid, st) : launch_one<W, VB, 8, false>(roles, a, grid, st);
}
template <int VB>
bool launch_w(int w, bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  switch (w) {
    case 8: launch_q<8, VB>(roles, a, grid, st); return true;
    case 6: launch_q<6, VB>(roles, a, grid, st); return true;
    default: return false;
  }
}

}  // namespace matrix
}  // namespace

bool PQ_MATRIX_LAUNCH(int w, bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  return matrix::launch_w<PQ_MATRIX_VB>(w, roles, a, grid, st);
}

}  // namespace pq
