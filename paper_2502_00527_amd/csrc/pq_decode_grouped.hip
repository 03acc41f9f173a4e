// Kernels of the grouped angle quantizer for 3 to 8 query heads a pass (pq_decode_matrix.hpp), and their launch ladder.
//
// This file is the fp16-value kernels and the score-only ones; pq_decode_grouped_v4.hip and pq_decode_grouped_v2.hip
// compile it again for 4-bit and 2-bit values.
#include "pq_decode_matrix.hpp"

#ifndef PQ_GROUPED_VB
#define PQ_GROUPED_VB 16
#define PQ_GROUPED_LAUNCH launch_attention_grouped_v16
#endif

namespace pq {
namespace {
namespace grouped {

#define PQ_GROUPED_ATTR __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))

template <int RB, int TB, int VB, int NH, bool kCut>
__global__ PQ_GROUPED_ATTR void pq_decode_partials_kernel(const DecodeArgs a) { attention_body<RB + TB, VB, NH, true, kCut, 4, RB>(a); }
template <int RB, int TB, int NH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TB == 5 ? 2 : 3, TB == 5 ? 2 : 3))) void pq_score_grouped_kernel(const DecodeArgs a) { grouped_scores_body<RB, TB, NH>(a); }

template <int RB, int TB, int NH>
void launch_heads(const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (a.cut_places > 0) hipLaunchKernelGGL((pq_decode_partials_kernel<RB, TB, PQ_GROUPED_VB, NH, true>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((pq_decode_partials_kernel<RB, TB, PQ_GROUPED_VB, NH, false>), grid, dim3(256), 0, st, a);
}
template <int RB, int TB>
bool launch(const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (a.n_heads <= 4) launch_heads<RB, TB, 4>(a, grid, st);
  else launch_heads<RB, TB, 8>(a, grid, st);
  return true;
}
template <int RB, int TB>
bool launch_scores(const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (a.n_heads <= 4) hipLaunchKernelGGL((pq_score_grouped_kernel<RB, TB, 4>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((pq_score_grouped_kernel<RB, TB, 8>), grid, dim3(256), 0, st, a);
  return true;
}

}  // namespace grouped
}  // namespace

#define PQ_FOR_RT(call)                    \
  switch (rt) {                            \
    case 44: return call<4, 4>(a, grid, st); \
    case 33: return call<3, 3>(a, grid, st); \
    case 53: return call<5, 3>(a, grid, st); \
    case 35: return call<3, 5>(a, grid, st); \
    case 42: return call<4, 2>(a, grid, st); \
    case 24: return call<2, 4>(a, grid, st); \
    default: return false;                 \
  }

bool PQ_GROUPED_LAUNCH(int rt, const DecodeArgs& a, dim3 grid, hipStream_t st) { PQ_FOR_RT(grouped::launch) }

#if PQ_GROUPED_VB == 16
bool launch_scores_grouped(int rt, const DecodeArgs& a, dim3 grid, hipStream_t st) { PQ_FOR_RT(grouped::launch_scores) }
#endif

}  // namespace pq
