// Instantiations of the attention kernel of the grouped angle quantizer (Section 3.2 as printed: per-group
// angle min / scale, table rebuilt per group) on the vector unit, for one and two query heads per KV head: fp16 and
// quantized values, all bit allocations.
#include "pq_decode_kernels.hpp"

namespace pq {
namespace {

template <int RB, int TB, int VB>
bool launch_g(int G, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  const dim3 block(kThreads);
  switch (G) {
    case 1: hipLaunchKernelGGL((pq_decode_partials_kernel<1, RB, TB, VB>), grid, block, 0, st, a); return true;
    case 2: hipLaunchKernelGGL((pq_decode_partials_kernel<2, RB, TB, VB>), grid, block, 0, st, a); return true;
    default: return false;
  }
}

template <int RB, int TB>
bool launch_v(int v_bits, int G, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  switch (v_bits) {
    case 16: return launch_g<RB, TB, 16>(G, a, grid, st);
    case 4: return launch_g<RB, TB, 4>(G, a, grid, st);
    case 2: return launch_g<RB, TB, 2>(G, a, grid, st);
    default: return false;
  }
}

}  // namespace

bool launch_attention_partials_ga(int rt, int G, int v_bits, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  switch (rt) {
    case 44: return launch_v<4, 4>(v_bits, G, a, grid, st);
    case 33: return launch_v<3, 3>(v_bits, G, a, grid, st);
    case 53: return launch_v<5, 3>(v_bits, G, a, grid, st);
    case 35: return launch_v<3, 5>(v_bits, G, a, grid, st);
    case 42: return launch_v<4, 2>(v_bits, G, a, grid, st);
    case 24: return launch_v<2, 4>(v_bits, G, a, grid, st);
    default: return false;
  }
}

}  // namespace pq
