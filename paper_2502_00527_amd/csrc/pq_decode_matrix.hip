// Kernels of the uniform angle grid (pq_decode_matrix.hpp) and their launch ladders.  The attention
// kernel runs under two names, which pq_decode_kernel_name() reports: pq_decode_roles_kernel for
// launches of 256 work-groups or more, pq_decode_partials_kernel for the others (and for
// quantized values with more than two query heads per KV head).
//
// This file is the fp16-value and score-only kernels; pq_decode_matrix_v4.hip and
// pq_decode_matrix_v2.hip compile it again for 4-bit and 2-bit values.
#include "pq_decode_matrix.hpp"

#ifndef PQ_MATRIX_VB
#define PQ_MATRIX_VB 16
#define PQ_MATRIX_LAUNCH launch_attention_matrix_v16
#endif

namespace pq {
namespace {
namespace matrix {

#define PQ_MATRIX_ATTR __launch_bounds__(kMatThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))

template <int W, int VB, int NH, bool Q32>
__global__ PQ_MATRIX_ATTR void pq_decode_roles_kernel(const DecodeArgs a) { attention_body<W, VB, NH, Q32>(a); }
template <int W, int VB, int NH, bool Q32>
__global__ PQ_MATRIX_ATTR void pq_decode_partials_kernel(const DecodeArgs a) { attention_body<W, VB, NH, Q32>(a); }

#if PQ_MATRIX_VB == 16
// Query-key scores only (the operation the paper times in Section 5.2): the score walk of the
// attention kernel, one work-group per (KV head, sequence, chunk); the raw q . k~ of valid tokens
// leave as 16 bytes a lane.
template <int W, int NH, bool Q32>
__global__ __launch_bounds__(kScoreWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void pq_score_matrix_kernel(const DecodeArgs a) {
  constexpr TokenOrder kOrder = TokenOrder::kPlain;
  constexpr uint32_t kCodesBytes = kBlocks * kGroup * 2 * W;
  struct Shared {
    __attribute__((aligned(16))) uint8_t lut[(1 << W) * kTableRow];
    QueryShared q;
    __attribute__((aligned(16))) uint32_t params[kScoreWaves][kPairs];
    int q_shift[kMaxHeads];
  };
  __shared__ Shared sh;
  const int kvh = blockIdx.x, seq = blockIdx.y, chunk = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63, row = lane >> 4, col = lane & 15, head = column_head<NH>(col);
  const int wave = uni(tid >> 6);
  const int page0 = chunk * a.pages_per_chunk;
  const QueryFetch qf = fetch_query_heads(a, Q32, (static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0) * kHeadDim, tid);
  PageIds<kScoreWaves> pids;
  pids.start(a, seq, page0 + wave);
  const int L = uni(clamped_len(a, seq));
  const int n_pages = pages_of_len(L);
  if (page0 >= n_pages) return;
  const int npg = min(a.pages_per_chunk, n_pages - page0);
  const int n_w = npg > wave ? (npg - wave + kScoreWaves - 1) / kScoreWaves : 0;
  const int res_page = (a.residual != nullptr && (L % kGroup) != 0) ? L / kGroup : -1;
  pids.n_p = n_w;

  auto page_setup = [&](int k, __amdgpu_buffer_rsrc_t& rc, __amdgpu_buffer_rsrc_t& rp, int& nv, int& rot) {
    const int pid = pids.get(k);
    const bool ok = pid >= 0;
    const int64_t ph = ok ? static_cast<int64_t>(pid) * a.n_kv_heads + kvh : 0;
    const int page = page0 + wave + kScoreWaves * k;
    nv = ok ? min(kGroup, L - page * kGroup) : 0;
    rot = ok ? (pid * 13 + kvh * 5) & 7 : 0;
    const bool packed = ok && page != res_page;
    rc = make_rsrc(a.codes + ph * kCodesBytes, packed ? kCodesBytes : 0u);
    rp = make_rsrc(a.params + ph * kPairs, packed ? kPairs * 4u : 0u);
  };
  __amdgpu_buffer_rsrc_t rc_cur, rp_cur, rc_nxt, rp_nxt;
  int nv_cur, nv_nxt, rot_cur, rot_nxt;
  ScoreWalk<W, kOrder, NH, Q32, 2, 2, 2> w;
  w.init(sh.lut, sh.q, sh.params[wave], lane);
  page_setup(0, rc_cur, rp_cur, nv_cur, rot_cur);
  w.load_params(rp_cur, lane);
#pragma unroll
  for (int t = 0; t < 8; ++t) w.load_unit_of(0, t, rc_cur, rot_cur);
  fill_key_table<W, kScoreWaves * 64>(sh.lut, key_table<W>(a.table_index), tid);           // while the first page is under way
  store_query_heads<NH, Q32>(sh.q, sh.q_shift, qf, 1.f, tid);
  __syncthreads();
  const int q_shift = sh.q_shift[head];
  float* const head_row = a.scores + (static_cast<int64_t>(seq) * a.n_q_heads + kvh * a.group_total + a.head0 + head) * a.scores_stride;

  const int turn = priority_turn();
  auto score_page = [&](auto set, int i) {
    const int pi = page0 + wave + kScoreWaves * i;
    alternate_priority(turn + i);
    page_setup(i + 1, rc_nxt, rp_nxt, nv_nxt, rot_nxt);
    int down = w.template run<decltype(set)::value>(rc_nxt, rp_nxt, rot_nxt, lane) + kTableShift + q_shift;
    if (pi == res_page) {
      w.residual(a.residual + (static_cast<int64_t>(seq) * a.n_kv_heads + kvh) * (kGroup * kHeadDim), L - res_page * kGroup,
                 rot_cur, lane);
      down = q_shift;
    }
    float* const out = head_row + static_cast<int64_t>(pi) * kGroup;
    if (head < a.n_heads) {
      if (nv_cur == kGroup) {
        // the columns of a head store a batch each
        constexpr int kCopies = 16 / NH;
        const int copy = col / NH;
#pragma unroll
        for (int u = 0; u < 8 / kCopies; ++u) {
          f32x4 v = w.s[kCopies * u];
#pragma unroll
          for (int c = 1; c < kCopies; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = copy == c ? w.s[kCopies * u + c][e] : v[e];
          f32x4u o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = __builtin_ldexpf(v[e], -down);
          const int tok = 16 * ((kCopies * u + copy + rot_cur) & 7) + 4 * row;
          __builtin_nontemporal_store(o, reinterpret_cast<f32x4u*>(out + tok));
        }
      } else if (col < NH) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int tok = batch_token<kOrder>(t, rot_cur) + 4 * row + e;
            if (tok < nv_cur) out[tok] = __builtin_ldexpf(w.s[t][e], -down);
          }
      }
    }
    rc_cur = rc_nxt; rp_cur = rp_nxt; nv_cur = nv_nxt; rot_cur = rot_nxt;
  };
  for (int i = 0; i < n_w; i += 2) {
    score_page(std::integral_constant<int, 0>{}, i);
    if (i + 1 < n_w) score_page(std::integral_constant<int, 1>{}, i + 1);
  }
}
#endif

template <int W, int VB, int NH, bool Q32>
void launch_one(bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  if (roles) hipLaunchKernelGGL((pq_decode_roles_kernel<W, VB, NH, Q32>), grid, dim3(kMatThreads), 0, st, a);
  else hipLaunchKernelGGL((pq_decode_partials_kernel<W, VB, NH, Q32>), grid, dim3(kMatThreads), 0, st, a);
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
#if PQ_MATRIX_VB == 16
template <int W>
void launch_scores_q(const DecodeArgs& a, dim3 grid, hipStream_t st) {
  const dim3 block(kScoreWaves * 64);
  if (a.q_is_f32) hipLaunchKernelGGL((pq_score_matrix_kernel<W, 8, true>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((pq_score_matrix_kernel<W, 8, false>), grid, block, 0, st, a);
}
#endif

}  // namespace matrix
}  // namespace

bool PQ_MATRIX_LAUNCH(int w, bool roles, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  return matrix::launch_w<PQ_MATRIX_VB>(w, roles, a, grid, st);
}

#if PQ_MATRIX_VB == 16
bool launch_scores_matrix(int w, const DecodeArgs& a, dim3 grid, hipStream_t st) {
  switch (w) {
    case 8: matrix::launch_scores_q<8>(a, grid, st); return true;
    case 6: matrix::launch_scores_q<6>(a, grid, st); return true;
    default: return false;
  }
}
#endif

}  // namespace pq
