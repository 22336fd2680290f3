// What the bf16 projection kernels share: softmax-statistics helpers of their epilogues and the launch plan of
// gemm_wide.hip.
#pragma once
#include <hip/hip_runtime.h>
#include "common.h"
#include "device_types.h"

namespace gs {

// Merge of two online-softmax pairs (max, sum exp(x - max)).
__device__ __forceinline__ void merge_stat(float& m, float& s, float m2, float s2) {
  const float M = fmaxf(m, m2);
  s = s * __expf(m - M) + s2 * __expf(m2 - M);
  m = M;
}

// Reductions over the 16 lanes of a DPP row (lanes 16 g .. 16 g + 15) with data-parallel-primitive moves, which
// are modifiers of ordinary vector instructions (a shuffle through the LDS crossbar costs an LDS instruction
// each): neighbours in a quad, the other pair of the quad, the mirrored quad of the half row, the mirrored half.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));      // quad_perm(1, 0, 3, 2)
  v = fmaxf(v, dpp_move<0x4E>(v));      // quad_perm(2, 3, 0, 1)
  v = fmaxf(v, dpp_move<0x141>(v));     // row_half_mirror
  return fmaxf(v, dpp_move<0x140>(v));  // row_mirror
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  return v + dpp_move<0x140>(v);
}

// Launch of gemm_bf16_wide_kernel: wm x wn waves of mt x nt tiles, kg groups of them, n_blocks column blocks.
struct WidePlan {
  int wm, wn, kg, mt, nt, m_chunks, n_blocks, splits, k_per;
};
// one_split: the projection must not be split over workgroups (its epilogue needs the whole sums).
WidePlan wide_plan(int M, int N, int K, bool one_split);
gs_status launch_wide(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K,
                      hipStream_t stream);
gs_status launch_wide_gate_up(const WidePlan& p, const bf16_t* x, const bf16_t* w, bf16_t* act, int M, int N, int K,
                              hipStream_t stream);
gs_status launch_wide_stats(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* y, float2* stats, int M, int N,
                            int K, hipStream_t stream);

}  // namespace gs
