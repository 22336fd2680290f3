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

// Maximum and sum over a wave, the same on every lane.
__device__ __forceinline__ float wave_max(float v) {
  v = row16_max(v);
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = row16_sum(v);
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// The item of a workgroup of a 1-D grid.  Workgroups are handed to the 8 XCDs round robin by their index; here an XCD takes a contiguous
// range of the items, at most one more than another.
__device__ __forceinline__ int xcd_item() {
  const int per_xcd = gridDim.x >> 3, more = gridDim.x & 7, xcd = blockIdx.x & 7;
  return xcd * per_xcd + min(xcd, more) + (int)(blockIdx.x >> 3);
}

// Blocks of a few rows run a layer in five launches: the norms and the rotation are part of the projections.  The projection
// that completes the residual stream x stores h = x * norm weight, not yet divided by the row's root mean square (one rounding
// to the storage type, as with the division), and the sums of x^2 over its 16-column tiles; the projection that reads h forms
// the row's factor from those sums while its first weights are on their way, and applies it to its own sums.
struct RowNorm {       // input side: x^2 sums [rows][blocks], blocks = d / 16
  const float* squares;
  int blocks;
  float d, eps;
};
struct QkvOut {        // where the fused QKV result goes (store_qkv_pair)
  const int4* row_slot;
  const float2* rope;
  void* q;
  void* k_pages;
  void* v_pages;
  int page_size, n_heads, n_kv, hd;
};
struct ResidualOut {   // x += result; h = x * norm (of the next projection's input); squares as in RowNorm; h null: x alone (bf16)
  float* x;
  const float* norm;
  void* h;
  float* squares;
  bool packed;         // h in fragment order
};
// bf16 activations in fragment order: the 16-byte pieces of a 16 x 64 tile in the order in which lanes and MFMAs take them,
// [row / 16][k / 64][half][lane][8] with lane (g, c) = row c, k = 16 g + 8 half of the tile.
__device__ __forceinline__ size_t packed_index(int row, int k, int K) {
  const size_t tile = (size_t)(row >> 4) * (K >> 6) + (k >> 6);
  return ((tile * 2 + ((k >> 3) & 1)) * 64 + ((k >> 4) & 3) * 16 + (row & 15)) * 8 + (k & 7);
}
// Most rows of such a block: what one row tile of gemm_rows.hip, and one row chunk of gemm_f32_kernel, holds.
constexpr int kMaxRows = 16, kMaxRowsF32 = 64;
constexpr int kRowNormMaxWidth = 8192;      // d: eight 16-byte loads per lane

// Row factors of a workgroup's rows, 16 lanes to a row (their sum is four row moves): load() early, store() into LDS where the
// loads may be waited for.  Branch-free loads, so that the wait does not cover the loads issued after them.
template <int ROWS, int WAVES>
struct RowFactors {
  static constexpr int PASSES = (ROWS + 4 * WAVES - 1) / (4 * WAVES), J = kRowNormMaxWidth / 1024;
  float4 v[PASSES][J];
  __device__ __forceinline__ void load(const RowNorm& n, int wave, int lane, int m0, int rows) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const float* src = n.squares + (size_t)(m0 + min((p * WAVES + wave) * 4 + (lane >> 4), rows - 1)) * n.blocks;
#pragma unroll
      for (int j = 0; j < J; ++j) v[p][j] = *reinterpret_cast<const float4*>(src + min((lane & 15) * 4 + j * 64, n.blocks - 4));
    }
  }
  __device__ __forceinline__ void store(const RowNorm& n, int wave, int lane, float* factor) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j)
        s += (lane & 15) * 4 + j * 64 < n.blocks ? (v[p][j].x + v[p][j].y) + (v[p][j].z + v[p][j].w) : 0.f;
      s = row16_sum(s);
      const int row = (p * WAVES + wave) * 4 + (lane >> 4);
      if ((lane & 15) == 0 && row < ROWS) factor[row] = 1.0f / sqrtf(s / n.d + n.eps);
    }
  }
};

// Rotates and stores the pair (a, b) = elements (i, i + hd / 2) of a head of the fused QKV result: Q [R][H][hd], K ([page][H_kv][slot][hd])
// and V ([page][H_kv][hd][slot]) into the layer's pages.
template <typename T>
__device__ __forceinline__ void store_qkv_pair(const QkvOut& o, int row, int head, int i, float a, float b, const int4& ps, const float2& cs) {
  const int half = o.hd >> 1;
  if (head < o.n_heads + o.n_kv) {
    T* dst = head < o.n_heads ? static_cast<T*>(o.q) + ((size_t)row * o.n_heads + head) * o.hd
                              : static_cast<T*>(o.k_pages) + (((size_t)ps.x * o.n_kv + (head - o.n_heads)) * o.page_size + ps.y) * o.hd;
    // (explicit multiply-adds: the same rounding in every kernel)
    Storage<T>::store(dst + i, fmaf(a, cs.x, -(b * cs.y)));
    Storage<T>::store(dst + i + half, fmaf(b, cs.x, a * cs.y));
  } else {
    T* dst = static_cast<T*>(o.v_pages) + ((size_t)ps.x * o.n_kv + (head - o.n_heads - o.n_kv)) * o.hd * o.page_size + ps.y;
    Storage<T>::store(dst + (size_t)i * o.page_size, a);
    Storage<T>::store(dst + (size_t)(i + half) * o.page_size, b);
  }
}

// Activation rows of the bf16 kernels are 128 bytes in LDS; their 16-byte pieces are XOR-swizzled by this value of the row.  A 16-byte
// read serves its lanes in sixteens, the first being lanes 0-3, 12-15 and 20-27: rows 0-3 and 12-15 of one piece and rows 4-11 of
// the piece two further on.  With the row pair itself these met on the same banks (40 % of the LDS cycles of 1 x 4 x 2 waves of
// 11 x 4 tiles were conflicts); exchanging the upper and the lower half of the pieces in every second two pairs keeps them apart.
__device__ __forceinline__ int row_swizzle(int row) { return ((row >> 1) & 7) ^ (row & 4); }

// What a projection kernel stores.  kPlain: the fp32 sums [split][M][N]; kGateUp (one split): act[M][F] = silu(gate) * up as bf16, of a
// [2F][K] matrix (N = 2F); kGateUpNorm: the same of rows that still need their factor (RowNorm), act in fragment order; kStats (one
// split): the sums and (max, sum exp) of every row over the workgroup's columns; kQkvHeads (one split): Q, K and V of the fused QKV
// projection, rotated and in their places (store_qkv_pair).
enum { kPlain = 0, kGateUp = 1, kStats = 2, kGateUpNorm = 3, kQkvHeads = 4 };

// Launch of gemm_bf16_wide_kernel or (block) gemm_bf16_block_kernel: wm x wn waves of mt x nt tiles, kg groups of them, n_blocks
// column blocks.
struct WidePlan {
  int wm, wn, kg, mt, nt, m_chunks, n_blocks, splits, k_per;
  bool block;
  float us;      // modelled time, for more than 64 rows
};
// kForWholeSums: the projection must not be split over workgroups (its epilogue needs the whole sums); kForStats: it leaves statistics
// where it needs no split.  kForHeads: whole sums, both halves of a rotation pair in one wave (gemm_block.hip).
enum PlanFor { kForSums, kForWholeSums, kForStats, kForHeads };
WidePlan wide_plan(int M, int N, int K, PlanFor use);
// Whether gate/up (N = 2 F, a multiple of 128) is better unsplit with the SwiGLU in its epilogue than in the K splits of its plan.
bool wide_gate_up_fused(int M, int N, int K);
// Whether the QKV projection is better unsplit with the rotation and the KV append in its epilogue than its plan and their launch.
bool block_qkv_fused(int M, int N, int K);
gs_status launch_block_qkv(const WidePlan& p, const bf16_t* x, const bf16_t* w, const QkvOut& out, int M, int N, int K, hipStream_t stream);
gs_status launch_wide(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K,
                      hipStream_t stream);
gs_status launch_wide_gate_up(const WidePlan& p, const bf16_t* x, const bf16_t* w, bf16_t* act, int M, int N, int K,
                              hipStream_t stream);
// x not yet divided by its root mean square, act in fragment order; up to kMaxRows rows (two row tiles)
gs_status launch_wide_gate_up_norm(const WidePlan& p, const bf16_t* x, const bf16_t* w, const RowNorm& norm, bf16_t* act, int M,
                                   int N, int K, hipStream_t stream);
// (mode: kPlain, kGateUp or kStats)
gs_status launch_block(int mode, const WidePlan& p, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K, float2* stats,
                       hipStream_t stream);
gs_status launch_wide_stats(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* y, float2* stats, int M, int N,
                            int K, hipStream_t stream);

}  // namespace gs
