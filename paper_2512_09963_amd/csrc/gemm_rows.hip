// bf16 projections of a few rows (up to kMaxRows) with whole sums in one workgroup: QKV with the rotation and the KV append,
// O and down with the residual sum (RowNorm in gemm_common.h).
//
// What bounds it: the weight stream, and at these sizes as much the number of launches.  The projections of gemm.hip cut K over
// workgroups and leave the sum of the parts, the norm and the rotation to kernels of their own, 4.7 us each.  Here a
// workgroup owns NT column tiles for all of K, its NW waves take the k steps in turn (so that all waves of the launch
// sweep the packed weights band by band) and their sums meet in LDS.  Weights and activations go from global memory
// straight into the MFMA operands, D steps ahead; an activation fragment is used by one wave of a workgroup, so LDS would not
// save a load, but every workgroup reads all activations: M x K x 2 bytes per compute unit beside 32 x NT x K of weights.  A compute
// unit takes 23 GB/s of its share of the HBM stream and 94 GB/s from L2, but not both at once (54 GB/s in all at two parts of
// activations to one of weights, whatever the number of loads in flight: a loop of the same loads alone), so beyond 16 rows
// the K splits are faster (53 rows: 40 us for the 4096 x 14336 projection, 24 and a norm with them).  The activations are stored in fragment
// order (packed_index), so that such a load is one kilobyte in a row (row-major 34.7 us against 28.9 at 32 rows).
// Per launch, us, 8B shape, 5 / 16 rows, and in brackets the K splits with their norm or rotation kernel at 5 rows:
//   6144 x 4096  11.2 / 12.0 (16.0)    4096 x 4096  8.2 / 9.6 (15.0)    4096 x 14336  21.1 / 25.1 (26.2)
#include "common.h"
#include "device_types.h"
#include "gemm_common.h"

namespace gs {
namespace {

typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

enum { kQkv = 0, kResidual = 1 };

// X: activations in fragment order; Wp: packed weights.  kQkv: tiles 2 p and 2 p + 1 of a workgroup are the halves of 16
// rotation pairs of a head.  grid: ceil(N / 16 / NT) workgroups.  One row tile: M up to 16.
template <int NT, int D, int NW, int MODE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_rows_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Wp, int M, int N, int K, RowNorm norm, QkvOut qkv, ResidualOut res) {
  static_assert(MODE != kQkv || NT % 2 == 0, "both halves of the rotation pairs");
  static_assert(kMaxRows <= 16, "one row tile");
  constexpr int W = NT * 16, THREADS = 64 * NW;
  __shared__ float red[NW][16][W];
  __shared__ float factor[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15;
  const int steps = K / 64, own = (steps - wave + NW - 1) / NW;
  const int half_tiles = MODE == kQkv ? qkv.hd >> 5 : 1;      // column tiles of half a head
  auto column_tile = [&](int t) {      // of tile t of the workgroup
    if constexpr (MODE == kQkv) {
      const int pair = blockIdx.x * (NT / 2) + (t >> 1), head = pair / half_tiles;
      return head * 2 * half_tiles + (pair - head * half_tiles) + (t & 1) * half_tiles;
    } else {
      return (int)blockIdx.x * NT + t;
    }
  };
  RowFactors<16, NW> factors;
  if constexpr (MODE == kQkv) factors.load(norm, wave, lane, 0, M);

  // lanes whose row or column does not exist read zeros (offset past the descriptor's range)
  unsigned woff[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) woff[n] = column_tile(n) * 16 < N ? (unsigned)column_tile(n) * 2048u + lane * 16u : 0x80000000u;
  const unsigned aoff = c < M ? lane * 16u : 0x80000000u;
  const size_t w_stride = (size_t)(N / 16) * 2048;
  const unsigned a_bytes = (unsigned)steps * 2048u;
  uintx4_t wr[D][NT][2], ar[D][2];
  // a step past the wave's last has empty descriptors: zeros
#define GS_LOAD(slot, s)                                                                                                     \
  {                                                                                                                          \
    const int step_ = min(wave + (s) * NW, steps - 1);                                                                       \
    const bool has_ = (s) < own;                                                                                             \
    auto rw = __builtin_amdgcn_make_buffer_rsrc(                                                                             \
        const_cast<char*>(reinterpret_cast<const char*>(Wp) + (size_t)step_ * w_stride), 0, has_ ? (unsigned)w_stride : 0u, 0x00020000); \
    auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(X) + (size_t)step_ * 2048), 0,   \
                                                has_ ? a_bytes - (unsigned)step_ * 2048u : 0u, 0x00020000);                  \
    _Pragma("unroll") for (int n = 0; n < NT; ++n) {                                                                         \
      wr[slot][n][0] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff[n], 0, 2);                                             \
      wr[slot][n][1] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff[n] + 1024, 0, 2);                                      \
    }                                                                                                                        \
    ar[slot][0] = __builtin_amdgcn_raw_buffer_load_b128(ra, aoff, 0, 0);                                                     \
    ar[slot][1] = __builtin_amdgcn_raw_buffer_load_b128(ra, aoff + 1024, 0, 0);                                              \
  }
  floatx4_t acc[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) acc[n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int d = 0; d < D; ++d) GS_LOAD(d, d);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (MODE == kQkv) factors.store(norm, wave, lane, factor);
  for (int base = 0; base < own; base += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int n = 0; n < NT; ++n)
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(&ar[d][h]),
                                                           *reinterpret_cast<const bf16x8_t*>(&wr[d][n][h]), acc[n], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      GS_LOAD(d, base + d + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#undef GS_LOAD
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][(lane >> 4) * 4 + i][n * 16 + c] = acc[n][i];
  __syncthreads();
  auto sum_of = [&](int row, int col) {      // the waves' sums, in a fixed order
    float s = red[0][row][col];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w][row][col];
    return s;
  };
  if constexpr (MODE == kQkv) {
    for (int e = tid; e < 16 * (W / 2); e += THREADS) {
      const int row = e / (W / 2), q = e - row * (W / 2), p = q >> 4;      // pair of tiles, lane of the tile
      const int pair = blockIdx.x * (NT / 2) + p;
      if (row >= M || pair * 32 >= N) continue;
      const int head = pair / half_tiles, i = (pair - head * half_tiles) * 16 + (q & 15);
      const float f = factor[row];
      store_qkv_pair<bf16_t>(qkv, row, head, i, sum_of(row, p * 32 + (q & 15)) * f, sum_of(row, p * 32 + 16 + (q & 15)) * f,
                             qkv.row_slot[row], qkv.rope[(size_t)row * (qkv.hd >> 1) + i]);
    }
  } else {
    for (int e = tid; e < 16 * W; e += THREADS) {
      const int row = e / W, q = e - row * W, col = blockIdx.x * W + q;
      const bool ok = row < M && col < N;
      float v = 0.f;
      if (ok) {
        v = res.x[(size_t)row * N + col] + sum_of(row, q);
        res.x[(size_t)row * N + col] = v;
        if (res.h)
          static_cast<bf16_t*>(res.h)[res.packed ? packed_index(row, col, N) : (size_t)row * N + col] = float_to_bf16(v * res.norm[col]);
      }
      if (!res.h) continue;
      const float sq = row16_sum(v * v);      // (16 lanes share a row and a tile)
      if (ok && (q & 15) == 0) res.squares[(size_t)row * (N >> 4) + (col >> 4)] = sq;
    }
  }
}

template <int MODE>
gs_status launch(const bf16_t* x, const bf16_t* w, int M, int N, int K, const RowNorm& norm, const QkvOut& qkv, const ResidualOut& res,
                 hipStream_t stream) {
  // one workgroup per compute unit: 16 columns where that is enough, otherwise 32; pairs of tiles, two where one would need
  // a second round (10240 x 8192 at 16 rows: 37.7 us with one)
  const int blocks = MODE == kQkv ? N / 32 : N / 16;
  const int nt = MODE == kQkv ? (blocks <= 256 ? 2 : 4) : (blocks <= 256 ? 1 : 2);
  const unsigned grid = ceil_div(N / 16, nt);
#define GS_ROWS(NT, D, NW) gemm_bf16_rows_kernel<NT, D, NW, MODE><<<grid, 64 * NW, 0, stream>>>(x, w, M, N, K, norm, qkv, res)
  if constexpr (MODE == kQkv) {
    if (nt == 2) GS_ROWS(2, 4, 8);
    else GS_ROWS(4, 4, 8);
  } else {
    if (nt == 1) GS_ROWS(1, 8, 4);
    else GS_ROWS(2, 4, 8);
  }
#undef GS_ROWS
  GS_LAUNCH_CHECK("gemm_bf16_rows");
  return GS_OK;
}

}  // namespace

gs_status launch_bf16_rows_qkv(const bf16_t* h, const bf16_t* w, const RowNorm& norm, const QkvOut& out, int M, int K, hipStream_t stream) {
  return launch<kQkv>(h, w, M, (out.n_heads + 2 * out.n_kv) * out.hd, K, norm, out, ResidualOut{}, stream);
}
gs_status launch_bf16_rows_residual(const bf16_t* in, const bf16_t* w, const ResidualOut& out, int M, int N, int K, hipStream_t stream) {
  return launch<kResidual>(in, w, M, N, K, RowNorm{}, QkvOut{}, out, stream);
}

}  // namespace gs
