// Dense projections Y = X * W^T of the decoder (QKV, O, gate/up, down, LM head).
//
// bf16 path (MFMA): the verify step has few rows (tens to a few hundred) against
// matrices of 10^7..10^9 weights, so every weight byte is used by only M rows: the kernels
// are weight-streaming kernels bound by HBM, and the layout serves the stream.  Most shapes go to the pipelined
// kernels of gemm_wide.hip and gemm_block.hip (same packed weights); the one here serves what GemmPlan says:
//   * the weights are stored tile-packed (gs_pack_weight): the 2 KB that one wavefront needs
//     per 64-wide k step for its 16 output columns is contiguous, and the blocks are ordered
//     [k_step][n_tile][half][lane][8 bf16]: at one k step the blocks of neighbouring column tiles
//     follow each other, so the waves of the whole launch, which advance through k at about the
//     same pace, sweep one contiguous band of memory at a time (the access pattern of a plain
//     copy, which keeps DRAM pages open) instead of thousands of unrelated 2 KB pieces.  Each
//     wave issues two fully coalesced 1 KB loads per step, straight into the MFMA B operand (no
//     LDS hop for weights); DEPTH steps are kept in flight
//   * the activations (the rows of a chunk, at most 128) are staged once per workgroup
//     in LDS (padded rows: conflict-free 16-byte reads) and shared by the four waves; their
//     global loads run DEPTH steps ahead as well, so a step never waits on the L2 round trip
//   * K is split across workgroups when N alone gives too few of them to fill 256 CUs; the
//     fp32 partial sums [S][M][N] are summed by the consumer kernel, in a fixed order
//   * the gate/up projection, where it runs without a K split, applies the SwiGLU in its epilogue and
//     stores the bf16 activation instead of fp32 sums (gemm_wide.hip).
// k order inside a step is permuted identically for both operands (lane group g takes
// k = 16g .. 16g+15, first half to the first MFMA, second half to the second), which leaves
// the dot products unchanged.  Measured without the activation side, on the gate/up shape: 6.2 TB/s
// in this order, 5.4 TB/s with each tile's k steps contiguous, 4.4 TB/s for row-major weight rows.
//
// fp32 path: gemm_f32_kernel, on the fp32 matrix instruction, for the small fp32 configuration.
#include "common.h"
#include "device_types.h"
#include "gemm_common.h"

namespace gs {
namespace {

// 16-byte load that does not displace cache lines: weights that a launch reads once (measured on the 8B shape
// at 50 rows: 4.52 instead of 4.56 ms per step)
typedef unsigned int uint4_vec __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load(const uint4* p) {
  const uint4_vec v = __builtin_nontemporal_load(reinterpret_cast<const uint4_vec*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

constexpr int kSkinnyWaves = 4;     // per workgroup (64 columns)
constexpr int kSkinnyDepth = 4;     // k steps of weights and activations in flight per wave
constexpr int kTargetWorkgroups = 512;   // about two per CU
constexpr int kBK = 64;           // k elements per step
constexpr int kLdsRow = kBK + 8;  // padded LDS row (bf16 elements): 144 bytes

// STATS (LM head, one K split): the epilogue also reduces every output row over the workgroup's columns to the
// pair (max, sum exp(y - max)) and stores it at stats[row][column block], so that the vocabulary softmax
// statistics (Section II-A-1) come out of the projection and the logits need not be read again for them.
template <int MT, int DEPTH, int NW, bool STATS = false>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_skinny_kernel(const bf16_t* __restrict__ X,
                                                                   const bf16_t* __restrict__ Wp,
                                                                   float* __restrict__ P, int M, int N, int K,
                                                                   int k_per_split, int m_chunks,
                                                                   float2* __restrict__ stats = nullptr,
                                                                   int n_stat_blocks = 0) {
  __shared__ __attribute__((aligned(16))) bf16_t xs[2][MT * 16 * kLdsRow];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c = lane & 15;
  // More rows than one workgroup takes (MT * 16): the row chunks of one column block are separate
  // workgroups that read the same weights.  Workgroups are handed to the 8 XCDs round robin by
  // their linear index, so the chunks of a column block get indices that are 8 apart: they land on
  // the same XCD one after the other, and all but the first read the weights from that XCD's L2.
  int n_block = blockIdx.x, m_chunk = 0;
  if (m_chunks > 1) {
    const int xcd = blockIdx.x & 7, t = blockIdx.x >> 3;
    m_chunk = t % m_chunks;
    n_block = (t / m_chunks) * 8 + xcd;
    if (n_block * (16 * NW) >= N) return;      // padding of the grid to a multiple of 8 column blocks
  }
  const int n_tile = n_block * NW + wave;
  const int n0 = n_tile * 16;
  const int split = blockIdx.y;
  const int m0 = m_chunk * (MT * 16);
  const int k_begin = split * k_per_split;
  const int k_end = min(K, k_begin + k_per_split);
  const int n_steps = (k_end - k_begin) / kBK;

  // activation tile: MT*16 rows x 64 k = MT*128 chunks of 16 bytes
  constexpr int kChunks = MT * 128;
  constexpr int kGemmThreads = 64 * NW;
  constexpr int kPasses = (kChunks + kGemmThreads - 1) / kGemmThreads;
  uint4 xreg[DEPTH][kPasses];
  auto load_x = [&](int slot, int step) {
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int ch = tid + p * kGemmThreads;
      const int row = ch >> 3, col = (ch & 7) * 8;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (ch < kChunks && m0 + row < M)
        v = *reinterpret_cast<const uint4*>(X + (size_t)(m0 + row) * K + k_begin + step * kBK + col);
      xreg[slot][p] = v;
    }
  };
  auto store_x = [&](int buf, int slot) {
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int ch = tid + p * kGemmThreads;
      const int row = ch >> 3, col = (ch & 7) * 8;
      if (ch < kChunks) *reinterpret_cast<uint4*>(&xs[buf][row * kLdsRow + col]) = xreg[slot][p];
    }
  };

  // packed weights: block (n_tile, k_step) is 128 uint4; lane l reads uint4 l (first half of its
  // 16 k values) and uint4 64 + l (second half)
  const size_t w_step_stride = (size_t)(N / 16) * 128;
  const uint4* wbase = reinterpret_cast<const uint4*>(Wp) + (size_t)(k_begin / kBK) * w_step_stride + (size_t)n_tile * 128 + lane;
  uint4 wreg[DEPTH][2];
  auto load_w = [&](int slot, int step) {
    const uint4* p = wbase + (size_t)step * w_step_stride;
    if (m_chunks == 1) {      // read once: do not displace the activations and partial sums in L2
      wreg[slot][0] = stream_load(p);
      wreg[slot][1] = stream_load(p + 64);
    } else {                  // the other row chunks of the column block read the same weights from L2
      wreg[slot][0] = p[0];
      wreg[slot][1] = p[64];
    }
  };

  floatx4_t acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int d = 0; d < DEPTH; ++d)
    if (d < n_steps) {
      load_w(d, d);
      load_x(d, d);
    }

  for (int base = 0; base < n_steps; base += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int step = base + d;
      if (step < n_steps) {
        const int buf = step & 1;
        store_x(buf, d);
        __syncthreads();
        const uint4 w0 = wreg[d][0], w1 = wreg[d][1];
        if (step + DEPTH < n_steps) {
          load_w(d, step + DEPTH);
          load_x(d, step + DEPTH);
        }
        const bf16x8_t b0 = *reinterpret_cast<const bf16x8_t*>(&w0);
        const bf16x8_t b1 = *reinterpret_cast<const bf16x8_t*>(&w1);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const bf16_t* ap = &xs[buf][(mt * 16 + c) * kLdsRow + g * 16];
          const bf16x8_t a0 = *reinterpret_cast<const bf16x8_t*>(ap);
          const bf16x8_t a1 = *reinterpret_cast<const bf16x8_t*>(ap + 8);
          acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, acc[mt], 0, 0, 0);
          acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, acc[mt], 0, 0, 0);
        }
      }
    }
  }

  float* out = P + (size_t)split * M * N;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = m0 + mt * 16 + g * 4 + i;
      if (row < M) out[(size_t)row * N + n0 + c] = acc[mt][i];
    }
  }
  if constexpr (STATS) {
    // lanes (g, 0..15) hold the 16 columns of row mt*16 + g*4 + i: reduce over c, then over the waves
    __shared__ float2 st[NW][MT * 16];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = acc[mt][i];
        const float mx = row16_max(v);
        const float e = row16_sum(__expf(v - mx));
        if (c == 0) st[wave][mt * 16 + g * 4 + i] = make_float2(mx, e);
      }
    __syncthreads();
    if (tid < MT * 16 && m0 + tid < M) {
      float m = st[0][tid].x, sum = st[0][tid].y;
#pragma unroll
      for (int w = 1; w < NW; ++w) merge_stat(m, sum, st[w][tid].x, st[w][tid].y);
      stats[(size_t)(m0 + tid) * n_stat_blocks + n_block] = make_float2(m, sum);
    }
  }
}

// fp32 (v_mfma_f32_16x16x4_f32: fp32 products, fp32 sums).  The fp32 models are small (K of a few hundred, a few dozen
// rows), so a launch is bound by the latency of its loads, not by a rate: what counts is that no wave walks
// a long serial k chain, that enough waves run, and how many launches a layer has.  A workgroup's 8 waves are ks slices of K
// times 8 / ks column tiles of 16; a wave takes 16 columns and MT * 16 rows straight from global memory (lane (g, c) reads
// 16 bytes of row c at k + 4 g, the k order inside a 16-wide step being permuted alike in both operands), two to eight steps
// in flight, and the slices' sums meet in LDS in a fixed order.  2-layer model of width 256 / 1024 at 16 rows: a plain launch
// 4 us, with the rotation or the SwiGLU and the rows' factors 5.7, the residual forms 4.6 (K = 256) and 6 (K = 1024); the whole
// step 86 -> 74 us against separate kernels for norms, rotation and SwiGLU (25 launches, 15 now).
// grid (column groups, row chunks of MT * 16).
constexpr int kF32Waves = 8;
// LOADS: kWholeSteps where K is a multiple of 16 and the operands are 16-byte aligned, kVec4 where K is a multiple of 4,
// kElements otherwise.  (The modes of fused layers never have a K that is no multiple of 16.)
enum { kElements = 0, kVec4 = 1, kWholeSteps = 2 };
template <int LOADS>
__device__ __forceinline__ float4 load4_f32(const float* __restrict__ row, int k, int K) {
  if constexpr (LOADS == kWholeSteps) return *reinterpret_cast<const float4*>(row + k);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if constexpr (LOADS == kVec4) {
    if (k < K) v = *reinterpret_cast<const float4*>(row + k);
  } else {
    if (k + 0 < K) v.x = row[k + 0];
    if (k + 1 < K) v.y = row[k + 1];
    if (k + 2 < K) v.z = row[k + 2];
    if (k + 3 < K) v.w = row[k + 3];
  }
  return v;
}
// MODE: kF32Plain stores Y [M][N].  The others (gemm_common.h; up to 64 rows, one row chunk) take pairs of column tiles, or
// whole tiles, through LDS: kF32Qkv and kF32GateUp, whose input rows still need their factor, the two halves of a head's
// rotation pairs and the gate and up tile of 16 features, kF32Head tiles of the logits, kF32Residual of the residual stream.
enum { kF32Plain = 0, kF32Qkv = 1, kF32GateUp = 2, kF32Residual = 3, kF32Head = 4 };
template <int MT, int LOADS, int MODE>
__global__ __launch_bounds__(64 * kF32Waves) void gemm_f32_kernel(const float* __restrict__ X,
                                                                  const float* __restrict__ W, float* __restrict__ Y,
                                                                  int M, int N, int K, int ks_log2, int k_per, RowNorm norm,
                                                                  QkvOut qkv, ResidualOut res) {
  constexpr bool PAIRS = MODE == kF32Qkv || MODE == kF32GateUp, NORM = PAIRS || MODE == kF32Head;
  __shared__ float red[kF32Waves][MT * 256];
  __shared__ float factor[MT * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int ks = 1 << ks_log2, tiles_per_wg = kF32Waves >> ks_log2;
  const int tile = blockIdx.x * tiles_per_wg + (wave >> ks_log2), slice = wave & (ks - 1);
  const int half_log2 = MODE == kF32Qkv ? (qkv.hd == 128 ? 2 : 1) : 0;      // 16-column tiles of half a head
  // first column of a tile; tiles 2 p and 2 p + 1 of a pair
  auto first_column = [&](int t) {
    if constexpr (MODE == kF32Qkv) {
      const int pair = t >> 1, head = pair >> half_log2;
      return head * qkv.hd + (pair - (head << half_log2)) * 16 + (t & 1) * (qkv.hd >> 1);
    } else if constexpr (MODE == kF32GateUp) {
      return (t >> 1) * 16 + (t & 1) * (N >> 1);
    } else {
      return t * 16;
    }
  };
  const int n0 = first_column(tile);
  const int m0 = blockIdx.y * (MT * 16);
  const int k_begin = slice * k_per, k_end = min(K, k_begin + k_per);
  RowFactors<MT * 16, kF32Waves> factors;
  if constexpr (NORM) factors.load(norm, wave, lane, m0, M - m0);
  // what the epilogue needs from memory for this lane's first element, fetched before the products
  const int e_t = tid / (MT * 256), e_o = tid - e_t * (MT * 256), e_row = m0 + (e_o >> 4);
  int4 e_slot = make_int4(0, 0, 0, 0);
  float2 e_rope = make_float2(0.f, 0.f), e_res = e_rope;
  if constexpr (MODE == kF32Qkv) {
    const int pair = blockIdx.x * (tiles_per_wg / 2) + e_t;
    if (e_t < tiles_per_wg / 2 && e_row < M && pair * 32 < N) {
      e_slot = qkv.row_slot[e_row];
      e_rope = qkv.rope[(size_t)e_row * (qkv.hd >> 1) + (pair & ((1 << half_log2) - 1)) * 16 + (e_o & 15)];
    }
  }
  if constexpr (MODE == kF32Residual) {
    const int col = (blockIdx.x * tiles_per_wg + e_t) * 16 + (e_o & 15);
    if (e_t < tiles_per_wg && e_row < M && col < N) e_res = make_float2(res.x[(size_t)e_row * N + col], res.norm[col]);
  }
  // rows and columns past the end re-read the last one; their sums are not stored
  const float* wrow = W + (size_t)min(n0 + c, N - 1) * K;
  const float* xrow[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) xrow[mt] = X + (size_t)min(m0 + mt * 16 + c, M - 1) * K;
  // MT = 1: four accumulators, so that a product does not wait for the one before it
  constexpr int CHAINS = MT == 1 ? 4 : 1;
  floatx4_t part[MT][CHAINS];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int j = 0; j < CHAINS; ++j) part[mt][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  constexpr int U = MT == 4 ? 2 : MT == 2 ? 4 : 8;      // steps in flight
  float4 w[U], x[U][MT];
  auto load_steps = [&](int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (a step past the slice's end is neither read nor used, or reads zeros: its bound is the slice's end)
      if (LOADS == kWholeSteps && k0 + 16 * u >= k_end) break;
      const int k = k0 + 16 * u + 4 * g;
      w[u] = load4_f32<LOADS>(wrow, k, k_end);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) x[u][mt] = load4_f32<LOADS>(xrow[mt], k, k_end);
    }
  };
  if (k_begin < k_end) load_steps(k_begin);
  if constexpr (NORM) factors.store(norm, wave, lane, factor);
  for (int k0 = k_begin; k0 < k_end; k0 += 16 * U) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (LOADS != kWholeSteps || k0 + 16 * u < k_end)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            part[mt][j % CHAINS] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&x[u][mt])[j],
                                                                        reinterpret_cast<const float*>(&w[u])[j], part[mt][j % CHAINS], 0, 0, 0);
    if (k0 + 16 * U < k_end) load_steps(k0 + 16 * U);
  }
  floatx4_t acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = CHAINS == 4 ? (part[mt][0] + part[mt][1]) + (part[mt][CHAINS - 2] + part[mt][CHAINS - 1]) : part[mt][0];
  // register i of lane (g, c) is row 4 g + i, column c of the tile
  if constexpr (MODE == kF32Plain) {
    if (ks == 1) {
      if (n0 + c < N) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = m0 + mt * 16 + g * 4 + i;
            if (row < M) Y[(size_t)row * N + n0 + c] = acc[mt][i];
          }
      }
      return;
    }
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][(mt * 16 + g * 4 + i) * 16 + c] = acc[mt][i];
  __syncthreads();
  // element o of tile t of the workgroup
  auto sum_of = [&](int t, int o) {
    float sum = red[t * ks][o];
#pragma unroll
    for (int s = 1; s < kF32Waves; ++s) sum += s < ks ? red[min(t * ks + s, kF32Waves - 1)][o] : 0.f;
    return sum;
  };
  if constexpr (PAIRS) {
    for (int e = tid; e < tiles_per_wg / 2 * MT * 256; e += 64 * kF32Waves) {
      const int p = e / (MT * 256), o = e - p * (MT * 256);
      const int row = m0 + (o >> 4), pair = blockIdx.x * (tiles_per_wg / 2) + p;
      if (row >= M || pair * 32 >= N) continue;
      const float f = factor[o >> 4], a = sum_of(2 * p, o) * f, b = sum_of(2 * p + 1, o) * f;
      if constexpr (MODE == kF32GateUp) {
        Y[(size_t)row * (N >> 1) + pair * 16 + (o & 15)] = a / (1.0f + expf(-a)) * b;
      } else {
        const int head = pair >> half_log2, i = (pair - (head << half_log2)) * 16 + (o & 15);
        const bool first = e == tid;
        store_qkv_pair<float>(qkv, row, head, i, a, b, first ? e_slot : qkv.row_slot[row],
                              first ? e_rope : qkv.rope[(size_t)row * (qkv.hd >> 1) + i]);
      }
    }
    return;
  }
  for (int e = tid; e < tiles_per_wg * MT * 256; e += 64 * kF32Waves) {
    const int t = e / (MT * 256), o = e - t * (MT * 256);
    const int row = m0 + (o >> 4), col = (blockIdx.x * tiles_per_wg + t) * 16 + (o & 15);
    const float sum = sum_of(t, o);
    if constexpr (MODE == kF32Residual) {
      float v = 0.f;
      if (row < M && col < N) {
        const float2 xn = e == tid ? e_res : make_float2(res.x[(size_t)row * N + col], res.norm[col]);
        v = xn.x + sum;
        res.x[(size_t)row * N + col] = v;
        static_cast<float*>(res.h)[(size_t)row * N + col] = v * xn.y;
      }
      const float sq = row16_sum(v * v);      // (16 lanes share a row and a tile)
      if ((o & 15) == 0 && row < M && col < N) res.squares[(size_t)row * (N >> 4) + (col >> 4)] = sq;
    } else {
      if (row < M && col < N) Y[(size_t)row * N + col] = MODE == kF32Head ? sum * factor[o >> 4] : sum;
    }
  }
}

// Row-major [N][K] bf16 -> tile-packed [K/64][N/16][2][64][8]: one thread moves one 16-byte piece.
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                          int N, int K) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;      // destination uint4 index
  const size_t total = (size_t)N * K / 8;
  if (idx >= total) return;
  const int lane = (int)(idx & 63), half = (int)((idx >> 6) & 1);
  const size_t block = idx >> 7;
  const int n_tiles = N / 16;
  const int n_tile = (int)(block % n_tiles), k_step = (int)(block / n_tiles);
  const int g = lane >> 4, c = lane & 15;
  const size_t row = (size_t)n_tile * 16 + c;
  const int k = k_step * kBK + g * 16 + half * 8;
  dst[idx] = src[(row * K + k) / 8];
}

}  // namespace

gs_status launch_pack_weight(const void* src, void* dst, int N, int K, hipStream_t stream) {
  const size_t total = (size_t)N * K / 8;
  pack_weight_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(static_cast<const uint4*>(src),
                                                                          static_cast<uint4*>(dst), N, K);
  GS_LAUNCH_CHECK("pack_weight");
  return GS_OK;
}

// Which bf16 kernel serves a shape, and how the launch is cut.
struct GemmPlan {
  enum Kind {
    kSkinny,      // column counts that are no multiple of 128, and small matrices of a few rows (wide_serves)
    kWide         // gemm_wide.hip: everything else
  } kind;
  int mt;         // row tiles per workgroup
  int m_chunks;   // row chunks (separate workgroups)
  int splits;     // K splits
  int k_per;      // k elements per split (multiple of 64)
  WidePlan wide;
};

// Whether the wide kernel serves a shape.  Up to 64 rows it takes the projections without K splits and the large ones: where the
// 64-column workgroups and 512-element K splits of the skinny kernel leave at most one workgroup to a compute unit, a launch is
// over before the wide kernel's three buffers and exchange of K groups pay.  Isolated launches, skinny and wide, us at 20 / 64 rows:
// 1024 x 4096 5.3 / 6.0 and 6.7 / 8.1, 2048 x 2048 5.3 / 6.0 and 6.6 / 8.0, 4096 x 2048 7.2 / 7.8 and 7.5 / 8.8; beyond the line 1536 x 6144
// 7.9 / 9.3 and 7.5 / 9.1, 3072 x 3072 7.9 / 9.6 and 7.6 / 9.1.  Nor with fewer than eight blocks of 128 columns, which its grid leaves
// on as many XCDs (512 x 20480 8.8 / 11.3 and 12.9 / 16.3).  Larger ones gain in the step as well by fewer partial results: 4 layers of the 8B
// shape at 24 / 32 / 60 rows 649 / 648 / 707 us -> 615 / 630 / 688, 2 layers of the 70B shape at 24 / 60 rows 996 / 1049 -> 912 / 989.
bool wide_serves(int M, int N, int K) {
  if (N % 128 != 0) return false;
  if (M > 64 || wide_plan(M, N, K, kForSums).splits == 1) return true;
  return N >= 1024 && (long)(N / 64) * (K / 512) > 256;
}

static GemmPlan gemm_plan(int M, int N, int K, PlanFor use = kForSums) {
  GemmPlan p;
  const int tiles = ceil_div(M, 16);
  int n_blocks;
  if (N % 128 == 0) p.wide = wide_plan(M, N, K, use);
  if (wide_serves(M, N, K)) {
    p.kind = GemmPlan::kWide;
    p.mt = p.wide.mt;
    p.m_chunks = p.wide.m_chunks;
    p.splits = p.wide.splits;
    p.k_per = p.wide.k_per;
    return p;
  } else {
    p.kind = GemmPlan::kSkinny;
    p.mt = tiles <= 1 ? 1 : tiles <= 2 ? 2 : tiles <= 4 ? 4 : 8;
    n_blocks = N / (16 * kSkinnyWaves);
  }
  p.m_chunks = ceil_div(tiles, p.mt);
  const int wgs = n_blocks * p.m_chunks;
  int want = (kTargetWorkgroups + wgs / 2) / wgs;                // about two workgroups per CU
  const int max_s = K / 512 > 0 ? K / 512 : 1;             // at least 8 steps per split
  int s = want < max_s ? want : max_s;
  if (s < 1) s = 1;
  p.k_per = ceil_div(ceil_div(K, s), kBK) * kBK;
  p.splits = ceil_div(K, p.k_per);
  return p;
}

int gemm_w4_splits(int M, int N, int K);
gs_status launch_gemm_w4(const void* X, const void* Wpacked, float* P, int M, int N, int K, hipStream_t stream);
bool w4_gate_up_fused(int M, int F);
gs_status launch_gemm_w4_gate_up(const void* X, const void* Wpacked, void* act, int M, int F, int K, hipStream_t stream);

// Number of K splits the projection kernel will use for this shape (1 for fp32).
int gemm_splits(int dtype, int M, int N, int K) {
  if (M <= 0) return 1;
  if (dtype == GS_W4) return gemm_w4_splits(M, N, K);
  if (dtype != GS_BF16) return 1;
  return gemm_plan(M, N, K).splits;
}

template <bool STATS>
static void launch_skinny(const GemmPlan& p, const bf16_t* x, const bf16_t* w, float* P, int M, int N, int K,
                          float2* stats, int n_stat_blocks, hipStream_t stream) {
  constexpr int NW = kSkinnyWaves;
  const int n_blocks = N / (16 * NW);
  const int gx = p.m_chunks > 1 ? ceil_div(n_blocks, 8) * 8 * p.m_chunks : n_blocks;
  const dim3 grid(gx, p.splits, 1);
#define GS_SKINNY(MT_, CHUNKS_)                                                                                     \
  gemm_bf16_skinny_kernel<MT_, kSkinnyDepth, NW, STATS><<<grid, 64 * NW, 0, stream>>>(x, w, P, M, N, K, p.k_per,     \
                                                                                    CHUNKS_, stats, n_stat_blocks)
  switch (p.mt) {
    case 1: GS_SKINNY(1, 1); break;
    case 2: GS_SKINNY(2, 1); break;
    case 4: GS_SKINNY(4, 1); break;
    default: GS_SKINNY(8, p.m_chunks);
  }
#undef GS_SKINNY
}

// Whether the gate/up projection of this shape runs with the SwiGLU fused: 4-bit where its kernel does; bf16 up to 64 rows
// and where the whole sums take no longer.
bool gate_up_fused(int dtype, int M, int F, int K) {
  if (dtype == GS_W4) return M > 0 && w4_gate_up_fused(M, F);
  if (dtype != GS_BF16 || M <= 0 || F % 64 != 0 || K % kBK != 0) return false;
  return wide_gate_up_fused(M, 2 * F, K);      // (2 F is a multiple of 128)
}

// Whether the QKV projection of this shape leaves Q, K and V in their places (launch_gemm_qkv): bf16 of many rows, operands that direct
// loads of 16 bytes into LDS can take, places that its stores of 4 bytes (Q, K) and 8 bytes (V) can.
bool qkv_fused(int dtype, const void* X, const void* W, const QkvOut& out, int M, int K) {
  auto aligned = [](const void* p, int bytes) { return reinterpret_cast<uintptr_t>(p) % bytes == 0; };
  return dtype == GS_BF16 && K % kBK == 0 && aligned(X, 16) && aligned(W, 16) && aligned(out.q, 4) && aligned(out.k_pages, 4) &&
         aligned(out.v_pages, 8) && block_qkv_fused(M, (out.n_heads + 2 * out.n_kv) * out.hd, K);
}

// Q, K and V of M rows, rotated and stored; only for shapes qkv_fused accepts.
gs_status launch_gemm_qkv(const void* X, const void* W, const QkvOut& out, int M, int K, hipStream_t stream) {
  const int N = (out.n_heads + 2 * out.n_kv) * out.hd;
  return launch_block_qkv(wide_plan(M, N, K, kForHeads), static_cast<const bf16_t*>(X),
                          static_cast<const bf16_t*>(W), out, M, N, K, stream);
}

// act [M][F] (bf16) = silu(X Wg^T) * (X Wu^T), W = [Wg; Wu] packed; only for shapes gate_up_fused accepts.
gs_status launch_gemm_gate_up(int dtype, const void* X, const void* W, void* act, int M, int F, int K,
                              hipStream_t stream) {
  if (dtype == GS_W4) return launch_gemm_w4_gate_up(X, W, act, M, F, K, stream);
  const bf16_t* x = static_cast<const bf16_t*>(X);
  const bf16_t* w = static_cast<const bf16_t*>(W);
  // (2 F is a multiple of 128)
  return launch_wide_gate_up(wide_plan(M, 2 * F, K, kForWholeSums), x, w, static_cast<bf16_t*>(act), M, 2 * F, K, stream);
}

// Number of column blocks per row of the statistics that launch_gemm_stats writes for this shape, or 0 where
// the projection of this shape does not emit them (fp32 and 4-bit models, shapes that need a K split).
int gemm_stat_blocks(int dtype, int M, int N, int K) {
  if (dtype != GS_BF16 || M <= 0) return 0;
  const GemmPlan p = gemm_plan(M, N, K, kForStats);
  if (p.splits != 1) return 0;
  return p.kind == GemmPlan::kWide ? p.wide.n_blocks : N / (16 * kSkinnyWaves);
}

// Y [M][N] = X W^T (one K split) and stats [M][gemm_stat_blocks] = per row and column block (max, sum exp(y - max)).
gs_status launch_gemm_stats(const void* X, const void* W, float* Y, void* stats, int M, int N, int K,
                            hipStream_t stream) {
  const GemmPlan p = gemm_plan(M, N, K, kForStats);
  const bf16_t* x = static_cast<const bf16_t*>(X);
  const bf16_t* w = static_cast<const bf16_t*>(W);
  float2* st = static_cast<float2*>(stats);
  const int nb = gemm_stat_blocks(GS_BF16, M, N, K);
  if (nb == 0) return fail(GS_EUNSUPPORTED, "this projection shape does not emit softmax statistics");
  if (p.kind == GemmPlan::kWide) return launch_wide_stats(p.wide, x, w, Y, st, M, N, K, stream);
  launch_skinny<true>(p, x, w, Y, M, N, K, st, nb, stream);
  GS_LAUNCH_CHECK("gemm_bf16_stats");
  return GS_OK;
}

template <int MODE>
static void launch_f32(const float* x, const float* w, float* y, int M, int N, int K, const RowNorm& norm, const QkvOut& qkv,
                       const ResidualOut& res, hipStream_t stream) {
  static_assert(kMaxRowsF32 <= 64, "one row chunk of four tiles");
  const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
  const int chunks = ceil_div(M, 16 * mt), tiles = ceil_div(N, 16);
  // K slices: doubled until the launch has a workgroup per CU, as long as a slice keeps a 16-wide step of its own (and a
  // workgroup that takes pairs of tiles has two)
  constexpr int kMost = MODE == kF32Qkv || MODE == kF32GateUp ? kF32Waves / 2 : kF32Waves;
  int ks_log2 = 0;
  while ((1 << ks_log2) < kMost && ceil_div(tiles, kF32Waves >> ks_log2) * chunks < 256 && (32 << ks_log2) <= K) ++ks_log2;
  const int ks = 1 << ks_log2;
  const int k_per = ceil_div(ceil_div(K, ks), 16) * 16;
  const dim3 grid(ceil_div(tiles, kF32Waves / ks), chunks);
  const bool aligned = reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0;
#define GS_F32(MT_, LOADS_) \
  gemm_f32_kernel<MT_, LOADS_, MODE><<<grid, 64 * kF32Waves, 0, stream>>>(x, w, y, M, N, K, ks_log2, k_per, norm, qkv, res)
#define GS_F32_ROWS(LOADS_)           \
  if (mt == 1) GS_F32(1, LOADS_);     \
  else if (mt == 2) GS_F32(2, LOADS_); \
  else GS_F32(4, LOADS_);
  if (aligned && K % 16 == 0) {
    GS_F32_ROWS(kWholeSteps)
  } else {
    if constexpr (MODE == kF32Plain) {
      if (aligned && K % 4 == 0) {
        GS_F32_ROWS(kVec4)
        return;
      }
    }
    GS_F32_ROWS(kElements)
  }
#undef GS_F32_ROWS
#undef GS_F32
}

// Whether a block of M rows runs a layer in the launches below (see RowNorm); hq = heads x head size, qkv: columns of the QKV
// projection.  fp32: one row chunk; the tiles of the QKV and gate/up projections come in pairs, the sums of squares in whole
// 16-byte loads.
bool rows_fused(int dtype, int M, int d, int hq, int qkv, int F) {
  if (M <= 0 || d > kRowNormMaxWidth || d % 64 != 0) return false;
  if (dtype == GS_F32) return M <= kMaxRowsF32 && F % 16 == 0;
  // bf16: up to 16 rows, 8 where a workgroup has 32 columns; beyond, K splits and separate norms are faster (8B shape, 4 layers, us
  // fused and not: 5 rows 545 / 590, 16 rows 590 / 600, 20 rows 623 / 609; 70B shape, 2 layers: 5 rows 898 / 904, 12 rows
  // 927 / 912).  A K of many times the columns wants K splits, few workgroups would stream it alone, and more so the more rows they
  // read beside it: F up to eight times d, heads and F together up to ten times (at least 10240) for 8 rows and eight times (at
  // least 9216) for more.  Replayed calls of 4 layers at 8 / 16 rows, fused to not, F = 4 d: hq = 4 d 0.92 / 0.97 at d = 1024 and 0.94 / 1.00 at
  // 2048, 6 d 0.94 / 1.00 and 0.97 / 1.03, 8 d 1.00 / 1.06 at 1024, 16 d 1.16 / 1.23 at 1024; hq = d, F = 8 d 0.92 / 0.96 at 1024, 0.99 / 1.06 at 2048.
  // A QKV projection of up to 16384 columns is one workgroup per compute unit; more start a second round, which only pays for up
  // to 8 rows of wide models (18432 columns: d = 512 1.07 / 1.14, 2048 1.00 / 1.05, 3072 1.01 / 1.06; 24576 at 4096 0.98 / 1.02).
  if (dtype == GS_BF16) {
    const bool few = M <= kMaxRows / 2;
    return M <= (d <= 4096 ? kMaxRows : kMaxRows / 2) && F <= 8 * d && hq + F <= (few ? std::max(10 * d, 10240) : std::max(8 * d, 9216)) &&
           (qkv <= 16384 || (few && d >= 4096));
  }
  return false;
}
gs_status launch_bf16_rows_qkv(const bf16_t* h, const bf16_t* w, const RowNorm& norm, const QkvOut& out, int M, int K, hipStream_t stream);
gs_status launch_bf16_rows_residual(const bf16_t* in, const bf16_t* w, const ResidualOut& out, int M, int N, int K, hipStream_t stream);
// More rows would be left out, or overrun the sums of squares.
static gs_status check_rows(int dtype, int M) {
  const int most = dtype == GS_BF16 ? kMaxRows : kMaxRowsF32;
  return M <= most ? GS_OK : fail(GS_EUNSUPPORTED, "%d rows in a layer of at most %d", M, most);
}
// bf16: h, attn and act of these calls are in fragment order, but for the h that the gate/up projection reads
gs_status launch_rows_qkv(int dtype, const void* h, const void* w, const RowNorm& norm, const QkvOut& out, int M, int K,
                          hipStream_t stream) {
  if (gs_status st = check_rows(dtype, M); st != GS_OK) return st;
  if (dtype == GS_BF16)
    return launch_bf16_rows_qkv(static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(w), norm, out, M, K, stream);
  const int N = (out.n_heads + 2 * out.n_kv) * out.hd;
  launch_f32<kF32Qkv>(static_cast<const float*>(h), static_cast<const float*>(w), nullptr, M, N, K, norm, out, ResidualOut{}, stream);
  GS_LAUNCH_CHECK("rows_qkv");
  return GS_OK;
}
gs_status launch_rows_gate_up(int dtype, const void* h, const void* w, const RowNorm& norm, void* act, int M, int F, int K,
                              hipStream_t stream) {
  if (gs_status st = check_rows(dtype, M); st != GS_OK) return st;
  if (dtype == GS_BF16)
    return launch_wide_gate_up_norm(wide_plan(M, 2 * F, K, kForWholeSums), static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(w), norm,
                                    static_cast<bf16_t*>(act), M, 2 * F, K, stream);
  launch_f32<kF32GateUp>(static_cast<const float*>(h), static_cast<const float*>(w), static_cast<float*>(act), M, 2 * F, K, norm,
                         QkvOut{}, ResidualOut{}, stream);
  GS_LAUNCH_CHECK("rows_gate_up");
  return GS_OK;
}
// Logits of rows that still need their factor: fp32 (the others take a norm of their own, their LM heads being the plain ones).
gs_status launch_rows_head_f32(const float* h, const float* w, const RowNorm& norm, float* logits, int M, int N, int K, hipStream_t stream) {
  if (gs_status st = check_rows(GS_F32, M); st != GS_OK) return st;
  launch_f32<kF32Head>(h, w, logits, M, N, K, norm, QkvOut{}, ResidualOut{}, stream);
  GS_LAUNCH_CHECK("rows_head");
  return GS_OK;
}
gs_status launch_rows_residual(int dtype, const void* in, const void* w, const ResidualOut& out, int M, int N, int K,
                               hipStream_t stream) {
  if (gs_status st = check_rows(dtype, M); st != GS_OK) return st;
  if (dtype == GS_BF16)
    return launch_bf16_rows_residual(static_cast<const bf16_t*>(in), static_cast<const bf16_t*>(w), out, M, N, K, stream);
  launch_f32<kF32Residual>(static_cast<const float*>(in), static_cast<const float*>(w), nullptr, M, N, K, RowNorm{}, QkvOut{}, out,
                           stream);
  GS_LAUNCH_CHECK("rows_residual");
  return GS_OK;
}

// P [splits][M][N] fp32 partial sums of X [M][K] * W[N][K]^T (W tile-packed for bf16, packed 4-bit for
// GS_W4 with bf16 activations, row-major for fp32).
gs_status launch_gemm(int dtype, const void* X, const void* W, float* P, int M, int N, int K, hipStream_t stream) {
  if (M <= 0) return GS_OK;
  if (dtype == GS_W4) return launch_gemm_w4(X, W, P, M, N, K, stream);
  if (dtype == GS_BF16) {
    const GemmPlan p = gemm_plan(M, N, K);
    const bf16_t* x = static_cast<const bf16_t*>(X);
    const bf16_t* w = static_cast<const bf16_t*>(W);
    if (p.kind == GemmPlan::kWide) return launch_wide(p.wide, x, w, P, M, N, K, stream);
    launch_skinny<false>(p, x, w, P, M, N, K, nullptr, 0, stream);
    GS_LAUNCH_CHECK("gemm_bf16");
  } else {
    launch_f32<kF32Plain>(static_cast<const float*>(X), static_cast<const float*>(W), P, M, N, K, RowNorm{}, QkvOut{}, ResidualOut{}, stream);
    GS_LAUNCH_CHECK("gemm_f32");
  }
  return GS_OK;
}

}  // namespace gs
