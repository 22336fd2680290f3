// bf16 projections (MFMA): the packed weight stream of gemm.hip with a software pipeline
// that leaves neither the matrix pipe nor the stream waiting.
//
// What bounds it: up to about 130 rows the weight stream (HBM), above the matrix pipe together with the LDS
// reads of the activations: a 1 KB activation fragment feeds NT MFMAs of 16 cycles, so at NT = 2 the LDS delivers its
// limit of 128 bytes per cycle and compute unit.
// The predecessor of this kernel (two LDS buffers, fragments read where they are used, all loads of a step in one
// burst behind the barrier) was held up by neither: the loads' addresses, the LDS stores and the first fragment reads
// of a step ran while the matrix pipe was idle, and the compiler sank the loads to the end of the step, where the
// next one waited for them.  Here
//   * a step (64 of k) is a sequence of MT blocks, one per row tile, each of which issues its share of the next weight
//     loads, one piece of the next activation tile (LDS store of the piece that has landed, load of the one after)
//     and the fragment reads of the row tile two blocks ahead, and then its 2 NT MFMAs; a scheduling barrier after
//     every block keeps the compiler from undoing that order
//   * the activation tile lives in three LDS buffers, so that the fragments of the next step's first two blocks can be
//     read before the barrier that ends the step (the buffer they come from was published one barrier earlier)
//   * activation rows are 128 bytes in LDS, their 16-byte pieces XOR-swizzled (row_swizzle): conflict-free reads
//   * loads are buffer loads: the descriptor moves with k on the scalar unit and the lane offsets are constant, so a
//     load costs no vector instruction for its address; rows past the end read as zero by the descriptor's range
// The shapes: WM x WN waves, each with MT x NT tiles of 16 x 16, KG groups of them that share K (which one a launch takes: kWideShapes):
//   1 x 8 (256 columns, wide matrices), up to 192 rows: no weight byte is loaded twice
//   1 x 4 (128 columns) with KG = 2, all rows (up to 160) in one workgroup: the two halves of K in one workgroup, their sums meet
//     in LDS: as many waves as 1 x 8 without halving the workgroups of a narrower matrix, and half the partial results of a
//     further K split (which the gate/up projection, whose epilogue applies the SwiGLU, must not have)
//   1 x 2 (64 columns) with KG = 4, up to 64 rows: the same for matrices of 4096 columns or so, which would need eight K splits
//     (small matrices of up to 64 rows stay on the kernel of gemm.hip: wide_serves)
//   1 x 4 (128 columns) in row chunks of 64 to 192 rows, two workgroups per compute unit: narrow matrices and middling row counts,
//     where the time of one workgroup is the time of the launch
// More rows, where what the waves load for themselves is the bound: gemm_block.hip.
// Measured inside a verification step (us per launch; predecessor in brackets), N x K:
//   50 rows    gate/up 28672 x 4096 38.4 (46.0) = 6.1 TB/s, LM head 128256 x 4096 179 (188)
//   98 rows    gate/up 57344 x 8192 142 (181) = 6.6 TB/s, 8192 x 28672 and 8192 x 8192 55 (60) on average, 10240 x 8192
//              36.4 (37.9), LM head 128256 x 8192 331 (455) = 6.3 TB/s
#include "common.h"
#include "device_types.h"
#include "gemm_common.h"
#include <algorithm>

namespace gs {
namespace {

typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

// MODE: kPlain stores the fp32 sums [split][M][N] at P; kGateUp (one split): the wave's tiles are NT / 2 feature tiles of
// the gate half and the same ones of the up half of a [2F][K] matrix (N = 2F), and act[M][F] = silu(gate) * up is
// stored as bf16 at P; kGateUpNorm: the same of rows that still need their factor (RowNorm), act in fragment order; kStats (one split): also (max, sum exp) of every row over the workgroup's columns.
// DB, DA: steps of weights and of activations held in registers: three and one (a step in use, two of weights on their way).  More loads in
// flight queue up in the memory system and delay each other: whole steps, us, with 5 / 4 / 3 / 2 of weights: 8 servers of the 8B shape 4104 / 4066 /
// 4022 / 4011, 16 of the 70B shape 1852 / 1840 / 1827 / 1831, one server 888 / 884 / 881; two steps of activations instead of one: 4089 and 4058.
// POL: cache policy of the weight loads (2: do not
// displace other lines; for weights that one workgroup reads once).
// 1-D grid: K splits x column blocks x row chunks.  Workgroups are handed to the 8 XCDs round robin by their index; an XCD takes a
// contiguous range of (split, column block, row chunk), so the row chunks of a column block run on one XCD, and all but the first find
// the weights in its L2.  No XCD has more than one workgroup more than another.  (Column blocks dealt to the XCDs one by one, rounded up
// to a multiple of 8, left XCDs idle where a matrix has a few: replayed launches of 304 / 1024 rows, us, that way -> this one:
// 1536 x 6144 17.2 -> 12.2 / 36.3 -> 25.5, 3584 x 3584 at 304 rows 23.6 -> 16.8, 512 x 20480 23.5 -> 15.3 / 49.3 -> 28.4; column counts that
// divide evenly are within 2 % but for the LM head 128256 x 4096, 53 rows 180 -> 172.5; 15 matrices x 13 rows 1.07 on average.)
template <int WM, int WN, int KG, int MT, int NT, int DB, int DA, int POL, int WPE, int MODE>
__global__ __launch_bounds__(64 * WM * WN * KG) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void gemm_bf16_wide_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Wp, float* __restrict__ P, int M, int N, int K,
    int k_per_split, int m_chunks, float2* __restrict__ stats, int n_stat_blocks, RowNorm norm) {
  constexpr bool GATE_UP = MODE == kGateUp || MODE == kGateUpNorm;
  static_assert(MT >= 2, "fragments are read two row tiles ahead");
  static_assert(DB % DA == 0, "the unrolled ring addresses the activation slots statically");
  static_assert(KG == 1 || MODE != kStats, "whole sums");
  constexpr int ROWS = WM * MT * 16, THREADS = 64 * WM * WN;       // of one K group
  constexpr int PASSES = (ROWS * 8 + THREADS - 1) / THREADS;
  constexpr int TILE = ROWS * 128;                                 // bytes of one activation buffer
  __shared__ __attribute__((aligned(16))) unsigned char xs_all[KG * 3 * TILE];
  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave_all / (WM * WN), wave = wave_all % (WM * WN);
  const int tid = threadIdx.x - kg * THREADS;
  unsigned char* xs = xs_all + kg * 3 * TILE;
  const int g = lane >> 4, c = lane & 15;
  const int item = xcd_item();
  const int m_chunk = item % m_chunks, column = item / m_chunks, n_blocks = N / (16 * NT * WN);
  const int split = column / n_blocks, n_block = column - split * n_blocks;
  const int wm = wave / WN, wn = wave % WN;
  const int n_tile0 = (n_block * WN + wn) * (GATE_UP ? NT / 2 : NT);
  const int m0 = m_chunk * ROWS;
  const int split_begin = split * k_per_split, split_end = min(K, split_begin + k_per_split);
  // the K groups take the halves of the split, rounded to steps; both run the same number of steps (barriers), a
  // step past the end multiplies zeros by zeros
  const int split_steps = (split_end - split_begin) / 64;
  const int n_steps = (split_steps + KG - 1) / KG;
  const int own_steps = min(n_steps, split_steps - kg * n_steps);
  const int k_begin = split_begin + (own_steps > 0 ? kg * n_steps * 64 : 0);
  const int last = max(own_steps - 1, 0);
  const char* xbase = reinterpret_cast<const char*>(X + (size_t)m0 * K + k_begin);
  const unsigned x_bytes = ((unsigned)min(ROWS, M - m0) * (unsigned)K - (unsigned)k_begin) * 2u;
  const size_t w_stride = (size_t)(N / 16) * 2048;
  const char* wbase = reinterpret_cast<const char*>(Wp) + (size_t)(k_begin / 64) * w_stride + (size_t)n_tile0 * 2048;
  const unsigned w_bytes = (unsigned)w_stride - (unsigned)n_tile0 * 2048u;
  unsigned xoff[PASSES], loff[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    // (a last pass with fewer pieces than lanes moves the last piece several times)
    const int ch = min(tid + p * THREADS, ROWS * 8 - 1), row = ch >> 3, piece = ch & 7;
    xoff[p] = (unsigned)row * (unsigned)K * 2u + piece * 16u;
    loff[p] = row * 128 + ((piece ^ row_swizzle(row)) << 4);
  }
  // a step past the K group's own end has an empty descriptor: it reads zeros
  auto x_rsrc = [&](int step) {
    const int s = min(step, last);      // (KG = 1: re-read, never used)
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(xbase + (size_t)s * 128), 0,
                                             (KG == 1 || step < own_steps) ? x_bytes - (unsigned)s * 128u : 0u, 0x00020000);
  };
  auto w_rsrc = [&](int step) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wbase + (size_t)min(step, last) * w_stride), 0,
                                             (KG == 1 || step < own_steps) ? w_bytes : 0u, 0x00020000);
  };
  __shared__ float factor[MODE == kGateUpNorm ? ROWS : 1];
  RowFactors<MODE == kGateUpNorm ? ROWS : 4, WM * WN * KG> factors;      // (one row chunk)
  if constexpr (MODE == kGateUpNorm) factors.load(norm, wave_all, lane, 0, M);
  uintx4_t xreg[DA][PASSES];
  uintx4_t wreg[DB][NT][2];
  const unsigned woff = lane * 16;
  const unsigned up_off = GATE_UP ? (unsigned)(N / 32) * 2048u - (unsigned)(NT / 2) * 2048u : 0u;
#define GS_LOAD_X(slot, p, r) xreg[slot][p] = __builtin_amdgcn_raw_buffer_load_b128(r, xoff[p], 0, 0)
  // piece i of the wave's weights of a step: tile i / 2, half i % 2
#define GS_LOAD_W(slot, i, r)                                                                                       \
  wreg[slot][(i) >> 1][(i) & 1] = __builtin_amdgcn_raw_buffer_load_b128(                                            \
      r, woff + (i) * 1024, (GATE_UP && (i) >= NT) ? up_off : 0u, POL)
  floatx4_t acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // fragment of row tile mt: lane (g, c) holds row c, pieces 2 g (first MFMA) and 2 g + 1 (second)
  const int a0 = (wm * MT * 16 + c) * 128 + (((2 * g) ^ row_swizzle(c)) << 4);
  const int a1 = (wm * MT * 16 + c) * 128 + (((2 * g + 1) ^ row_swizzle(c)) << 4);
  {
    uintx4_t r0[PASSES], r1[PASSES];
    auto rx0 = x_rsrc(0), rx1 = x_rsrc(1);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) r0[p] = __builtin_amdgcn_raw_buffer_load_b128(rx0, xoff[p], 0, 0);
#pragma unroll
    for (int d = 0; d < DB - 1; ++d) {
      auto rw = w_rsrc(d);
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i) GS_LOAD_W(d, i, rw);
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) r1[p] = __builtin_amdgcn_raw_buffer_load_b128(rx1, xoff[p], 0, 0);
#pragma unroll
    for (int d = 0; d < DA; ++d) {
      auto rx = x_rsrc(d + 2);
#pragma unroll
      for (int p = 0; p < PASSES; ++p) GS_LOAD_X(d, p, rx);
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) *reinterpret_cast<uintx4_t*>(&xs[loff[p]]) = r0[p];
    if constexpr (MODE == kGateUpNorm) factors.store(norm, wave_all, lane, factor);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) *reinterpret_cast<uintx4_t*>(&xs[TILE + loff[p]]) = r1[p];
  }
  __syncthreads();
  bf16x8_t an[2][2];      // fragments of the next two row tiles
  auto frag = [&](int buf, int mt, bf16x8_t (&a)[2]) {
    a[0] = *reinterpret_cast<const bf16x8_t*>(&xs[buf + a0 + mt * 2048]);
    a[1] = *reinterpret_cast<const bf16x8_t*>(&xs[buf + a1 + mt * 2048]);
  };
  frag(0, 0, an[0]);
  frag(0, 1, an[1]);
  int b0 = 0;             // byte offset of the current step's buffer
  constexpr int WB = (2 * NT + MT - 1) / MT > 2 ? (2 * NT + MT - 1) / MT : 2;      // weight loads per block (early blocks)
  constexpr int XB = (PASSES + MT - 1) / MT;                                       // activation pieces per block
  for (int base = 0;; base += DB) {
    bool done = false;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const int step = base + d;
      if (!done) {
        const int b1 = b0 == 2 * TILE ? 0 : b0 + TILE, b2 = b1 == 2 * TILE ? 0 : b1 + TILE;
        auto rx = x_rsrc(step + 2 + DA);
        auto rw = w_rsrc(step + DB - 1);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const bf16x8_t ac[2] = {an[0][0], an[0][1]};
          an[0][0] = an[1][0];
          an[0][1] = an[1][1];
          if (mt + 2 < MT) frag(b0, mt + 2, an[1]); else frag(b1, mt + 2 - MT, an[1]);
#pragma unroll
          for (int i = mt * WB; i < (mt + 1) * WB; ++i)
            if (i < 2 * NT) GS_LOAD_W((d + DB - 1) % DB, i, rw);
#pragma unroll
          for (int p = mt * XB; p < (mt + 1) * XB; ++p)
            if (p < PASSES) {
              *reinterpret_cast<uintx4_t*>(&xs[b2 + loff[p]]) = xreg[d % DA][p];
              GS_LOAD_X(d % DA, p, rx);
            }
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  ac[h], *reinterpret_cast<const bf16x8_t*>(&wreg[d % DB][nt][h]), acc[mt][nt], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        b0 = b1;
        done = step + 1 >= n_steps;
      }
    }
    if (done) break;
  }
#undef GS_LOAD_X
#undef GS_LOAD_W

  // The K groups share the epilogue: group mt % KG owns row tile mt, takes its sums from all groups in a fixed order and stores it.
  auto owned = [&](int mt) { return KG == 1 || mt % KG == kg; };
  if constexpr (KG > 1) {
    // (the last step's barrier: all reads of the activation buffers are done but for fragments nobody uses)
    static_assert(KG * 3 * TILE >= MT * NT * (KG - 1) * 16 * THREADS, "the sums that change hands fit the activation buffers");
    __syncthreads();
    floatx4_t* sums = reinterpret_cast<floatx4_t*>(xs_all);
    auto place = [&](int src, int mt, int nt) {      // what group src hands to the owner of row tile mt
      const int o = mt % KG;
      return ((mt * (KG - 1) + (src < o ? src : src - 1)) * NT + nt) * THREADS + tid;
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (!owned(mt))
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sums[place(kg, mt, nt)] = acc[mt][nt];
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (owned(mt))
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const floatx4_t own = acc[mt][nt];
          floatx4_t v = mt % KG == 0 ? own : sums[place(0, mt, nt)];
#pragma unroll
          for (int src = 1; src < KG; ++src) v += mt % KG == src ? own : sums[place(src, mt, nt)];
          acc[mt][nt] = v;
        }
  }
  const int row0 = m0 + wm * MT * 16;
  if constexpr (GATE_UP) {
    bf16_t* act = reinterpret_cast<bf16_t*>(P);
    const int F = N / 2;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + mt * 16 + g * 4 + i;
        if (owned(mt) && row < M) {
#pragma unroll
          for (int ft = 0; ft < NT / 2; ++ft) {
            const float f = MODE == kGateUpNorm ? factor[row - m0] : 1.0f;
            const float gt = MODE == kGateUpNorm ? acc[mt][ft][i] * f : acc[mt][ft][i];
            const float up = MODE == kGateUpNorm ? acc[mt][NT / 2 + ft][i] * f : acc[mt][NT / 2 + ft][i];
            const int col = (n_tile0 + ft) * 16 + c;
            act[MODE == kGateUpNorm ? packed_index(row, col, F) : (size_t)row * F + col] =
                float_to_bf16(gt / (1.0f + expf(-gt)) * up);
          }
        }
      }
    return;
  }
  float* out = P + (size_t)split * M * N;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row0 + mt * 16 + g * 4 + i;
      if (owned(mt) && row < M) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) out[(size_t)row * N + (n_tile0 + nt) * 16 + c] = acc[mt][nt][i];
      }
    }
  if constexpr (MODE == kStats) {
    static_assert(3 * TILE >= WN * ROWS * (int)sizeof(float2), "the statistics fit the activation buffers");
    float2* st = reinterpret_cast<float2*>(xs_all);      // [WN][ROWS]
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float mx = acc[mt][0][i];
#pragma unroll
        for (int nt = 1; nt < NT; ++nt) mx = fmaxf(mx, acc[mt][nt][i]);
        mx = row16_max(mx);
        float e = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) e += __expf(acc[mt][nt][i] - mx);
        e = row16_sum(e);
        if (c == 0) st[wn * ROWS + wm * MT * 16 + mt * 16 + g * 4 + i] = make_float2(mx, e);
      }
    __syncthreads();
    for (int r = tid; r < ROWS; r += THREADS)
      if (m0 + r < M) {
        float m = st[r].x, sum = st[r].y;
#pragma unroll
        for (int w = 1; w < WN; ++w) merge_stat(m, sum, st[w * ROWS + r].x, st[w * ROWS + r].y);
        stats[(size_t)(m0 + r) * n_stat_blocks + n_block] = make_float2(m, sum);
      }
  }
}

}  // namespace

// The shapes for more than 64 rows, of this kernel and (block) of gemm_block.hip, and what a launch takes with them (us), fitted to 18000
// launches of 22 matrices of 768 x 3072 to 57344 x 8192 and 70 to 2047 rows in every shape and several K splits (rms 7 %):
//   the larger of loop = steps x step time of the workgroups a compute unit has one after the other, and stream = weight bytes /
//   7.8 TB/s; 0.45 of the smaller; 0.085 x tiles per SIMD and workgroup for the epilogue; 0.39 per MB of partial results (written
//   here, read by the next kernel).
// A step takes single_us, of two workgroups at once (shapes that fit a compute unit twice) pair_us.  Row chunks read the weights again,
// from L2 for the most part: 0.27 of the stream each.  The shape of least modelled time is within 1 % of the fastest one on average over
// those matrices (worst 1.2), and 1.048x as fast as the shape that the same rule chose before the shapes of gemm_block.hip (worst 0.945:
// 8192 x 28672 at 160 rows 94.7 -> 100.2 us; best 1.37: 57344 x 8192 at 256 rows 257 -> 203).
struct WideShape {
  bool block;
  int wm, wn, kg, mt, nt;
  float single_us, pair_us;      // pair: 0 where a compute unit holds one workgroup
};
static const WideShape kWideShapes[] = {
    {false, 1, 4, 2, 6, 2, 0.394f, 0.f},     {false, 1, 4, 2, 8, 2, 0.490f, 0.f},     {false, 1, 4, 2, 10, 2, 0.578f, 0.f},
    {false, 1, 4, 1, 4, 2, 0.322f, 0.500f},  {false, 1, 4, 1, 6, 2, 0.389f, 0.601f},  {false, 1, 4, 1, 8, 2, 0.436f, 0.737f},
    {false, 1, 4, 1, 10, 2, 0.498f, 0.848f}, {false, 1, 4, 1, 12, 2, 0.563f, 0.992f}, {false, 1, 8, 1, 6, 2, 0.637f, 0.f},
    {false, 1, 8, 1, 8, 2, 0.719f, 0.f},     {false, 1, 8, 1, 10, 2, 0.854f, 0.f},    {false, 1, 8, 1, 12, 2, 0.936f, 0.f},
    {true, 2, 2, 1, 4, 4, 0.428f, 0.671f},   {true, 2, 2, 1, 4, 6, 0.450f, 0.f},      {true, 1, 4, 2, 8, 4, 0.585f, 0.f},
    {true, 1, 4, 2, 10, 4, 0.677f, 0.f},     {true, 1, 4, 2, 11, 4, 0.718f, 0.f},     {true, 4, 2, 1, 4, 7, 0.948f, 0.f},
    {true, 4, 2, 1, 4, 8, 0.949f, 0.f}};

static void cut_k(WidePlan& p, int K, int s) {
  p.k_per = ceil_div(ceil_div(K, s), 64) * 64;
  p.splits = ceil_div(K, p.k_per);
}

constexpr float kPartialUs = 0.39f * 64e-6f;      // of the 16 x 4 bytes that a column has per row tile and split

// The shape of kWideShapes and the K splits with the least time for more than 4 row tiles (N a multiple of 128).
static WidePlan fastest_shape(int tiles, int N, int K, PlanFor use) {
  constexpr long kCus = 256;
  const bool whole = use == kForWholeSums || use == kForHeads;
  WidePlan best{};
  for (const WideShape& w : kWideShapes) {
    const int cols = 16 * w.nt * w.wn;
    if (N % cols != 0 || (use == kForStats && cols % 128 != 0)) continue;
    if (use == kForHeads && (!w.block || w.nt % 2 != 0 || w.mt > 8)) continue;      // (more row tiles beside that epilogue spill)
    WidePlan p{w.wm, w.wn, w.kg, w.mt, w.nt, ceil_div(tiles, w.wm * w.mt), N / cols, 1, 0, w.block, 0.f};
    if (!w.block) {
      // where one workgroup has all rows, K groups are better than the same tile without; they are not for weights that several
      // workgroups read, nor 1 x 8 waves for more than two
      if (p.m_chunks > 1 ? w.kg == 2 || (w.wn == 8 && p.m_chunks > 2) : w.wn == 4 && w.kg == 1 && tiles <= 10) continue;
    } else if (tiles <= 8 && (cols > 128 || (long)N * K > 1L << 26)) {
      // one row chunk whose weights are the bound: straight into the registers (57344 x 8192 at 80 rows 142 us, here 155 to 167; 28672 x
      // 4096 at 112 rows 47 and 46, 4096 x 4096 at 80 rows 14.4 and 13.1)
      continue;
    }
    const bool pairs = w.pair_us > 0.f && (w.block || tiles > 12);
    const float units = 0.25f * (float)(w.mt * w.nt * w.wm * w.wn);
    const float stream = 2e-6f / 7.83f * (float)N * (float)K * (1.f + 0.267f * (float)(p.m_chunks - 1));
    const long blocks = (long)p.n_blocks * p.m_chunks;
    // K splits: as many as give every compute unit one workgroup (two where it holds two), at least 8 steps each
    for (long target = kCus; target <= (w.block && pairs && !whole && K >= 1024 ? 2 * kCus : kCus); target += kCus) {
      cut_k(p, K, whole ? 1 : std::max(1, std::min((int)(target / blocks), K / 512)));
      const long wgs = blocks * p.splits, per_cu = (wgs + kCus - 1) / kCus, last = wgs % (2 * kCus);
      const float steps_us = !pairs ? (float)per_cu * w.single_us
                                    : (float)(wgs / (2 * kCus)) * w.pair_us + (last == 0 ? 0.f : last <= kCus ? w.single_us : w.pair_us);
      const float loop = (float)(p.k_per / 64) * steps_us;
      const float us = std::max(loop, stream) + 0.446f * std::min(loop, stream) + 0.0855f * units * (float)per_cu +
                       kPartialUs * (float)p.splits * (float)tiles * (float)N;
      if (best.splits == 0 || us < best.us) {
        best = p;
        best.us = us;
      }
    }
  }
  return best;
}

WidePlan wide_plan(int M, int N, int K, PlanFor use) {
  const int tiles = ceil_div(M, 16);
  if (tiles <= 4) {
    WidePlan p{};
    p.wm = 1;
    p.nt = 2;
    p.mt = std::max(2, (tiles + 1) / 2 * 2);
    p.m_chunks = 1;
    // 256 columns per workgroup where that still leaves a workgroup for three compute units in four (28672 columns
    // of the 8B gate/up projection would leave 112); narrower matrices take 128
    p.wn = (N % 256 == 0 && N / 256 >= 192) ? 8 : 4;
    p.kg = p.wn == 8 ? 1 : 2;
    p.n_blocks = N / (32 * p.wn);
    cut_k(p, K, use == kForWholeSums ? 1 : std::max(1, std::min(256 / p.n_blocks, K / 512)));
    // Four K groups of 64 columns where that fills the chip with half of the K splits: half of the partial results
    // (four and fewer are not worth the larger share of the activations: 8192 x 28672 wants the two groups)
    const int blocks = N / 64, s4 = std::min(256 / blocks, K / 1024);
    if (p.splits > 4 && s4 > 1 && blocks * s4 >= 224) {
      p.wn = 2;
      p.kg = 4;
      p.n_blocks = blocks;
      cut_k(p, K, s4);
    }
    return p;
  }
  return fastest_shape(tiles, N, K, use);
}

bool wide_gate_up_fused(int M, int N, int K) {
  if (M <= 64) return true;
  const WidePlan whole = wide_plan(M, N, K, kForWholeSums), split = wide_plan(M, N, K, kForSums);
  // fused: no fp32 sums and one launch less (3 us)
  return split.splits == 1 || whole.us - kPartialUs * (float)ceil_div(M, 16) * (float)N <= split.us + 3.f;
}

bool block_qkv_fused(int M, int N, int K) {
  if (M <= 64 || N % 128 != 0) return false;
  const WidePlan whole = wide_plan(M, N, K, kForHeads), split = wide_plan(M, N, K, kForSums);
  // Its epilogue takes a little longer than storing fp32 sums (1024 rows of the 8B shape 51 -> 58 us per launch), in return for the launch that
  // would read them again (15), so only where the shape that serves it is modelled no slower than the plan, which is from the same shape
  // for the most part.  8B shape, 4 layers, us per pass at 800 / 1280 / 1800 rows 2294 -> 2240, 3235 -> 3216, 4668 -> 4637; beyond the line
  // 512 rows 1453 and 1450, 640 1857 both, 1500 3778 and 3849; 324 rows, 8 layers, 2627 and 2697.
  return whole.splits == 1 && whole.us <= split.us;
}

template <int MODE>
static gs_status launch_mode(const WidePlan& plan, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K,
                             float2* stats, const RowNorm& norm, hipStream_t stream) {
  WidePlan p = plan;
  if constexpr (MODE != kGateUpNorm) {
    if (p.block) {
      // (direct loads of 16 bytes into LDS want their addresses aligned; loads into registers do not)
      if (reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0)
        return launch_block(MODE, p, x, w, out, M, N, K, stats, stream);
      const int wn = MODE == kStats && p.n_blocks * 256 == N ? 8 : 4;      // (as many column blocks of statistics as planned)
      p = WidePlan{1, wn, 1, 8, 2, ceil_div(M, 128), N / (32 * wn), p.splits, p.k_per, false, 0.f};
    }
  }
  const int grid = p.n_blocks * p.m_chunks * p.splits;
#define GS_WIDE(WM, WN, KG, MT, NT, DB, DA, POL, WPE)                                                              \
  gemm_bf16_wide_kernel<WM, WN, KG, MT, NT, DB, DA, POL, WPE, MODE>                                                 \
      <<<grid, 64 * WM * WN * KG, 0, stream>>>(x, w, out, M, N, K, p.k_per, p.m_chunks, stats, p.n_blocks, norm)
  if constexpr (MODE == kGateUpNorm) {
    static_assert(kMaxRows <= 32, "two row tiles in one row chunk");
    if (p.wn == 8) GS_WIDE(1, 8, 1, 2, 2, 3, 1, 2, 2);
    else GS_WIDE(1, 4, 2, 2, 2, 3, 1, 2, 2);
    GS_LAUNCH_CHECK("gemm_bf16_wide");
    return GS_OK;
  }
  if constexpr (MODE != kGateUpNorm) {
  if (p.wn == 8) {
    switch (p.mt) {
      case 2: GS_WIDE(1, 8, 1, 2, 2, 3, 1, 2, 2); break;
      case 4: GS_WIDE(1, 8, 1, 4, 2, 3, 1, 2, 2); break;
      case 6: GS_WIDE(1, 8, 1, 6, 2, 3, 1, 2, 2); break;
      case 8: GS_WIDE(1, 8, 1, 8, 2, 3, 1, 2, 2); break;
      case 10: GS_WIDE(1, 8, 1, 10, 2, 3, 1, 2, 2); break;
      default: GS_WIDE(1, 8, 1, 12, 2, 3, 1, 2, 2);
    }
  } else if (MODE == kPlain && p.kg == 4) {
    if constexpr (MODE == kPlain) {
      if (p.mt == 2) GS_WIDE(1, 2, 4, 2, 2, 3, 1, 2, 2);
      else GS_WIDE(1, 2, 4, 4, 2, 3, 1, 2, 2);
    }
  } else if (MODE == kStats && p.m_chunks == 1 && p.mt == 12) {
    if constexpr (MODE == kStats) GS_WIDE(1, 4, 1, 12, 2, 3, 1, 2, 1);      // (spills where two workgroups share the registers)
  } else if (p.m_chunks == 1 && (MODE == kStats || p.kg == 2)) {
    // (the statistics take whole sums: one K group there, and two workgroups per compute unit)
    constexpr int KG = MODE == kStats ? 1 : 2;
    switch (p.mt) {
      case 2: GS_WIDE(1, 4, KG, 2, 2, 3, 1, 2, 2); break;
      case 4: GS_WIDE(1, 4, KG, 4, 2, 3, 1, 2, 2); break;
      case 6: GS_WIDE(1, 4, KG, 6, 2, 3, 1, 2, 2); break;
      case 8: GS_WIDE(1, 4, KG, 8, 2, 3, 1, 2, 2); break;
      default: GS_WIDE(1, 4, KG, 10, 2, 3, 1, 2, 2);
    }
  } else {
    switch (p.mt) {
      case 4: GS_WIDE(1, 4, 1, 4, 2, 3, 1, 0, 2); break;
      case 6: GS_WIDE(1, 4, 1, 6, 2, 3, 1, 0, 2); break;
      case 8: GS_WIDE(1, 4, 1, 8, 2, 3, 1, 0, 2); break;
      case 10: GS_WIDE(1, 4, 1, 10, 2, 3, 1, 0, 2); break;
      default: GS_WIDE(1, 4, 1, 12, 2, 3, 1, 0, 2);
    }
  }
  }
#undef GS_WIDE
  GS_LAUNCH_CHECK("gemm_bf16_wide");
  return GS_OK;
}

gs_status launch_wide(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K,
                      hipStream_t stream) {
  return launch_mode<kPlain>(p, x, w, out, M, N, K, nullptr, RowNorm{}, stream);
}
gs_status launch_wide_gate_up(const WidePlan& p, const bf16_t* x, const bf16_t* w, bf16_t* act, int M, int N, int K,
                              hipStream_t stream) {
  return launch_mode<kGateUp>(p, x, w, reinterpret_cast<float*>(act), M, N, K, nullptr, RowNorm{}, stream);
}
gs_status launch_wide_gate_up_norm(const WidePlan& p, const bf16_t* x, const bf16_t* w, const RowNorm& norm, bf16_t* act, int M,
                                   int N, int K, hipStream_t stream) {
  return launch_mode<kGateUpNorm>(p, x, w, reinterpret_cast<float*>(act), M, N, K, nullptr, norm, stream);
}
gs_status launch_wide_stats(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* y, float2* stats, int M, int N,
                            int K, hipStream_t stream) {
  return launch_mode<kStats>(p, x, w, y, M, N, K, stats, RowNorm{}, stream);
}

}  // namespace gs
