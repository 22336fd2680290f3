// bf16 projections (MFMA) of many rows: both operands through LDS, shared by all waves of a workgroup.
//
// What bounds it: the matrix pipe and, on ordinary data, the power it draws (2048 x 28672 x 4096: 1.3 to 1.4 PFLOP/s, 1.6 to 1.7
// on matrices of zeros, 1.8 with the loads of the loop taken out).  gemm_wide.hip loads the weights of a wave straight into its
// registers; from a few row chunks on, what a compute unit then takes from L2 (weights once per wave, 96 KB per step of 64 and
// 256 x 256 outputs) is what bounds it.  Here
//   * tiles of weights and activations go from global memory straight into LDS (16 bytes per lane, no registers in between): 64 KB
//     per step and 256 x 256 outputs, and every byte of them once
//   * a wave holds the fragments of one side (`stationary`, NI tiles, read for the next step while this one ends) and reads those of
//     the other one (`streamed`, NO tiles) AHEAD tiles before their MFMAs: LDS delivers 24 KB per wave and step for 64 MFMAs
//   * one barrier per step, AHEAD tiles before its end, when all fragments of the step have been read: it frees the activation
//     buffer of this step (refilled at once for the step after the next) and publishes the next step.  Weights have three buffers
//     and are loaded from the start of a step, for the step after the next: their way from memory is the longer one, and the
//     loads of a step are spread over it (all of them behind the barrier: 400 us against 318 for 2048 x 28672 x 4096 of zeros)
//   * activation rows are 128 bytes in LDS, their 16-byte pieces XOR-swizzled (row_swizzle); since a direct load places the
//     lanes' pieces one after the other, the swizzle is in the lanes' addresses
// Workgroups are dealt to the XCDs in contiguous ranges of (split, column block, row chunk), row chunks next to each other: those of
// an XCD share weights and activations in its L2, and no XCD gets more than one workgroup more than another.
// Shapes (kBlockShapes in gemm_wide.hip): WM x WN waves of MT x NT tiles of 16 x 16; KG = 2: two K groups, each takes one half of
// every 64-wide step, so that tiles of 176 x 64 leave room for two waves per SIMD.
// kQkvHeads: the QKV projection stores Q and the K and V pages itself.  The fp32 sums (25 MB at 1024 rows of 6144 columns) were written and read
// again by a launch of 15 us a layer, 27 at 2047 rows; whole passes 4212 -> 4135 (8 prompts of 128 tokens) and 4994 -> 4934 us (2047 tokens).
// Isolated launches, us, gemm_wide.hip before and this one (one machine):
//   1024 rows  gate/up 28672 x 4096 217 -> 190, 4096 x 14336 104 -> 91, 6144 x 4096 50 -> 45, LM head 128256 x 4096 932 -> 831
//   2047 rows  385 -> 358, 189 -> 172, 97 -> 79, 1810 -> 1614
//   324 rows   gate/up 81 -> 73, LM head 346 -> 330; 256 rows of 57344 x 8192 257 -> 203
#include "common.h"
#include "device_types.h"
#include "gemm_common.h"

namespace gs {
namespace {

// Direct load of 16 bytes per lane from global memory into LDS.  (The host pass of the compiler does not know the builtin.)
#ifdef __HIP_DEVICE_COMPILE__
#define GS_LOAD_LDS(rsrc, lds_ptr, voffset, soffset) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(lds_ptr), 16, voffset, soffset, 0, 0)
#else
#define GS_LOAD_LDS(rsrc, lds_ptr, voffset, soffset) ((void)(rsrc), (void)(lds_ptr), (void)(voffset), (void)(soffset))
#endif

// s_waitcnt for all but the newest n vector memory operations (n <= 63) and, lgkm: for all LDS reads.
#define GS_WAIT(n, lgkm) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | ((lgkm) ? 0 : 15 << 8))

constexpr int kBlockAhead = 2;      // streamed tiles read ahead (3: within 2 %)

// MODE as in gemm_wide.hip; qkv: kQkvHeads.  1-D grid: splits x column blocks x row chunks.
template <int WM, int WN, int KG, int MT, int NT, bool STATIONARY_B, int MODE>
__global__ __launch_bounds__(64 * WM * WN * KG) __attribute__((amdgpu_waves_per_eu(WM * WN * KG == 4 && NT > 4 ? 1 : 2))) void gemm_bf16_block_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Wp, float* __restrict__ P, int M, int N, int K, int k_per_split,
    int m_chunks, int n_blocks, float2* __restrict__ stats, QkvOut qkv) {
  constexpr bool GATE_UP = MODE == kGateUp;
  constexpr int WAVES = WM * WN * KG, ROWS = WM * MT * 16, COL_TILES = WN * NT;
  constexpr int NO = STATIONARY_B ? MT : NT, NI = STATIONARY_B ? NT : MT, NH = 2 / KG;
  constexpr int A_BYTES = ROWS * 128, B_BYTES = COL_TILES * 2048, B0 = 2 * A_BYTES, LDS_BYTES = B0 + 3 * B_BYTES;
  constexpr int LA = (A_BYTES / 1024 + WAVES - 1) / WAVES, LB = (B_BYTES / 1024 + WAVES - 1) / WAVES;      // loads of a wave and step
  constexpr int AHEAD = kBlockAhead;
  static_assert(NO > AHEAD && LDS_BYTES <= 160 * 1024, "");
  static_assert(KG == 1 || (KG == 2 && WM == 1), "");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_BYTES];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = KG == 1 ? 0 : wave / (WM * WN), wv = wave - kg * (WM * WN);
  const int wm = wv / WN, wn = wv % WN;
  const int g = lane >> 4, c = lane & 15;
  const int item = xcd_item();
  const int m_chunk = item % m_chunks, column = item / m_chunks;
  const int split = column / n_blocks, n_block = column - split * n_blocks;
  const int m0 = m_chunk * ROWS;
  const int k_begin = split * k_per_split, n_steps = (min(K, k_begin + k_per_split) - k_begin) / 64;

  const char* xbase = reinterpret_cast<const char*>(X + (size_t)m0 * K + k_begin);
  const unsigned x_bytes = ((unsigned)min(ROWS, M - m0) * (unsigned)K - (unsigned)k_begin) * 2u;
  const size_t w_stride = (size_t)(N / 16) * 2048;
  const char* wbase = reinterpret_cast<const char*>(Wp) + (size_t)(k_begin / 64) * w_stride;
  // pieces of 1 KB (eight activation rows; half a column tile) that this wave moves, the last one more than once where they do
  // not divide among the waves; rows past the end re-read the last one
  constexpr bool HEADS = MODE == kQkvHeads;
  static_assert(!HEADS || NT % 2 == 0, "both halves of the rotation pairs");
  const int half_tiles = HEADS ? qkv.hd >> 5 : 1, pair0 = n_block * (COL_TILES / 2);      // column tiles of half a head; first pair of tiles
  int a_piece[LA], b_piece[LB];
  unsigned a_off[LA], b_off[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    a_piece[i] = min(wave + i * WAVES, A_BYTES / 1024 - 1);
    const int r = a_piece[i] * 8 + (lane >> 3);
    a_off[i] = (unsigned)min(r, M - 1 - m0) * (unsigned)K * 2u + (((lane & 7) ^ row_swizzle(r)) << 4);
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    b_piece[i] = min(wave + i * WAVES, B_BYTES / 1024 - 1);
    // gate/up: the first half of the workgroup's column tiles are gate features, the second the same ones of the up half
    const int t = b_piece[i] >> 1;
    int tile = GATE_UP ? n_block * (COL_TILES / 2) + (t < COL_TILES / 2 ? t : t - COL_TILES / 2 + N / 32) : n_block * COL_TILES + t;
    if constexpr (HEADS) {
      // the first half of a wave's tiles are first halves of rotation pairs, the others the second halves of the same ones
      const int u = t % NT, pair = pair0 + t / NT * (NT / 2) + u % (NT / 2);
      tile = pair / half_tiles * 2 * half_tiles + pair % half_tiles + (u < NT / 2 ? 0 : half_tiles);
    }
    b_off[i] = (unsigned)tile * 2048u + (b_piece[i] & 1) * 1024u;
  }
  const unsigned lane16 = lane * 16;
  // (a step past the end has an empty descriptor: it moves nothing, and the number of loads in flight stays what it is)
  auto load_a = [&](int step, int buf, int i) {
    const int s = min(step, n_steps - 1);
    auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(xbase + (size_t)s * 128), 0,
                                               step < n_steps ? x_bytes - (unsigned)s * 128u : 0u, 0x00020000);
    GS_LOAD_LDS(r, lds + buf * A_BYTES + a_piece[i] * 1024, a_off[i], 0);
  };
  auto load_b = [&](int step, int slot, int i) {
    const int s = min(step, n_steps - 1);
    auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wbase + (size_t)s * w_stride), 0,
                                               step < n_steps ? (unsigned)w_stride : 0u, 0x00020000);
    GS_LOAD_LDS(r, lds + slot + b_piece[i] * 1024, lane16, b_off[i]);
  };

  // fragments: lane (g, c) holds row (column) c, k = 16 g + 8 h .. of the step for half h
  constexpr bool PAIRED = GATE_UP && NT % 2 == 0;      // a wave has NT / 2 gate tiles and the same up tiles; else gate or up tiles
  const int a0 = (wm * MT * 16 + c) * 128 + (((2 * g + kg) ^ row_swizzle(c)) << 4);
  const int a1 = (wm * MT * 16 + c) * 128 + (((2 * g + 1) ^ row_swizzle(c)) << 4);
  const int b0 = (PAIRED ? wn * (NT / 2) : wn * NT) * 2048 + kg * 1024 + lane16;
  auto frag = [&](bool b, int buf, int slot, int tile, int h) {
    if (!b) return *reinterpret_cast<const bf16x8_t*>(&lds[buf * A_BYTES + (h ? a1 : a0) + tile * 2048]);
    const int up = PAIRED && tile >= NT / 2 ? (COL_TILES / 2 - NT / 2) * 2048 : 0;
    return *reinterpret_cast<const bf16x8_t*>(&lds[slot + b0 + up + tile * 2048 + h * 1024]);
  };
  floatx4_t acc[NO][NI];
#pragma unroll
  for (int o = 0; o < NO; ++o)
#pragma unroll
    for (int i = 0; i < NI; ++i) acc[o][i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  bf16x8_t str[AHEAD][NH], stat[2][NI][NH];
#pragma unroll
  for (int i = 0; i < LB; ++i) load_b(0, B0, i);
#pragma unroll
  for (int i = 0; i < LA; ++i) load_a(0, 0, i);
#pragma unroll
  for (int i = 0; i < LB; ++i) load_b(1, B0 + B_BYTES, i);
#pragma unroll
  for (int i = 0; i < LA; ++i) load_a(1, 1, i);
  GS_WAIT(LA + LB, false);
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < NI * NH; ++i) stat[0][i / NH][i % NH] = frag(STATIONARY_B, 0, B0, i / NH, i % NH);
#pragma unroll
  for (int i = 0; i < AHEAD * NH; ++i) str[i / NH][i % NH] = frag(!STATIONARY_B, 0, B0, i / NH, i % NH);
  constexpr int LB_TILE = (LB + NO - AHEAD - 1) / (NO - AHEAD);      // weight loads per streamed tile before the barrier
  int slot = B0;      // of this step's weights
  for (int base = 0;; base += 2) {
    bool done = false;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const int step = base + d;
      if (!done) {
        // next: the weights of the next step; free: of the step before, read by all waves before its barrier
        const int next = slot == B0 + 2 * B_BYTES ? B0 : slot + B_BYTES, free = next == B0 + 2 * B_BYTES ? B0 : next + B_BYTES;
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          if (o == NO - AHEAD) {
            GS_WAIT(LB, true);      // this wave's loads of the next step, its reads of this one
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
          }
          bf16x8_t cur[NH];
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            cur[h] = str[0][h];
#pragma unroll
            for (int i = 0; i + 1 < AHEAD; ++i) str[i][h] = str[i + 1][h];
            str[AHEAD - 1][h] = o + AHEAD < NO ? frag(!STATIONARY_B, d, slot, o + AHEAD, h) : frag(!STATIONARY_B, d ^ 1, next, o + AHEAD - NO, h);
          }
          if (o < NO - AHEAD) {
#pragma unroll
            for (int i = o * LB_TILE; i < (o + 1) * LB_TILE; ++i)
              if (i < LB) load_b(step + 2, free, i);
          } else {
            const int q = o - (NO - AHEAD);
#pragma unroll
            for (int i = q * NI * NH / AHEAD; i < (q + 1) * NI * NH / AHEAD; ++i)
              stat[d ^ 1][i / NH][i % NH] = frag(STATIONARY_B, d ^ 1, next, i / NH, i % NH);
#pragma unroll
            for (int i = q * LA / AHEAD; i < (q + 1) * LA / AHEAD; ++i) load_a(step + 2, d, i);
          }
#pragma unroll
          for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int i = 0; i < NI; ++i)
              acc[o][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(STATIONARY_B ? cur[h] : stat[d][i][h],
                                                                  STATIONARY_B ? stat[d][i][h] : cur[h], acc[o][i], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        slot = next;
        done = step + 1 >= n_steps;
      }
    }
    if (done) break;
  }
  GS_WAIT(0, true);      // no load may still be on its way into LDS when its contents change or the workgroup ends
  auto sum = [&](int mt, int nt) -> floatx4_t& { return STATIONARY_B ? acc[mt][nt] : acc[nt][mt]; };
  auto owned = [&](int mt) { return KG == 1 || (mt & 1) == kg; };
  if constexpr (KG == 2) {
    // the K groups share the epilogue: group mt % 2 takes row tile mt; one direction after the other through the same LDS
    static_assert((MT + 1) / 2 * NT * 1024 * WN <= LDS_BYTES, "the sums that change hands fit the buffers");
    floatx4_t* sums = reinterpret_cast<floatx4_t*>(lds) + wv * 64 + lane;
#pragma unroll
    for (int owner = 0; owner < 2; ++owner) {
      __syncthreads();
      if (kg != owner) {
#pragma unroll
        for (int mt = owner; mt < MT; mt += 2)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) sums[((mt >> 1) * NT + nt) * WN * 64] = sum(mt, nt);
      }
      __syncthreads();
      if (kg == owner) {
#pragma unroll
        for (int mt = owner; mt < MT; mt += 2)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) sum(mt, nt) += sums[((mt >> 1) * NT + nt) * WN * 64];
      }
    }
  }
  const int row0 = m0 + wm * MT * 16 + g * 4;
  if constexpr (GATE_UP) {
    bf16_t* act = reinterpret_cast<bf16_t*>(P);
    const int F = N / 2;
    auto store = [&](int row, int feature_tile, float gt, float up) {
      act[(size_t)row * F + feature_tile * 16 + c] = float_to_bf16(gt / (1.0f + expf(-gt)) * up);
    };
    if constexpr (PAIRED) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (owned(mt) && row0 + mt * 16 + i < M) {
#pragma unroll
            for (int ft = 0; ft < NT / 2; ++ft)
              store(row0 + mt * 16 + i, (n_block * WN + wn) * (NT / 2) + ft, sum(mt, ft)[i], sum(mt, NT / 2 + ft)[i]);
          }
    } else {
      // the first wave column has gate, the second up features: half of the row tiles change hands
      static_assert(!GATE_UP || PAIRED || (WN == 2 && KG == 1 && MT % 2 == 0 && WM * MT * NT * 1024 <= LDS_BYTES), "");
      floatx4_t* other = reinterpret_cast<floatx4_t*>(lds) + wm * MT * NT * 64 + lane;
      __syncthreads();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        if ((mt < MT / 2) != (wn == 0)) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) other[(mt * NT + nt) * 64] = sum(mt, nt);
        }
      __syncthreads();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        if ((mt < MT / 2) == (wn == 0)) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const floatx4_t own = sum(mt, nt), its = other[(mt * NT + nt) * 64];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (row0 + mt * 16 + i < M) store(row0 + mt * 16 + i, n_block * NT + nt, wn == 0 ? own[i] : its[i], wn == 0 ? its[i] : own[i]);
          }
        }
    }
    return;
  }
  if constexpr (HEADS) {
    // pair of column tiles after pair, row tile after row tile: the factors and places of the next one are loaded while this one is stored
    // (loaded where they are used, and stores of 2 bytes: a 2047-token prompt 33 us a layer slower)
    const int half = qkv.hd >> 1;
    const bool odd = c & 1;
    auto pair_of = [&](int p) { return pair0 + wn * (NT / 2) + p; };
    float2 cs[2][4];
    int2 at[2][4];
    auto fetch = [&](int b, int p, int mt) {
      const int i = pair_of(p) % half_tiles * 16 + c;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = min(row0 + mt * 16 + r, M - 1);
        cs[b][r] = qkv.rope[(size_t)row * half + i];
        at[b][r] = *reinterpret_cast<const int2*>(qkv.row_slot + row);
      }
    };
    static_assert(!HEADS || MT / KG % 2 == 0, "the two sets of a pair's row tiles end on the second one");
    fetch(0, 0, kg);
#pragma unroll
    for (int p = 0; p < NT / 2; ++p) {
      const int pair = pair_of(p), head = pair / half_tiles, i0 = pair % half_tiles * 16 + c;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (!owned(mt)) continue;
        const int b = mt / KG & 1;
        if (mt + KG < MT) fetch(b ^ 1, p, mt + KG);
        else if (p + 1 < NT / 2) fetch(0, p + 1, kg);
        const floatx4_t u = sum(mt, p), v = sum(mt, NT / 2 + p);
        const int row = row0 + mt * 16;
        if (head < qkv.n_heads + qkv.n_kv) {
          // neighbouring columns share their stores: the even lane takes the first row of two, the odd one the second, 4 bytes each
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            float lo[2], hi[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const float2 f = cs[b][2 * j + k];
              lo[k] = fmaf(u[2 * j + k], f.x, -(v[2 * j + k] * f.y));      // (as in store_qkv_pair)
              hi[k] = fmaf(v[2 * j + k], f.x, u[2 * j + k] * f.y);
            }
            const float lo_n = dpp_move<0xB1>(odd ? lo[0] : lo[1]), hi_n = dpp_move<0xB1>(odd ? hi[0] : hi[1]);
            const int2 ps = odd ? at[b][2 * j + 1] : at[b][2 * j];
            const int r = row + 2 * j + (int)odd;
            bf16_t* dst = head < qkv.n_heads
                              ? static_cast<bf16_t*>(qkv.q) + ((size_t)r * qkv.n_heads + head) * qkv.hd
                              : static_cast<bf16_t*>(qkv.k_pages) + (((size_t)ps.x * qkv.n_kv + (head - qkv.n_heads)) * qkv.page_size + ps.y) * qkv.hd;
            dst += i0 - (int)odd;
            if (r < M) {
              *reinterpret_cast<uint32_t*>(dst) = odd ? pack_bf16x2(lo_n, lo[1]) : pack_bf16x2(lo[0], lo_n);
              *reinterpret_cast<uint32_t*>(dst + half) = odd ? pack_bf16x2(hi_n, hi[1]) : pack_bf16x2(hi[0], hi_n);
            }
          }
        } else {
          // four rows of a lane are four slots of a channel, next to each other in most cases: one store of 8 bytes
          bool run = row + 3 < M && at[b][0].y % 4 == 0 && qkv.page_size % 4 == 0;
#pragma unroll
          for (int r = 1; r < 4; ++r) run = run && at[b][r].x == at[b][0].x && at[b][r].y == at[b][0].y + r;
          auto place = [&](int r, int channel) {
            return static_cast<bf16_t*>(qkv.v_pages) +
                   (((size_t)at[b][r].x * qkv.n_kv + (head - qkv.n_heads - qkv.n_kv)) * qkv.hd + channel) * qkv.page_size + at[b][r].y;
          };
          if (run) {
            *reinterpret_cast<uint2*>(place(0, i0)) = make_uint2(pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3]));
            *reinterpret_cast<uint2*>(place(0, i0 + half)) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (row + r < M) {
                *place(r, i0) = float_to_bf16(u[r]);
                *place(r, i0 + half) = float_to_bf16(v[r]);
              }
          }
        }
      }
    }
    return;
  }
  float* out = P + (size_t)split * M * N + (size_t)(n_block * COL_TILES + wn * NT) * 16 + c;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row0 + mt * 16 + i;
      if (owned(mt) && row < M) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) out[(size_t)row * N + nt * 16] = sum(mt, nt)[i];
      }
    }
  if constexpr (MODE == kStats) {
    static_assert(LDS_BYTES >= WN * ROWS * (int)sizeof(float2), "the statistics fit the buffers");
    float2* st = reinterpret_cast<float2*>(lds);      // [WN][ROWS]
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (owned(mt)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float mx = sum(mt, 0)[i];
#pragma unroll
          for (int nt = 1; nt < NT; ++nt) mx = fmaxf(mx, sum(mt, nt)[i]);
          mx = row16_max(mx);
          float e = 0.f;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) e += __expf(sum(mt, nt)[i] - mx);
          e = row16_sum(e);
          if (c == 0) st[wn * ROWS + (wm * MT + mt) * 16 + g * 4 + i] = make_float2(mx, e);
        }
      }
    __syncthreads();
    for (int r = threadIdx.x; r < ROWS; r += 64 * WAVES)
      if (m0 + r < M) {
        float m = st[r].x, s = st[r].y;
#pragma unroll
        for (int w = 1; w < WN; ++w) merge_stat(m, s, st[w * ROWS + r].x, st[w * ROWS + r].y);
        stats[(size_t)(m0 + r) * n_blocks + n_block] = make_float2(m, s);
      }
  }
}

}  // namespace

template <int MODE>
static gs_status launch_mode(const WidePlan& p, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K, float2* stats,
                             hipStream_t stream, const QkvOut& qkv = QkvOut{}) {
  const int grid = p.n_blocks * p.m_chunks * p.splits;
#define GS_BLOCK(WM, WN, KG, MT, NT, STATIONARY_B)                                                                     \
  gemm_bf16_block_kernel<WM, WN, KG, MT, NT, STATIONARY_B, MODE><<<grid, 64 * WM * WN * KG, 0, stream>>>(               \
      x, w, out, M, N, K, p.k_per, p.m_chunks, p.n_blocks, stats, qkv)
  if (p.wm == 4 && p.nt == 8) GS_BLOCK(4, 2, 1, 4, 8, false);
  else if (p.wm == 2 && p.nt == 4) GS_BLOCK(2, 2, 1, 4, 4, true);
  else if (p.wm == 1 && p.mt == 8) GS_BLOCK(1, 4, 2, 8, 4, true);
  else if constexpr (MODE == kQkvHeads) {
    if (p.wm != 2) return fail(GS_EUNSUPPORTED, "no heads of %d x %d tiles", p.mt, p.nt);
    GS_BLOCK(2, 2, 1, 4, 6, false);
  }
  else if (p.wm == 1 && p.mt == 10) GS_BLOCK(1, 4, 2, 10, 4, true);
  else if (p.wm == 1 && p.mt == 11) GS_BLOCK(1, 4, 2, 11, 4, true);
  else if (MODE == kStats) return fail(GS_EUNSUPPORTED, "column blocks of %d do not leave statistics", 16 * p.wn * p.nt);
  else if constexpr (MODE != kStats) {
    if (p.wm == 4) GS_BLOCK(4, 2, 1, 4, 7, false);
    else GS_BLOCK(2, 2, 1, 4, 6, false);
  }
#undef GS_BLOCK
  GS_LAUNCH_CHECK("gemm_bf16_block");
  return GS_OK;
}

gs_status launch_block(int mode, const WidePlan& p, const bf16_t* x, const bf16_t* w, float* out, int M, int N, int K, float2* stats,
                       hipStream_t stream) {
  switch (mode) {
    case kPlain: return launch_mode<kPlain>(p, x, w, out, M, N, K, stats, stream);
    case kGateUp: return launch_mode<kGateUp>(p, x, w, out, M, N, K, stats, stream);
    default: return launch_mode<kStats>(p, x, w, out, M, N, K, stats, stream);
  }
}

gs_status launch_block_qkv(const WidePlan& p, const bf16_t* x, const bf16_t* w, const QkvOut& out, int M, int N, int K, hipStream_t stream) {
  return launch_mode<kQkvHeads>(p, x, w, nullptr, M, N, K, nullptr, stream, out);
}

}  // namespace gs
