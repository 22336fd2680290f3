// Projections with 4-bit weights (weight-only quantisation in groups of 128 inputs, the format family of
// the AWQ checkpoints the paper's 70B verifier uses, Section IV-A): Y = X * W^T with
// W[n][k] = (code[n][k] - zero[n][k/128]) * scale[n][k/128], codes and zeros in 0..15, scales bf16.
//
// Same streaming design as the bf16 kernels, with a quarter of the weight bytes, which moves the bound from
// HBM to the dequantisation arithmetic and the MFMA pipe: a wave owns NT tiles of 32 output columns and up to 128 rows and
// reads, per 64-wide k step and tile, 16 bytes per lane (32 codes of one column) plus, every two steps, one 32-bit word with
// the column's scale and zero point; the codes are turned into bf16 in registers and fed to the 32x32x16 MFMA as the B
// operand.  Every dequantised weight is (c - zero) * scale, exact in fp32 (4 x 8 significant bits), rounded to bf16 (nearest
// even): a function of (c, zero, scale) alone, the same on every path.
//
// Packed layout (gs_pack_weight_w4):
//   codes [K/64][N/32][64 lanes][4 words]: lane l holds column l%32, and word kg holds inputs
//         16 kg + 8 (l/32) + i, i = 0..7 (the B fragment of k group kg); in a word, codes 0..3 sit in the low
//         nibbles of bytes 0..3 and codes 4..7 in the high nibbles, so that (word & 0x0F0F0F0F) and
//         ((word >> 4) & 0x0F0F0F0F) each hold four codes, one per byte
//   meta  [K/128][N] words: bf16 scale in the high half, zero point in the low byte
// Rows beyond 128 are served in chunks of 128 by separate workgroups (XCD-aware order, see the bf16 kernel).
#include "common.h"
#include "device_types.h"
#include "gemm_common.h"
#include <algorithm>
#include <type_traits>

namespace gs {
namespace {

constexpr int kBK = 64;
constexpr int kGroup = 128;

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

// word: codes 0..3 in the even nibbles of bytes 0..3, codes 4..7 in the odd nibbles.  A nibble OR-ed into the mantissa of
// 1024 is the half-precision number 1024 + c (even nibble) or 1024 + 16 c (odd nibble), two to a word, and the
// mixed-precision fma reads either half: (1024 + c) * scale - (1024 + z) * scale = (c - z) * scale, exact in fp32
// (11 x 8 significant bits, one rounding at the end, which has nothing to round).  17 instructions per 8 codes
// (23 with byte conversions).  The constant term of a scale of kLargeScale and more may overflow: such groups are rare enough
// that a wave which meets one goes on in a second loop that repairs their weights (dequant8_large), b holding the zero point
// instead.  (8 layers of the 8B shape at 53 rows: this and its check of every scale group cost 0.1 to 0.4 % of the step, a branch
// between any two blocks of the one loop 1.5 %; a choice between two bodies per step spills.)
// (The 1024 trick is that of Kim et al., "Who Says Elephants Can't Run: Bringing Large Scale MoE Models into Cloud Scale
// Production", 2022.)
typedef _Float16 half2_vec __attribute__((ext_vector_type(2)));
constexpr float kLargeScale = 0x1p117f;
struct DequantScale {
  float s, b, s16, b16;
};
__device__ __forceinline__ bool large(const DequantScale& d) { return !(fabsf(d.s) < kLargeScale); }
__device__ __forceinline__ DequantScale dequant_scale(uint32_t meta) {
  DequantScale d;
  const float z = (float)(meta & 0xffu);
  d.s = __uint_as_float(meta & 0xffff0000u);
  d.b = large(d) ? z : -(1024.0f + z) * d.s;
  d.s16 = d.s * 0.0625f;
  d.b16 = -(64.0f + z) * d.s;
  return d;
}
__device__ __forceinline__ bf16x8_t dequant8(uint32_t word, const DequantScale& d) {
  uint32_t magic = 0x64006400u;
  asm("" : "+v"(magic));      // (in a register: and-or takes one constant)
  auto halves = [&](uint32_t w, uint32_t mask) {
    const uint32_t h = (w & mask) | magic;
    return *reinterpret_cast<const half2_vec*>(&h);
  };
  const half2_vec e = halves(word, 0x000F000Fu), o = halves(word, 0x00F000F0u);                  // codes 0, 2 and 4, 6
  const half2_vec e8 = halves(word >> 8, 0x000F000Fu), o8 = halves(word >> 8, 0x00F000F0u);      // codes 1, 3 and 5, 7
  uint4 out;
  out.x = pack_bf16x2(fmaf((float)e[0], d.s, d.b), fmaf((float)e8[0], d.s, d.b));
  out.y = pack_bf16x2(fmaf((float)e[1], d.s, d.b), fmaf((float)e8[1], d.s, d.b));
  out.z = pack_bf16x2(fmaf((float)o[0], d.s16, d.b16), fmaf((float)o8[0], d.s16, d.b16));
  out.w = pack_bf16x2(fmaf((float)o[1], d.s16, d.b16), fmaf((float)o8[1], d.s16, d.b16));
  return *reinterpret_cast<const bf16x8_t*>(&out);
}

// The weights of a large scale, by the definition.
__device__ __forceinline__ bf16x8_t dequant8_large(uint32_t word, const DequantScale& d) {
  float v[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = ((float)((word >> (8 * i)) & 15u) - d.b) * d.s;
    v[4 + i] = ((float)((word >> (8 * i + 4)) & 15u) - d.b) * d.s;
  }
  const uint4 out = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
  return *reinterpret_cast<const bf16x8_t*>(&out);
}

typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

// WN waves side by side, each with NT 32-column tiles and all MT 32-row tiles; KG groups of them take K slices of the
// workgroup's range, and their sums meet in LDS.  DB, DA: steps (64 of k) of weights and of activations in
// registers.
// MODE kGateUp (one K split): the wave's tiles are NT / 2 feature tiles of the gate half and the same ones of the up half of a
// [2F][K] matrix (N = 2F), and act[M][F] = silu(gate) * up is stored as bf16 at P.
// Pipeline, as in gemm_wide.hip: a step is four blocks, one per k group of 16, each of which reads the activation
// fragments of two blocks ahead from LDS (three buffers), dequantises the weights of the next block, moves its share of
// the next activation tile and weights, and issues its MT * NT MFMAs.
// 1-D grid: K splits x column blocks x row chunks, an even contiguous range of them for every XCD (as in gemm_wide.hip).
template <int WN, int KG, int MT, int NT, int DB, int DA, int WPE, int MODE>
__global__ __launch_bounds__(64 * WN * KG) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void gemm_w4_kernel(
    const bf16_t* __restrict__ X, const uint4* __restrict__ codes, const uint32_t* __restrict__ meta,
    float* __restrict__ P, int M, int N, int K, int k_per_split, int m_chunks) {
  static_assert(MODE != kGateUp || NT % 2 == 0, "gate and up tile of every feature tile");
  static_assert(DB % 2 == 0 && DB % DA == 0, "a scale group is two steps; rings are addressed statically");
  constexpr int ROWS = MT * 32, THREADS = 64 * WN;      // THREADS: of one K group
  constexpr int PASSES = (ROWS * 8 + THREADS - 1) / THREADS;
  constexpr int TILE = ROWS * 128;
  // three activation buffers per K group; after the loop the sums that the K groups exchange
  constexpr int RING = KG * 3 * TILE, SUMS = MT * 4 * (KG - 1) * NT * THREADS * 16;
  __shared__ __attribute__((aligned(16))) unsigned char xs_all[RING > SUMS ? RING : SUMS];
  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave_all / WN, wn = wave_all % WN;
  const int tid = threadIdx.x - kg * THREADS;
  unsigned char* xs = xs_all + kg * 3 * TILE;
  const int h = lane >> 5, c32 = lane & 31;
  const int item = xcd_item();
  const int m_chunk = item % m_chunks, column = item / m_chunks, n_blocks = N / (32 * NT * WN);
  const int split = column / n_blocks, n_block = column - split * n_blocks;
  const int n_tile0 = (n_block * WN + wn) * (MODE == kGateUp ? NT / 2 : NT);
  const int m0 = m_chunk * ROWS;
  const int split_begin = split * k_per_split, split_end = min(K, split_begin + k_per_split);
  // the K groups take whole scale groups (two steps) and run the same number of steps (barriers); a step past a group's
  // own end multiplies zeros by weights of scale zero
  const int split_steps = (split_end - split_begin) / 64;
  const int n_steps = (split_steps / 2 + KG - 1) / KG * 2;
  const int own_steps = min(n_steps, split_steps - kg * n_steps);
  const int k_begin = split_begin + (own_steps > 0 ? kg * n_steps * 64 : 0);
  const int last = max(own_steps - 1, 0);
  const char* xbase = reinterpret_cast<const char*>(X + (size_t)m0 * K + k_begin);
  const unsigned x_bytes = ((unsigned)min(ROWS, M - m0) * (unsigned)K - (unsigned)k_begin) * 2u;
  const size_t c_stride = (size_t)(N / 32) * 1024;      // code bytes of one step
  const char* cbase = reinterpret_cast<const char*>(codes) + (size_t)(k_begin / 64) * c_stride + (size_t)n_tile0 * 1024;
  const unsigned c_bytes = (unsigned)c_stride - (unsigned)n_tile0 * 1024u;
  const char* mbase = reinterpret_cast<const char*>(meta + (size_t)(k_begin / kGroup) * N + n_tile0 * 32);
  const unsigned m_bytes = (unsigned)(N - n_tile0 * 32) * 4u;
  unsigned xoff[PASSES], loff[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    // (a last pass with fewer pieces than lanes moves the last piece several times)
    const int ch = min(tid + p * THREADS, ROWS * 8 - 1), row = ch >> 3, piece = ch & 7;
    xoff[p] = (unsigned)row * (unsigned)K * 2u + piece * 16u;
    loff[p] = row * 128 + ((piece ^ ((row >> 1) & 7)) << 4);
  }
  auto x_rsrc = [&](int step) {      // rows past the end and steps past the K group's end read as zero
    const int s = min(step, last);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(xbase + (size_t)s * 128), 0,
                                             (KG == 1 || step < own_steps) ? x_bytes - (unsigned)s * 128u : 0u, 0x00020000);
  };
  auto c_rsrc = [&](int step) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(cbase + (size_t)min(step, last) * c_stride), 0,
                                             (KG == 1 || step < own_steps) ? c_bytes : 0u, 0x00020000);
  };
  auto m_rsrc = [&](int step) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(mbase + (size_t)(min(step, last) >> 1) * N * 4), 0,
                                             (KG == 1 || step < own_steps) ? m_bytes : 0u, 0x00020000);
  };
  uintx4_t xreg[DA][PASSES];
  uintx4_t creg[DB][NT];
  unsigned mreg[DB / 2][NT];
  constexpr int UP = MODE == kGateUp ? NT / 2 : NT;      // first tile of the up half
  const unsigned up_tiles = MODE == kGateUp ? (unsigned)(N / 64 - NT / 2) : 0u;
  const unsigned coff = lane * 16, moff = c32 * 4;
#define GS_LOAD_X(slot, p, r) xreg[slot][p] = __builtin_amdgcn_raw_buffer_load_b128(r, xoff[p], 0, 0)
#define GS_LOAD_C(slot, nt, r) \
  creg[slot][nt] = __builtin_amdgcn_raw_buffer_load_b128(r, coff + (nt) * 1024, (nt) >= UP ? up_tiles * 1024u : 0u, 0)
#define GS_LOAD_M(slot, nt, r) \
  mreg[slot][nt] = __builtin_amdgcn_raw_buffer_load_b32(r, moff + (nt) * 128, (nt) >= UP ? up_tiles * 128u : 0u, 0)
  floatx16_t acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mt][nt][e] = 0.f;
  // fragment of row tile mt, k group q: lane holds row lane % 32, piece 2 q + lane / 32
  int a_off[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) a_off[q] = c32 * 128 + (((2 * q + h) ^ ((c32 >> 1) & 7)) << 4);
  {
    uintx4_t r0[PASSES], r1[PASSES];
    auto rx0 = x_rsrc(0), rx1 = x_rsrc(1);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) r0[p] = __builtin_amdgcn_raw_buffer_load_b128(rx0, xoff[p], 0, 0);
#pragma unroll
    for (int d = 0; d < DB - 1; ++d) {
      auto rc = c_rsrc(d), rm = m_rsrc(d);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        GS_LOAD_C(d, nt, rc);
        if (d % 2 == 0) GS_LOAD_M(d / 2, nt, rm);
      }
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
#pragma unroll
    for (int p = 0; p < PASSES; ++p) *reinterpret_cast<uintx4_t*>(&xs[TILE + loff[p]]) = r1[p];
  }
  __syncthreads();
  bf16x8_t an[4][MT];      // fragments of this block and the next two
  auto frag = [&](int buf, int q, bf16x8_t (&a)[MT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) a[mt] = *reinterpret_cast<const bf16x8_t*>(&xs[buf + a_off[q] + mt * 4096]);
  };
  frag(0, 0, an[0]);
  frag(0, 1, an[1]);
  DequantScale ds[NT];
  bf16x8_t bn[2][NT];      // dequantised weights of this block and the next
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    ds[nt] = dequant_scale(mreg[0][nt]);
    bn[0][nt] = dequant8(creg[0][nt][0], ds[nt]);
  }
  int b0 = 0;
  auto repair = [&](int nt, uint32_t word, bf16x8_t& w) {
    if (large(ds[nt])) w = dequant8_large(word, ds[nt]);
  };
  // One step.  REPAIR: after every block the weights it has dequantised are repaired where their scale is large.
  auto run_step = [&](auto REPAIR, int d, int step, int b1, int b2) __attribute__((always_inline)) {
    auto rx = x_rsrc(step + 2 + DA);
    auto rc = c_rsrc(step + DB - 1), rm = m_rsrc(step + DB - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < 2) frag(b0, q + 2, an[q + 2]); else frag(b1, q - 2, an[q - 2]);
      if (q == 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) GS_LOAD_C((d + DB - 1) % DB, nt, rc);
      }
      if ((d + DB - 1) % 2 == 0 && q == 1) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) GS_LOAD_M((d + DB - 1) % DB / 2, nt, rm);
      }
#pragma unroll
      for (int p = q * PASSES / 4; p < (q + 1) * PASSES / 4; ++p) {
        *reinterpret_cast<uintx4_t*>(&xs[b2 + loff[p]]) = xreg[d % DA][p];
        GS_LOAD_X(d % DA, p, rx);
      }
      // the next block's weights: k group q + 1 of this step, or group 0 of the next (another scale group after
      // an odd step)
      if (q < 3) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bn[(q + 1) % 2][nt] = dequant8(creg[d % DB][nt][q + 1], ds[nt]);
      } else {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if (d % 2 == 1) ds[nt] = dequant_scale(mreg[(d + 1) % DB / 2][nt]);
          bn[(q + 1) % 2][nt] = dequant8(creg[(d + 1) % DB][nt][0], ds[nt]);
        }
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(an[q][mt], bn[q % 2][nt], acc[mt][nt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(REPAIR)::value) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          repair(nt, q < 3 ? creg[d % DB][nt][(q + 1) % 4] : creg[(d + 1) % DB][nt][0], bn[(q + 1) % 2][nt]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // whether some lane's current scale group has a large scale (uniform over the wave)
  auto any_large = [&]() {
    bool any = false;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) any |= large(ds[nt]);
    return __any(any);
  };
  auto next_buffers = [&](int& b1, int& b2) {
    b1 = b0 == 2 * TILE ? 0 : b0 + TILE;
    b2 = b1 == 2 * TILE ? 0 : b1 + TILE;
  };
  int step = 0, first_large = -1;
  while (first_large < 0 && step < n_steps) {
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      if (d % 2 == 0 && __builtin_expect(any_large(), false)) {
        first_large = step;
        break;
      }
      int b1, b2;
      next_buffers(b1, b2);
      run_step(std::false_type(), d, step, b1, b2);
      __syncthreads();
      b0 = b1;
      if (++step >= n_steps) break;
    }
  }
  if (__builtin_expect(first_large >= 0, false)) {      // the rest of the steps, with every block's weights repaired
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) repair(nt, (first_large & 2) ? creg[2 % DB][nt][0] : creg[0][nt][0], bn[0][nt]);
    for (int base = first_large & ~(DB - 1); step < n_steps; base += DB) {
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        if (base + d != step || step >= n_steps) continue;
        int b1, b2;
        next_buffers(b1, b2);
        run_step(std::true_type(), d, step, b1, b2);
        __syncthreads();
        b0 = b1;
        ++step;
      }
    }
  }
#undef GS_LOAD_X
#undef GS_LOAD_C
#undef GS_LOAD_M

  // register v of a tile is row 8 (v / 4) + 4 (lane / 32) + v % 4: chunk q = (row tile, v / 4) is four rows of the lane's column.  The
  // K groups share the epilogue: group q % KG owns chunk q, takes its sums from all groups in a fixed order, and stores it.
  // (One group that takes over all sums, round by round, and stores everything is a quarter of the waves at work for 4 us:
  // gate/up of the 8B shape at 53 rows 28.1 us, 25.9 this way; LM head 86.5 and 80.2, 4096 x 14336 16.9 and 14.8.)
  auto owned = [&](int q) { return KG == 1 || q % KG == kg; };
  if constexpr (KG > 1) {
    static_assert(MT * 4 % KG == 0, "every group owns as many chunks");
    floatx4_t* sums = reinterpret_cast<floatx4_t*>(xs_all);
    // what group src hands to the owner of chunk q
    auto place = [&](int src, int q, int nt) {
      const int o = q % KG;
      return (((src * (MT * 4 / KG) + q / KG) * (KG - 1) + (o < src ? o : o - 1)) * NT + nt) * THREADS + tid;
    };
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MT * 4; ++q)
      if (!owned(q))
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const floatx16_t& t = acc[q / 4][nt];
          sums[place(kg, q, nt)] = floatx4_t{t[q % 4 * 4], t[q % 4 * 4 + 1], t[q % 4 * 4 + 2], t[q % 4 * 4 + 3]};
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MT * 4; ++q)
      if (owned(q))
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          floatx16_t& t = acc[q / 4][nt];
          const floatx4_t own = floatx4_t{t[q % 4 * 4], t[q % 4 * 4 + 1], t[q % 4 * 4 + 2], t[q % 4 * 4 + 3]};
          floatx4_t v = q % KG == 0 ? own : sums[place(0, q, nt)];
#pragma unroll
          for (int src = 1; src < KG; ++src) v += q % KG == src ? own : sums[place(src, q, nt)];
#pragma unroll
          for (int j = 0; j < 4; ++j) t[q % 4 * 4 + j] = v[j];
        }
  }
  float* out = P + (size_t)split * M * N;
#pragma unroll
  for (int q = 0; q < MT * 4; ++q) {
    if (!owned(q)) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = m0 + q / 4 * 32 + q % 4 * 8 + h * 4 + j, v = q % 4 * 4 + j;
      if (row >= M) continue;
      if constexpr (MODE == kGateUp) {
#pragma unroll
        for (int ft = 0; ft < NT / 2; ++ft) {
          const float gt = acc[q / 4][ft][v];
          reinterpret_cast<bf16_t*>(P)[(size_t)row * (N / 2) + (n_tile0 + ft) * 32 + c32] =
              float_to_bf16(gt / (1.0f + expf(-gt)) * acc[q / 4][NT / 2 + ft][v]);
        }
      } else {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) out[(size_t)row * N + (n_tile0 + nt) * 32 + c32] = acc[q / 4][nt][v];
      }
    }
  }
}

// One thread per packed code word (8 codes of one column) or per meta word.
__global__ __launch_bounds__(256) void pack_w4_kernel(const uint8_t* __restrict__ q, const bf16_t* __restrict__ scales,
                                                      const uint8_t* __restrict__ zeros, uint32_t* __restrict__ codes,
                                                      uint32_t* __restrict__ meta, int N, int K) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t n_code_words = (size_t)N * K / 8;
  const size_t n_meta = (size_t)(K / kGroup) * N;
  if (idx < n_code_words) {
    const int kg = (int)(idx & 3), lane = (int)((idx >> 2) & 63);
    const size_t block = idx >> 8;
    const int n_tiles = N / 32;
    const int n_tile = (int)(block % n_tiles), k_step = (int)(block / n_tiles);
    const int h = lane >> 5, c32 = lane & 31;
    const uint8_t* src = q + (size_t)(n_tile * 32 + c32) * K + k_step * kBK + kg * 16 + h * 8;
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w |= (uint32_t)(src[i] & 15u) << (8 * i);            // codes 0..3: even nibbles
      w |= (uint32_t)(src[4 + i] & 15u) << (8 * i + 4);    // codes 4..7: odd nibbles
    }
    codes[idx] = w;
  } else if (idx < n_code_words + n_meta) {
    const size_t j = idx - n_code_words;
    const int grp = (int)(j / N), n = (int)(j % N);
    const size_t s = (size_t)n * (K / kGroup) + grp;
    meta[j] = ((uint32_t)scales[s] << 16) | (uint32_t)(zeros[s] & 15u);
  }
}

}  // namespace

size_t w4_code_bytes(int N, int K) { return (size_t)N * K / 2; }
size_t w4_packed_bytes(int N, int K) { return w4_code_bytes(N, K) + (size_t)(K / kGroup) * N * 4; }

gs_status launch_pack_weight_w4(const void* q, const void* scales, const void* zeros, void* packed, int N, int K,
                                hipStream_t stream) {
  const size_t total = (size_t)N * K / 8 + (size_t)(K / kGroup) * N;
  uint32_t* codes = static_cast<uint32_t*>(packed);
  uint32_t* meta = reinterpret_cast<uint32_t*>(static_cast<char*>(packed) + w4_code_bytes(N, K));
  pack_w4_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(
      static_cast<const uint8_t*>(q), static_cast<const bf16_t*>(scales), static_cast<const uint8_t*>(zeros), codes,
      meta, N, K);
  GS_LAUNCH_CHECK("pack_w4");
  return GS_OK;
}

// Launch shape of the 4-bit kernel: waves x kg waves per workgroup, nt column tiles per wave, mt row tiles of 32.
//   up to 32 rows: the weight stream is all there is; 8 waves side by side, K splits for two workgroups per compute unit up to
//     16 rows, for one beyond, where the partial results weigh more (32 rows, 8192 x 8192: 14.5 us and 16.8 MB with two, 13.8 us
//     and 8.4 MB with one)
//   33 to 96 rows: 4 waves x 2 K groups, or 2 x 4 (narrow matrices, below); two column tiles per wave (a fragment read from LDS feeds two MFMAs) for matrices of
//     192 blocks of 256 columns and more, and where every wave still gets 16 steps; otherwise one
//     (92 rows, isolated: 8192 x 28672 49 us with two, 54 with one; 8192 x 8192 22.0 and 20.8; 10240 x 8192 26.5 and 25.8)
//   more rows: chunks of 128; 4 waves x 2 K groups with two column tiles where that gives three compute units in four a workgroup of at least
//     eight steps per group, else 8 waves side by side with one tile and shorter K splits.  With one tile the fragments read from LDS
//     are at its limit of 128 bytes per cycle; two tiles fit the registers with one step of weights and activations ahead.  Isolated,
//     us, one tile -> two: 28672 x 4096 at 128 / 256 / 1024 / 2047 rows 37.3 -> 35.2, 63.6 -> 57.8, 247 -> 233, 461 -> 435; 1024 rows of 4096 x 14336
//     111 -> 103, of 6144 x 4096 55.4 -> 51.2; 312 rows of 57344 x 8192 340 -> 313, of 8192 x 28672 180 -> 163; at the line 4096 x 4096 at 300 rows
//     19.3 -> 19.1, 6144 x 4096 at 160 18.7 -> 18.5; before it 4096 x 4096 at 250 rows 16.0 -> 18.8, 2560 x 2560 at 1024 21.0 -> 22.9.  (512 columns
//     per workgroup, 8 x 1 waves: 217 for the first at 1024 rows, but 1026 for 128256 x 4096, 964 this way; one wave per SIMD 250.)
// Inside a verification step, us per launch (predecessor, with two LDS buffers and one burst of loads per step, in
// brackets): 92 rows, 70B shape: gate/up 101 (123, and 8.5 for the separate SwiGLU), 8192 x 28672 52, 8192 x 8192 22.9 (67
// on average), QKV 27.3 (33.5), LM head 205 (250); 53 rows, 8B shape: gate/up 26.3 (32, and 6), 4096 x 14336 and 4096 x 4096 13.2 on
// average (14.9), QKV 10.7 (15.1), LM head 83.5 (89.6).
struct W4Plan {
  int mt, m_chunks, waves, kg, nt, n_blocks, splits, k_per;
};

static W4Plan w4_plan(int M, int N, int K) {
  W4Plan p;
  p.mt = M <= 32 ? 1 : M <= 64 ? 2 : M <= 96 ? 3 : 4;
  p.m_chunks = ceil_div(M, 32 * p.mt);
  int target = 256;      // workgroups: one per compute unit
  p.nt = 1;
  if (p.mt == 1) {
    p.waves = N % 256 == 0 ? 8 : 4;
    p.kg = p.waves == 8 ? 1 : 2;
    if (M <= 16) target = 512;
  } else if (p.mt == 4) {
    const bool fills = (long)(N / 256) * p.m_chunks * (K / 1024) >= 192;
    p.nt = N % 256 == 0 && fills ? 2 : 1;
    p.waves = N % 256 == 0 && !fills ? 8 : 4;
    p.kg = p.waves == 8 ? 1 : 2;
  } else {
    p.waves = 4;
    p.kg = 2;
    if (N % 256 == 0) {
      const int blocks = N / 256, s = blocks >= 192 ? 1 : std::max(1, target / blocks);
      if (blocks >= 192 || K / 64 >= 16 * p.kg * s) p.nt = 2;
    }
  }
  // narrow matrices at 33 to 64 rows: 64 columns and four K groups per workgroup, down to four steps each, where that gives seven
  // compute units in eight a workgroup with half of the K splits, or as many splits as K allows (8B shape, 8 layers, 53 rows 952 -> 934 us;
  // 1024 x 4096 8.6 -> 7.0 us; but 6144 x 12288, 5 splits on 240 workgroups, 18.6 -> 21.9 with 2 on 192).  From 128 blocks on the
  // larger share of the activations costs more: 70B shape, 2 layers, 45 rows 587 -> 604.
  const int blocks64 = N / 64, splits64 = std::max(1, std::min(target / blocks64, K / 1024));
  const bool narrow = p.mt == 2 && p.nt == 1 && blocks64 < 128 && (blocks64 * splits64 >= 224 || splits64 >= K / 1024);
  if (narrow || N % (32 * p.waves * p.nt) != 0) {      // N is a multiple of 64
    p.waves = 2;
    p.kg = p.mt == 4 ? 2 : 4;      // (LDS: kg x 3 activation buffers)
  }
  p.n_blocks = N / (32 * p.waves * p.nt);
  // K splits: every one adds an M x N fp32 partial result to write and re-read, so as many as fill the chip once, with
  // at least 8 steps per K group (4 in narrow matrices)
  const int wgs = p.n_blocks * p.m_chunks;
  const int s = std::max(1, std::min(target / wgs, K / ((narrow ? 256 : 512) * p.kg)));
  p.k_per = ceil_div(ceil_div(K, s), kGroup) * kGroup;      // whole scale groups per split
  p.splits = ceil_div(K, p.k_per);
  return p;
}

int gemm_w4_splits(int M, int N, int K) { return M <= 0 ? 1 : w4_plan(M, N, K).splits; }

// Whether the gate/up projection runs unsplit with the SwiGLU in its epilogue: up to 64 rows with 2 waves x 4 K groups
// (128 columns per workgroup; 53 rows of the 8B shape 26 us, against 25 and a separate SwiGLU of 6), up to 96 with 4 x 2
// (256 columns), where that fills more than half of the compute units.
static int w4_gate_up_blocks(int M, int F) {
  if (M <= 64) return F % 64 == 0 ? F / 64 : 0;
  return M <= 96 && F % 128 == 0 ? F / 128 : 0;
}
bool w4_gate_up_fused(int M, int F) { return w4_gate_up_blocks(M, F) > 128; }

// Steps in registers: four of weights, of activations one up to 64 rows (registers: isolated 53 x 4096 x 14336 17.2 -> 16.7 us with one
// instead of two, LM head at 53 / 12 rows 92.6 -> 90.9 / 68.9 -> 66.6) and two for 96 (LM head of the 70B shape 217.5 -> 215.7);
// 128 rows with two tiles: two and one.  Whole step of the 8B shape, 8 servers: 908 -> 892 us.
#define GS_W4(WN, KG, MT, NT, WPE, MODE)                                                                            \
  gemm_w4_kernel<WN, KG, MT, NT, (MT) == 4 && (NT) == 2 ? 2 : 4, (MT) == 3 || ((MT) == 4 && (NT) == 1) ? 2 : 1, WPE, MODE><<<grid, 64 * WN * KG, 0, stream>>>(x, codes, meta, P, M, N, K, k_per, chunks)

// act [M][F] (bf16) = silu(X Wg^T) * (X Wu^T); only where w4_gate_up_fused.
gs_status launch_gemm_w4_gate_up(const void* X, const void* Wpacked, void* act, int M, int F, int K, hipStream_t stream) {
  const bf16_t* x = static_cast<const bf16_t*>(X);
  const int N = 2 * F, k_per = K, chunks = 1;
  const uint4* codes = static_cast<const uint4*>(Wpacked);
  const uint32_t* meta = reinterpret_cast<const uint32_t*>(static_cast<const char*>(Wpacked) + w4_code_bytes(N, K));
  float* P = static_cast<float*>(act);
  const int grid = w4_gate_up_blocks(M, F);
  if (M <= 32) GS_W4(2, 4, 1, 2, 2, kGateUp);
  else if (M <= 64) GS_W4(2, 4, 2, 2, 2, kGateUp);
  else GS_W4(4, 2, 3, 2, 2, kGateUp);
  GS_LAUNCH_CHECK("gemm_w4_gate_up");
  return GS_OK;
}

// P [splits][M][N] fp32 partial sums of X [M][K] (bf16) * W^T with W given in the packed 4-bit layout.
gs_status launch_gemm_w4(const void* X, const void* Wpacked, float* P, int M, int N, int K, hipStream_t stream) {
  if (M <= 0) return GS_OK;
  const W4Plan p = w4_plan(M, N, K);
  const bf16_t* x = static_cast<const bf16_t*>(X);
  const uint4* codes = static_cast<const uint4*>(Wpacked);
  const uint32_t* meta = reinterpret_cast<const uint32_t*>(static_cast<const char*>(Wpacked) + w4_code_bytes(N, K));
  const int k_per = p.k_per, chunks = p.m_chunks;
  const int grid = p.n_blocks * p.m_chunks * p.splits;
  switch (p.mt) {
    case 1:
      if (p.waves == 8) GS_W4(8, 1, 1, 1, 4, kPlain);
      else if (p.waves == 4) GS_W4(4, 2, 1, 1, 4, kPlain);
      else GS_W4(2, 4, 1, 1, 4, kPlain);
      break;
    case 2:
      if (p.nt == 2) GS_W4(4, 2, 2, 2, 2, kPlain);
      else if (p.waves == 4) GS_W4(4, 2, 2, 1, 2, kPlain);
      else GS_W4(2, 4, 2, 1, 2, kPlain);
      break;
    case 3:
      if (p.nt == 2) GS_W4(4, 2, 3, 2, 2, kPlain);
      else if (p.waves == 4) GS_W4(4, 2, 3, 1, 2, kPlain);
      else GS_W4(2, 4, 3, 1, 2, kPlain);
      break;
    default:
      if (p.nt == 2) GS_W4(4, 2, 4, 2, 2, kPlain);
      else if (p.waves == 8) GS_W4(8, 1, 4, 1, 2, kPlain);
      else if (p.waves == 4) GS_W4(4, 2, 4, 1, 2, kPlain);
      else GS_W4(2, 2, 4, 1, 1, kPlain);
  }
  GS_LAUNCH_CHECK("gemm_w4");
  return GS_OK;
}
#undef GS_W4

}  // namespace gs
