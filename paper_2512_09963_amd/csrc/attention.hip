// Ragged, paged-KV, grouped-query causal attention for the speculative blocks.
//
// Row j of server i (position L_i + j) attends to keys 0 .. L_i + j of that server; the
// cache holds L_i keys and the block's own T_i keys were appended just before.  Page layouts:
//   K pages [page][H_kv][slot][hd]   (key-major: a key's head vector is contiguous)
//   V pages [page][H_kv][hd][slot]   (transposed: the slots of one channel are contiguous)
//
// bf16 path (MFMA): one workgroup per (server, group of query rows, KV head, KV split), one wave per 32 of the
// T_i * G query rows that share the KV head (token-major, head-minor), so each K/V byte leaves
// HBM once per workgroup; K/V stream through a two-stage LDS buffer filled by direct global->LDS
// loads.  The first product is computed transposed (S^T = K Q^T), which leaves a query's scores in
// the registers of two lanes, in exactly the order the second product (O^T += V^T P) wants its P
// operand, so P never leaves registers and neither product needs an LDS transpose.  Blocks of a few rows are one
// group; prompt blocks are cut into groups of 4 waves, each with the keys up to its own last row.  The number of
// KV splits of a group follows its own key count (a fixed number of 32-key steps per
// workgroup), so ragged batches stay balanced.  Partial results of the splits are merged by
// attn_combine_kernel; the result of a group that is not split is final and stored by the kernel itself.
//
// fp32 path (attn_rowwise_kernel): one workgroup per (row, head), 128 keys at a time, 16 lanes to a key; the softmax state is one per
// workgroup.
#include "common.h"
#include "attn_work.h"
#include "device_types.h"
#include "gemm_common.h"
#include <algorithm>
#include <cmath>

namespace gs {
namespace {

constexpr float kNegBig = -1.0e30f;

// ------------------------------------------------------------------------------------------
// fp32 path.  grid (R, H), 4 waves, kRowKeys keys at a time.  Scores: 16 lanes share a key (a lane has HD / 16 of its
// channels, the sum is four row moves).  Output: a lane has the keys 4 i .. 4 i + 3 of HD / 64 channels, so that both
// products read memory in whole lines; the four lanes of a channel are neighbours.  Latency bound (a few dozen rows and
// keys): all loads of K and V of a chunk are issued before the first score, so a chunk costs two dependent trips to memory
// (pages, then K and V), and the softmax state is formed by every wave for itself from the scores in LDS.  A lane per key
// with the lanes' states merged at the end took 13.6 us at 16 rows of 4 heads, 69 keys and head size 64, this takes 5.6.
// VEC: 16-byte loads (16-byte aligned pages, page size a multiple of 4).  AHEAD: the pages of the next chunk are looked up while
// this one is computed, one dependent trip per chunk; for launches of at most two workgroups per compute unit, which wait
// for loads and not for the units (kRowAheadItems).  Writes attn_out [R][H*hd].
// ------------------------------------------------------------------------------------------
constexpr int kRowThreads = 256;
constexpr int kRowKeys = 128;
constexpr int kRowAheadItems = 512;
template <int HD, bool VEC, bool AHEAD>
__global__ __launch_bounds__(kRowThreads) void attn_rowwise_kernel(const float* __restrict__ q,
                                                                   const float* __restrict__ k_pages,
                                                                   const float* __restrict__ v_pages,
                                                                   const int* __restrict__ block_table, int max_blocks,
                                                                   const int4* __restrict__ row_info,
                                                                   const int* __restrict__ cu_rows,
                                                                   const int* __restrict__ ctx_len,
                                                                   int page_size, int n_heads, int n_kv,
                                                                   float* __restrict__ attn_out) {
  constexpr int C4 = HD / 64;                // groups of 4 channels of a lane (scores); channels of a lane (output)
  constexpr int KP = kRowKeys / 16;          // passes over the keys of a chunk: 16 keys each
  const int r = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int srv = row_info[r].w;
  const int n_keys = ctx_len[srv] + (r - cu_rows[srv]) + 1;
  const int kh = h / (n_heads / n_kv);
  const int* bt = block_table + (size_t)srv * max_blocks;
  __shared__ float score[kRowKeys], prob[kRowKeys];
  const int kl = tid >> 4, cl = (tid & 15) * 4;      // scores: key of a pass, first channel
  const int vq = (tid & 3) * 4, vd = tid >> 2;       // output: first key of a pass, channel
  float4 qv[C4];
#pragma unroll
  for (int j = 0; j < C4; ++j) qv[j] = *reinterpret_cast<const float4*>(q + ((size_t)r * n_heads + h) * HD + j * 64 + cl);
  const float scale = 1.0f / sqrtf((float)HD);
  float m = kNegBig, l = 0.f;
  float o[C4];
#pragma unroll
  for (int j = 0; j < C4; ++j) o[j] = 0.f;
  static_assert(VEC || !AHEAD, "one page per four keys");
  int k_page[KP], v_page[KP];      // AHEAD
  auto look_up = [&](int base) {
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      k_page[p] = bt[min(base + p * 16 + kl, n_keys - 1) / page_size];
      v_page[p] = bt[min(base + p * 16 + vq, n_keys - 1) / page_size];
    }
  };
  if constexpr (AHEAD) look_up(0);
  for (int base = 0; base < n_keys; base += kRowKeys) {
    float4 kv[KP][C4], vv[KP][C4];
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      const int key = min(base + p * 16 + kl, n_keys - 1);      // (keys past the end re-read the last one)
      const int blk = key / page_size;
      const int page = AHEAD ? k_page[p] : bt[blk];
      const float* kp = k_pages + (((size_t)page * n_kv + kh) * page_size + (key - blk * page_size)) * HD + cl;
#pragma unroll
      for (int j = 0; j < C4; ++j)
        kv[p][j] = VEC ? *reinterpret_cast<const float4*>(kp + j * 64)
                       : make_float4(kp[j * 64], kp[j * 64 + 1], kp[j * 64 + 2], kp[j * 64 + 3]);
    }
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      const int key0 = base + p * 16 + vq;
#pragma unroll
      for (int j = 0; j < C4; ++j) vv[p][j] = make_float4(0.f, 0.f, 0.f, 0.f);
      // four keys share a page where the page size is a multiple of 4; slots past the end hold stale data, never used
      if constexpr (VEC) {
        if (key0 < n_keys) {
          const int blk = key0 / page_size;
          const int page = AHEAD ? v_page[p] : bt[blk];
          const float* vp = v_pages + (((size_t)page * n_kv + kh) * HD + vd) * page_size + (key0 - blk * page_size);
#pragma unroll
          for (int j = 0; j < C4; ++j) vv[p][j] = *reinterpret_cast<const float4*>(vp + (size_t)j * 64 * page_size);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (key0 + i < n_keys) {
            const int blk = (key0 + i) / page_size;
            const float* vp = v_pages + (((size_t)bt[blk] * n_kv + kh) * HD + vd) * page_size + (key0 + i - blk * page_size);
#pragma unroll
            for (int j = 0; j < C4; ++j) reinterpret_cast<float*>(&vv[p][j])[i] = vp[(size_t)j * 64 * page_size];
          }
      }
    }
    if (AHEAD && base + kRowKeys < n_keys) look_up(base + kRowKeys);
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < C4; ++j)
        s += (qv[j].x * kv[p][j].x + qv[j].y * kv[p][j].y) + (qv[j].z * kv[p][j].z + qv[j].w * kv[p][j].w);
      s = row16_sum(s);
      if ((tid & 15) == 0) score[p * 16 + kl] = base + p * 16 + kl < n_keys ? s * scale : kNegBig;
    }
    __syncthreads();
    // every wave forms the chunk's maximum and sum for itself; waves 0 and 1 store the weights
    const float s0 = score[lane], s1 = score[64 + lane];
    const float m_new = fmaxf(m, wave_max(fmaxf(s0, s1)));      // (a chunk has a key: m_new is a score)
    const float corr = expf(m - m_new);
    const float p0 = base + lane < n_keys ? expf(s0 - m_new) : 0.f, p1 = base + 64 + lane < n_keys ? expf(s1 - m_new) : 0.f;
    l = l * corr + wave_sum(p0 + p1);
    m = m_new;
    if (tid < 64) prob[lane] = p0;
    else if (tid < 128) prob[64 + lane] = p1;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C4; ++j) o[j] *= corr;
#pragma unroll
    for (int p = 0; p < KP; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float w = prob[p * 16 + vq + i];
        const bool has = base + p * 16 + vq + i < n_keys;      // (a weight of zero must not meet stale infinities)
#pragma unroll
        for (int j = 0; j < C4; ++j) o[j] = fmaf(w, has ? reinterpret_cast<const float*>(&vv[p][j])[i] : 0.f, o[j]);
      }
    // (the next chunk's scores are written after its loads; its barrier comes after all reads of prob here, and prob is
    // written behind that barrier)
  }
#pragma unroll
  for (int j = 0; j < C4; ++j) {
    float v = o[j];
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    if ((tid & 3) == 0) attn_out[((size_t)r * n_heads + h) * HD + j * 64 + vd] = v / l;
  }
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA path.  1-D grid over the (work list entry, KV head) items (item_of_workgroup), NW waves per workgroup, or KW key
// groups of NW waves that take the steps of the split in turn (kKeyGroups).
//
// A workgroup owns one split of one (server, query group, KV head): a group's steps are dealt evenly to its
// ceil(steps / steps_per_split) splits; a step is 32
// keys = two 16-key tiles = 16 KB of K and V at hd 128.  K/V go from global memory straight into
// a two-stage LDS buffer with direct global->LDS loads (no register staging).  A stage has four
// parts, K and V of either tile; part p is loaded by wave p % NW (waves 0..3 when NW > 4), whose
// HD/32 load instructions of 1 KB each share one scalar base address.  One barrier per step both
// publishes the stage that has landed and frees the stage that is refilled next.  (Deeper buffers
// were measured, with and without the arithmetic: no gain.)  K is placed in LDS so that lane (g, c) of fragment (tile, ks) holds
// key c, channels 32 ks + 8 g .. at fragment * 1 KB + lane * 16; V pages are copied verbatim
// ([channel][16 slots] per tile).
// Wave w computes query rows 32 w .. 32 w + 31 of the group's rows that share the KV head (token-major,
// head-minor); both products use the 32x32x16 MFMA (twice the issue rate of the 16x16x32 one on this
// chip):
//   S^T (32 keys x 32 queries) = K Q^T : A = K, lane l holds key l%32 (tile l%32/16 of the step),
//       channels 16 kk + 8 (l/32) .. of k step kk; B = Q^T, lane l holds query row l%32, same channels.
//       Result register v of lane l is row 8 (v/4) + 4 (l/32) + v%4 of query l%32; row r is key r with bits 2 and 3
//       exchanged, so that registers 8 kk' .. 8 kk' + 7 are the keys 16 kk' + 8 (l/32) .. + 7.
//   O^T (hd x 32 queries) += V^T P : B = P straight from the result registers of the first product:
//       k slot i of k step kk' (16 keys) is register 8 kk' + i, i.e. key 16 kk' + 8 (l/32) + i;
//       A = V^T in the same key order: channel 32 dt + l%32, 16 contiguous bytes of the transposed page (rows in
//       key order would make it two runs of 8 bytes, with half of the LDS banks idle: a 2047-token prompt 114 us per layer, so
//       104; 16 servers of the 70B shape 58.2 and 56.6, 8 of the 8B shape 18.0 and 17.5).
// A query row lives in lanes l and l + 32: one lane swap finishes its max and its sum, and the
// accumulator rescale is a per-lane multiply.  P enters the second product as a two-term bf16 sum.
// partial_o [R][H][max_splits][HD] fp32, partial_ml [R][H][max_splits][2]; splits beyond a group's own
// count are never written and never read.
// ------------------------------------------------------------------------------------------
// Which (work list entry, KV head) a workgroup of the 1-D attention grid takes: the items, entry-major (the KV
// heads of an entry are neighbours, so they go to the 8 XCDs), in rounds of one item per compute unit, the
// rounds alternately forwards and backwards, counted from the last one, which is taken forwards (it may be
// partial, and the grid has no workgroup beyond the items: padding workgroups in the middle of a launch that
// fills every slot kept the last workgroups of one XCD waiting for a slot).  The list being sorted by
// length, the sums of the items that meet on a compute unit are nearly equal, and the compute units that get
// one item more get the shortest ones on top of the smaller sums.
constexpr int kComputeUnits = 256;
constexpr int kGroupWaves = 4;      // of the query groups of a prompt (attention_groups)
__device__ __forceinline__ void item_of_workgroup(int wg, int n_items, int n_kv, int& entry, int& kh) {
  const int rounds = (n_items + kComputeUnits - 1) / kComputeUnits;
  const int round = wg / kComputeUnits, c = wg - round * kComputeUnits;
  const bool backwards = ((rounds - 1 - round) & 1) != 0;      // (a backward round is never the partial one)
  const int item = round * kComputeUnits + (backwards ? kComputeUnits - 1 - c : c);
  entry = item / n_kv;
  kh = item - entry * n_kv;
}

// cache policy of the K/V loads (the builtin's last argument; bit 1 = non-temporal).  A block of one row tile reads its
// keys and values once; they should not displace the partial results and the block tables in L2 (32 ragged servers:
// 3.4 instead of 3.6 ms of attention per step, 8 servers unchanged).  The query groups of a long prompt each read all
// of its keys, and the policy costs them nothing: 112 to 114 us per layer with and without it for a prompt of 2047
// tokens, 15.4 with and without for 8 of 128; 149 with, 176 without for one of 256 beside 24 blocks on 8192.
constexpr int kKvLoadPolicy = 2;

// The reference that a row's exponentials are taken against follows its maximum only when that is 2^8 above it: the weights are up to
// 256 instead of 1, with the same relative precision in all sums (and in their two-term bf16 form), and most steps neither multiply the
// accumulators nor wait for the factor.  us per layer: 8 servers at 2048 tokens 17.5 -> 16.5, 16 of the 70B shape 56.6 -> 54.2.
constexpr float kRescaleAt = 8.f;

__device__ __forceinline__ void wait_all_vector_loads() {
  // s_waitcnt vmcnt(0) alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8;
  // the other two fields at their maximum mean "do not wait")
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
}

typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

__device__ __forceinline__ float halves_max(float x) {
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// a / l correctly rounded, with inv = 1 / l correctly rounded: a product whose remainder is divided as well (Markstein, IBM J. Res.
// Dev. 34, 1990).  The 64 quotients of a lane share l: four instructions each instead of ten.  The remainder of an infinity is NaN, which
// the median turns into a finite number, so that infinities stay what they are.  8 layers of 32 heads of 128 over 8, one server on 20 tokens,
// replayed: product alone 208 us, this 212, with a comparison and a selection instead of the median 214.
__device__ __forceinline__ float quotient(float a, float l, float inv) {
  const float q = a * inv;
  return fmaf(__builtin_amdgcn_fmed3f(fmaf(-q, l, a), -3.0e38f, 3.0e38f), inv, q);
}

// (165 vector registers: three waves per SIMD, i.e. up to four 3-wave workgroups per CU, which hides a
// workgroup's start-up and barrier stalls behind the others' loads)
template <int HD, int G, int NW, int KW>
__global__ __launch_bounds__(64 * NW * KW) __attribute__((amdgpu_waves_per_eu(NW * KW == 4 && KW > 1 ? 1 : NW == 1 || KW > 1 ? 2 : 3))) void attn_kernel(const bf16_t* __restrict__ q,
                                                         const bf16_t* __restrict__ k_pages,
                                                         const bf16_t* __restrict__ v_pages,
                                                         const int* __restrict__ block_table, int max_blocks,
                                                         const int* __restrict__ work, int n_work, int page_size,
                                                         int n_heads, int n_kv, int steps_per_split,
                                                         int max_splits, float* __restrict__ partial_o,
                                                         float* __restrict__ partial_ml,
                                                         bf16_t* __restrict__ attn_out, bool packed) {
  constexpr int KS = HD / 32;            // 1 KB loads per part
  constexpr int KK = HD / 16;            // k steps of the first product
  constexpr int DT = HD / 32;            // 32-channel tiles of the second product
  constexpr int PART = HD * 32;          // bytes of K (or V) of one 16-key tile
  constexpr int STAGE = 4 * PART;        // K tile 0, K tile 1, V tile 0, V tile 1
  constexpr int STATES = KW / 2 * NW * (HD * 128 + 512);      // of half of the key groups, see the merge
  __shared__ __attribute__((aligned(16))) unsigned char rings[KW * 2 * STAGE > STATES ? KW * 2 * STAGE : STATES];

  int entry, kh;
  item_of_workgroup(blockIdx.x, n_work * n_kv, n_kv, entry, kh);
  // (n_work never exceeds the list's capacity, so the entry may be read before the device's count is known)
  const AttnWork wk = *reinterpret_cast<const AttnWork*>(work + 8 + 8 * entry);
  if (entry >= work[0]) return;
  const int srv = wk.srv, split = wk.split, row0 = wk.row0, T = wk.n_tokens, L = wk.ctx;
  const int first_pages[2] = {wk.page0, wk.page1};
  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int key_group = KW > 1 ? wave_all / NW : 0, wave = KW > 1 ? wave_all % NW : wave_all;
  unsigned char* ring = rings + key_group * 2 * STAGE;
  const int h = lane >> 5, c32 = lane & 31;
  const int g = lane >> 4, c = lane & 15;            // loader roles
  const int n_keys = L + T;
  const int n_steps_all = (n_keys + 31) >> 5;
  // the group's steps are dealt evenly to its ceil(steps / steps_per_split) splits (sizes differ by at most
  // one): a short remainder split would leave its slot idle while the full-length ones decide the duration
  const int n_splits = (n_steps_all + steps_per_split - 1) / steps_per_split;
  if (split >= n_splits) return;
  const int base_steps = n_steps_all / n_splits, extra = n_steps_all - base_steps * n_splits;
  const int n_wg = base_steps + (split < extra ? 1 : 0);
  // the key groups take the steps of the split in turn
  const int step_begin = split * base_steps + min(split, extra) + key_group;
  const int n = KW > 1 ? (n_wg - key_group + KW - 1) / KW : n_wg;
  const int* bt = block_table + (size_t)srv * max_blocks;
  const bool page_pow2 = (page_size & (page_size - 1)) == 0;
  const int page_shift = 31 - __builtin_clz(page_size);
  const int last_tile_key = ((n_keys - 1) >> 4) << 4;

  // ---- this wave's 32 query rows
  const int tile_row0 = wk.tok0 * G + wave * 32;
  const int rows = T * G - tile_row0;
  const bool has_rows = rows > 0;
  const int my_lr = tile_row0 + c32;
  const bool my_ok = c32 < rows;
  const int my_j = my_ok ? my_lr / G : 0, my_hg = my_ok ? my_lr - my_j * G : 0;
  const int limit = my_ok ? L + my_j : -1;
  const int first_limit = L + tile_row0 / G;      // every row of the wave sees the keys up to here
  const int j_max = min(T - 1, (tile_row0 + 31) / G);
  const int my_step_end = has_rows ? ((L + j_max) >> 5) + 1 : 0;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
  bf16x8_t qf[KK];
  {
    const bf16_t* src = q + ((size_t)(row0 + my_j) * n_heads + kh * G + my_hg) * HD + h * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (my_ok) v = *reinterpret_cast<const uint4*>(src + kk * 16);
      qf[kk] = *reinterpret_cast<const bf16x8_t*>(&v);
    }
  }
  float m_run = kNegBig, l_run = 0.f;
  floatx16_t oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[dt][e] = 0.f;

  // block-table entry and first slot of the two 16-key tiles of a step (a tile past the end re-reads the last one)
  auto locate = [&](int step, int (&blk)[2], int (&slot0)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int key0 = min(step * 32 + t * 16, last_tile_key);
      blk[t] = page_pow2 ? key0 >> page_shift : key0 / page_size;
      slot0[t] = key0 - blk[t] * page_size;
    }
  };
  auto lookup = [&](int step, int (&page)[2], int (&slot0)[2]) {
    int blk[2];
    locate(step, blk, slot0);
    page[0] = bt[blk[0]];
    page[1] = bt[blk[1]];
  };
  const unsigned k_lane_off = (unsigned)(c * HD + g * 8) * 2u;
  const unsigned v_lane_off = (unsigned)((lane >> 1) * page_size + (lane & 1) * 8) * 2u;
  const char* k_bytes = reinterpret_cast<const char*>(k_pages);
  const char* v_bytes = reinterpret_cast<const char*>(v_pages);
  auto issue = [&](int slot, const int (&page)[2], const int (&slot0)[2]) {
    unsigned char* stage = ring + slot * STAGE;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      if (wave != (NW > 4 ? p : p % NW)) continue;
      const int t = p & 1;
      const size_t head = (size_t)page[t] * n_kv + kh;
      if (p < 2) {
        const char* src = k_bytes + (head * page_size + slot0[t]) * (HD * 2) + k_lane_off;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          __builtin_amdgcn_global_load_lds(src + ks * 64,
                                           (__attribute__((address_space(3))) void*)(stage + p * PART + ks * 1024),
                                           16, 0, kKvLoadPolicy);
      } else {
        const char* src = v_bytes + (head * HD * page_size + slot0[t]) * 2 + v_lane_off;
        const size_t stride = (size_t)64 * page_size;
#pragma unroll
        for (int ch = 0; ch < KS; ++ch)
          __builtin_amdgcn_global_load_lds(src + ch * stride,
                                           (__attribute__((address_space(3))) void*)(stage + p * PART + ch * 1024),
                                           16, 0, kKvLoadPolicy);
      }
    }
  };

  int pg_next[2], sl_next[2];
  if (key_group == 0) {
    int blk[2];
    locate(step_begin, blk, sl_next);
    issue(0, first_pages, sl_next);
  } else if (n > 0) {
    lookup(step_begin, pg_next, sl_next);
    issue(0, pg_next, sl_next);
  }
  if (1 < n) lookup(step_begin + KW, pg_next, sl_next);

  // K fragment of k step kk for this lane: tile c32/16, fragment kk/2, lane group 2 (kk%2) + h, key c32%16 with bits 2 and 3 exchanged
  const int k_lane = ((c32 >> 4) * KS * 64 + h * 16 + ((c32 & 3) | ((c32 & 4) << 1) | ((c32 & 8) >> 1))) * 16;
  // V: channel c32 of a 32-channel tile is 32 bytes per 16-key tile; this lane's run starts at slot 8h
  const int v_lane = 2 * PART + c32 * 32 + h * 16;

  for (int s = 0; s < (KW > 1 ? (n_wg + KW - 1) / KW : n); ++s) {
    const int step = step_begin + s * KW;
    wait_all_vector_loads();     // this wave's parts of stage s have landed
    __syncthreads();             // stage s complete for all waves; the other stage is free
    if (s + 1 < n) {
      issue((s + 1) & 1, pg_next, sl_next);
      if (s + 2 < n) lookup(step + 2 * KW, pg_next, sl_next);     // for the next iteration's issue
    }
    if (s >= n || step >= my_step_end) continue;

    const unsigned char* base = ring + (s & 1) * STAGE;
    bf16x8_t kf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      kf[kk] = *reinterpret_cast<const bf16x8_t*>(base + k_lane + (kk >> 1) * 1024 + (kk & 1) * 512);
    floatx16_t sacc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], sacc, 0, 0, 0);

    float p[16];
    float corr;
    if (step * 32 + 31 <= first_limit) {
      float mx = sacc[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sacc[e]);
      mx = halves_max(mx) * scale_log2;
      const float m_new = mx > m_run + kRescaleAt ? mx : m_run;
      corr = __builtin_amdgcn_exp2f(m_run - m_new);
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[e], scale_log2, -m_new));
        sum += p[e];
      }
      l_run = l_run * corr + halves_sum(sum);
      m_run = m_new;
    } else {
      float sv[16];
      float mx = kNegBig;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = step * 32 + (e >> 3) * 16 + h * 8 + (e & 7);
        sv[e] = key <= limit ? sacc[e] * scale_log2 : kNegBig;
        mx = fmaxf(mx, sv[e]);
      }
      mx = halves_max(mx);
      const float m_new = mx > m_run + kRescaleAt ? mx : m_run;
      corr = __builtin_amdgcn_exp2f(m_run - m_new);
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        p[e] = (sv[e] > kNegBig) ? __builtin_amdgcn_exp2f(sv[e] - m_new) : 0.f;
        sum += p[e];
      }
      l_run = l_run * corr + halves_sum(sum);
      m_run = m_new;
    }
    // P as a two-term bf16 sum (value and rounding remainder); k step kk' takes registers 8 kk' .. 8 kk' + 7
    bf16x8_t pf[2], pf_lo[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      uint4 hi, lo;
      const float* pp = p + 8 * kk;
      hi.x = pack_bf16x2(pp[0], pp[1]);
      hi.y = pack_bf16x2(pp[2], pp[3]);
      hi.z = pack_bf16x2(pp[4], pp[5]);
      hi.w = pack_bf16x2(pp[6], pp[7]);
      lo.x = pack_bf16x2(pp[0] - __uint_as_float(hi.x << 16), pp[1] - __uint_as_float(hi.x & 0xffff0000u));
      lo.y = pack_bf16x2(pp[2] - __uint_as_float(hi.y << 16), pp[3] - __uint_as_float(hi.y & 0xffff0000u));
      lo.z = pack_bf16x2(pp[4] - __uint_as_float(hi.z << 16), pp[5] - __uint_as_float(hi.z & 0xffff0000u));
      lo.w = pack_bf16x2(pp[6] - __uint_as_float(hi.w << 16), pp[7] - __uint_as_float(hi.w & 0xffff0000u));
      pf[kk] = *reinterpret_cast<const bf16x8_t*>(&hi);
      pf_lo[kk] = *reinterpret_cast<const bf16x8_t*>(&lo);
    }
    // the rescale factor of a query row sits in the lanes that hold the row: a per-lane multiply, skipped while no
    // row's maximum has passed its reference by 2^8
    if (__any(corr != 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[dt][e] *= corr;
    }
    // second product, two channel tiles at a time (16 fragment registers live instead of 32)
    const bool tail = step * 32 + 32 > n_keys;
    uint4 keep[2];
    if (tail) {
      // keys past the end of the sequence inside the last page hold stale data: zero their V
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int kb0 = step * 32 + 16 * kk + 8 * h, kb1 = kb0 + 4;
        keep[kk].x = (kb0 + 0 < n_keys ? 0x0000ffffu : 0u) | (kb0 + 1 < n_keys ? 0xffff0000u : 0u);
        keep[kk].y = (kb0 + 2 < n_keys ? 0x0000ffffu : 0u) | (kb0 + 3 < n_keys ? 0xffff0000u : 0u);
        keep[kk].z = (kb1 + 0 < n_keys ? 0x0000ffffu : 0u) | (kb1 + 1 < n_keys ? 0xffff0000u : 0u);
        keep[kk].w = (kb1 + 2 < n_keys ? 0x0000ffffu : 0u) | (kb1 + 3 < n_keys ? 0xffff0000u : 0u);
      }
    }
#pragma unroll
    for (int d0 = 0; d0 < DT; d0 += 2) {
      uint4 vv[2][2];
#pragma unroll
      for (int dd = 0; dd < 2; ++dd)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const unsigned char* vp = base + v_lane + kk * PART + (d0 + dd) * 1024;
          // (native vector type: an LDS read without type metadata makes the compiler wait for every
          // outstanding global->LDS load first, which would drain the prefetched stage in mid-step)
          const uintx4_t a = *reinterpret_cast<const uintx4_t*>(vp);
          vv[dd][kk] = make_uint4(a.x, a.y, a.z, a.w);
        }
      if (tail) {
#pragma unroll
        for (int dd = 0; dd < 2; ++dd)
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) {
            vv[dd][kk].x &= keep[kk].x; vv[dd][kk].y &= keep[kk].y; vv[dd][kk].z &= keep[kk].z; vv[dd][kk].w &= keep[kk].w;
          }
      }
#pragma unroll
      for (int dd = 0; dd < 2; ++dd)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const bf16x8_t vf = *reinterpret_cast<const bf16x8_t*>(&vv[dd][kk]);
          oacc[d0 + dd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kk], oacc[d0 + dd], 0, 0, 0);
          oacc[d0 + dd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf_lo[kk], oacc[d0 + dd], 0, 0, 0);
        }
    }
  }

  // ---- the key groups' states meet in LDS, half of them handing theirs to the other half
  if constexpr (KW > 1) {
#pragma unroll
    for (int half = KW / 2; half >= 1; half /= 2) {
      __syncthreads();      // (all fragment reads, or the reads of the round before, are done)
      float4* state = reinterpret_cast<float4*>(rings);
      float2* ml = reinterpret_cast<float2*>(rings + KW / 2 * NW * HD * 128);
      if (key_group >= half && key_group < 2 * half) {
        const int slot = (key_group - half) * NW + wave;
        ml[slot * 64 + lane] = make_float2(m_run, l_run);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            state[(slot * DT * 4 + dt * 4 + b) * 64 + lane] =
                make_float4(oacc[dt][4 * b], oacc[dt][4 * b + 1], oacc[dt][4 * b + 2], oacc[dt][4 * b + 3]);
      }
      __syncthreads();
      if (key_group < half) {
        const int slot = key_group * NW + wave;
        const float2 other = ml[slot * 64 + lane];
        const float m_new = fmaxf(m_run, other.x);
        const float f = __builtin_amdgcn_exp2f(m_run - m_new), f_other = __builtin_amdgcn_exp2f(other.x - m_new);
        l_run = l_run * f + other.y * f_other;
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const float4 v = state[(slot * DT * 4 + dt * 4 + b) * 64 + lane];
            oacc[dt][4 * b] = oacc[dt][4 * b] * f + v.x * f_other;
            oacc[dt][4 * b + 1] = oacc[dt][4 * b + 1] * f + v.y * f_other;
            oacc[dt][4 * b + 2] = oacc[dt][4 * b + 2] * f + v.z * f_other;
            oacc[dt][4 * b + 3] = oacc[dt][4 * b + 3] * f + v.w * f_other;
          }
      }
    }
    if (key_group != 0) return;
  }
  // ---- lane l holds query row l%32, channels 32 dt + 8 b + 4 h + (0..3)
  if (!my_ok) return;
  if (n_splits == 1) {      // the group is not split: the result is final
    const int row = row0 + my_j, col0 = (kh * G + my_hg) * HD + 4 * h, width = n_heads * HD;
    const float inv = 1.0f / l_run;
    auto o = [&](int dt, int i) { return quotient(oacc[dt][i], l_run, inv); };
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        *reinterpret_cast<uint2*>(attn_out + (packed ? packed_index(row, col0 + dt * 32 + b * 8, width)
                                                     : (size_t)row * width + col0 + dt * 32 + b * 8)) =
            make_uint2(pack_bf16x2(o(dt, 4 * b), o(dt, 4 * b + 1)), pack_bf16x2(o(dt, 4 * b + 2), o(dt, 4 * b + 3)));
    return;
  }
  const size_t out_idx = ((size_t)(row0 + my_j) * n_heads + kh * G + my_hg) * max_splits + split;
  if (h == 0) {
    partial_ml[out_idx * 2 + 0] = m_run;
    partial_ml[out_idx * 2 + 1] = l_run;
  }
  float* dst = partial_o + out_idx * HD + 4 * h;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int b = 0; b < 4; ++b)
      *reinterpret_cast<float4*>(dst + dt * 32 + b * 8) =
          make_float4(oacc[dt][4 * b], oacc[dt][4 * b + 1], oacc[dt][4 * b + 2], oacc[dt][4 * b + 3]);
}

// attn_out[r][h*HD + d] = sum_s o_s * 2^(m_s - M) / sum_s l_s * 2^(m_s - M) over the splits of the row's query
// group; the rows of a group that is not split are final already.  HD / 4 lanes to a (row, head), 16 bytes per lane and split
// (324 rows of 32 heads 6.1 us, 53 rows 4.7; a workgroup per (row, head) with a lane per channel 7.8 and 4.9).  grid ceil(R * H / (1024 / HD)).
constexpr int kCombineThreads = 256;
template <int HD>
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(const float* __restrict__ partial_o, const float* __restrict__ partial_ml,
                                                                       int max_splits, int steps_per_split, const int4* __restrict__ row_info,
                                                                       int n_rows, int n_heads, bf16_t* __restrict__ attn_out, bool packed) {
  constexpr int LANES = HD / 4, PER_WG = kCombineThreads / LANES;
  const int rh = blockIdx.x * PER_WG + threadIdx.x / LANES, d = threadIdx.x % LANES * 4;
  if (rh >= n_rows * n_heads) return;
  const int row = rh / n_heads;
  const int n_keys = row_info[row].z;      // keys of the row's query group (per-row table of the step)
  const int n_splits = (((n_keys + 31) >> 5) + steps_per_split - 1) / steps_per_split;
  if (n_splits == 1) return;
  // one pass with a running maximum, so that no load waits for the maximum over all splits
  const float2* ml = reinterpret_cast<const float2*>(partial_ml) + (size_t)rh * max_splits;
  const float* po = partial_o + (size_t)rh * max_splits * HD + d;
  float M = kNegBig, Lsum = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int s = 0; s < n_splits; ++s) {
    const float2 st = ml[s];
    const float4 o = *reinterpret_cast<const float4*>(po + (size_t)s * HD);
    const float Mn = fmaxf(M, st.x);
    const float c = exp2f(M - Mn), f = exp2f(st.x - Mn);
    Lsum = Lsum * c + st.y * f;
    acc.x = acc.x * c + o.x * f;
    acc.y = acc.y * c + o.y * f;
    acc.z = acc.z * c + o.z * f;
    acc.w = acc.w * c + o.w * f;
    M = Mn;
  }
  const int col = (rh - row * n_heads) * HD + d;
  *reinterpret_cast<uint2*>(attn_out + (packed ? packed_index(row, col, n_heads * HD) : (size_t)rh * HD + d)) =
      make_uint2(pack_bf16x2(acc.x / Lsum, acc.y / Lsum), pack_bf16x2(acc.z / Lsum, acc.w / Lsum));
}

}  // namespace

// Query groups: waves per workgroup and tokens per group.  Up to 8 tiles of 32 query rows (T * G rows share a KV
// head) a block is one group of as many waves.  Longer blocks (prompts) are cut into groups of 4 waves: the groups are
// workgroups of one launch, each with the keys up to its own last token, which halves the work of a causal prompt
// and needs no KV splits to fill the chip.  (One launch per 8 tiles, every one of them over all keys in up to 11
// splits, took 720 us per layer for a 2047-token prompt at 32 heads and 107 us to merge the partials; now 70 us: 114 in groups, 104 with
// contiguous reads of the values, 87 with the mask only in the steps that some row of the wave does not see in full and fewer
// rescales, 70 with two key groups.  8 prompts of 128 tokens: 30 us and 14 us, now 12.7 us.)
constexpr int kMaxWaves = 8;
// Key groups: where a launch leaves compute units idle and a block is one tile of query rows, four waves of a workgroup take the
// steps of its split in turn (0.85 us a step), each with a ring of its own, and merge their states in LDS.  8B shape, 4 layers, one
// server at 700 / 2048 keys 395 -> 385 and 400 -> 393 us, two servers 408 -> 397 and 415 -> 408.  A workgroup then fills the LDS of a
// compute unit: with 256 of them 8 servers at 2048 keys take 499 instead of 492; two tiles of rows gain nothing.  (Fewer splits
// instead, as the key groups would allow, are slower: a compute unit alone streams 26 GB/s, 700 keys unsplit take 22 us, in four
// splits with the merge 15.)  On contexts of two steps the start of four rings and the merge cost more than the step they save.
// Replayed calls of 8 layers on 64 / 96 / 128 / 160 keys, one key group and four, us: one server, 32 heads of 128 over 8 217 / 226 / 236 /
// 245 and 221 / 225 / 228 / 238; 4 heads of 64 over 2 183 / 188 / 196 / 203 and 186 / 185 / 187 / 193; 16 servers of the latter 261 / 268 / 275 /
// 282 and 262 / 265 / 269 / 275.
constexpr int kKeyGroups = 4, kKeyGroupItems = 192, kKeyGroupSteps = 3;
// Prompts: the groups of a causal prompt have 1, 2, 3, ... times the steps of the first, and a compute unit that is dealt the longest and
// the shortest has one wave per SIMD most of the time, whose loads, products and exponentials follow each other.  Two key groups
// give every SIMD two waves.  us per layer, one and two: a prompt of 2047 tokens 87.1 and 70.4; 8 of 128 tokens (one to four steps) 12.7 and
// 12.9: so where the longest split has 8 steps or more.
constexpr int kPromptKeyGroups = 2, kPromptKeyGroupSteps = 8;
void attention_groups(int group, long max_block_tokens, int* waves, int* group_tokens) {
  const long tiles = (max_block_tokens * group + 31) / 32;
  *waves = tiles > kMaxWaves ? kGroupWaves : tiles > 0 ? (int)tiles : 1;
  *group_tokens = std::max(1, *waves * 32 / group);      // (a batch has groups of 1, 2, 4 or 8: 32 is a multiple of them)
}

// Calls f(steps, tokens) for every (server, query group): its number of 32-key steps and of tokens.
template <typename F>
static void for_each_group(int n_servers, const int* gamma_host, const int* ctx_len_host, int group_tokens, F f) {
  for (int i = 0; i < n_servers; ++i) {
    const long T = gamma_host[i] + 1L;
    for (long t0 = 0; t0 < T; t0 += group_tokens) {
      const long t1 = std::min(T, t0 + group_tokens);
      f((ctx_len_host[i] + t1 + 31) / 32, t1 - t0);
    }
  }
}

// Entries of the work list: (server, query group, split) triples.
long attention_items(int n_servers, const int* gamma_host, const int* ctx_len_host, int group_tokens, int steps_per_split) {
  long n = 0;
  for_each_group(n_servers, gamma_host, ctx_len_host, group_tokens,
                 [&](long st, long) { n += (st + steps_per_split - 1) / steps_per_split; });
  return n;
}

// Most (server, query group) pairs of a batch of that size (a group has at least kGroupWaves * 32 / 8 tokens
// or is its server's last one).
long attention_max_groups(int max_rows, int max_servers) { return (long)max_servers + max_rows / (kGroupWaves * 4); }

// The most 32-key steps any compute unit is dealt when every group's steps are cut into splits of at most t
// steps: item_of_workgroup's serpentine over the (server, group, split, KV head) items in the order of decreasing
// length, which is the order of the work list.  items: their number.  The histogram of lengths lives on the stack: splits
// of 2047 steps and more are counted in units of 2, 4, ... steps, rounded up.
long attention_busiest_cu(int n_kv, int n_servers, const int* gamma_host, const int* ctx_len_host, int group_tokens,
                          long t, long* items_out) {
  constexpr long kCus = kComputeUnits, kMaxLen = 2048;
  long n_of_len[kMaxLen] = {0};
  long items = 0;
  int shift = 0;
  while ((t >> shift) + 2 > kMaxLen) ++shift;
  auto units = [&](long len) { return (len + (1L << shift) - 1) >> shift; };
  for_each_group(n_servers, gamma_host, ctx_len_host, group_tokens, [&](long st, long) {
    const long n = (st + t - 1) / t;
    const long base = st / n, rem = st - base * n;
    items += n * n_kv;
    if (rem > 0) n_of_len[units(base + 1)] += rem * n_kv;
    n_of_len[units(base)] += (n - rem) * n_kv;
  });
  if (items_out) *items_out = items;
  const long rounds = (items + kCus - 1) / kCus;
  long load[kCus] = {0};
  long pos = 0;
  for (long len = units(t); len >= 1; --len)
    for (long k = 0; k < n_of_len[len]; ++k, ++pos) {
      const long round = pos / kCus, c = pos - round * kCus;
      load[((rounds - 1 - round) & 1) ? kCus - 1 - c : c] += len;
    }
  return *std::max_element(load, load + kCus) << shift;
}

// The split length for query groups that fill the chip.  On contexts of one length the serpentine deals the unsplit groups
// evenly, and splits would only add partial results.  On unequal contexts the longest groups would run on when the rest of the
// chip is done.  Fitted over batches of both kinds (261 to 2047 rows, contexts of 0 to 131000 tokens, the longest group in 1 to
// 32 splits), a launch and its merge take 20 us + 0.91 us per step of the busiest compute unit + 6.3 us per split of 128 rows and
// compute unit (its partial result).  So: the split count of the longest group, 2 .. 32, with the least steps + 7 x partial
// results, unless that gains less than 8 % over none.  8 KV heads, group 4, us per layer unsplit and as chosen:
// 8 x 128 tokens on 1 .. 1024 cached 57 and 35, 7 x 128 on none and 128 on 8192 cached 336 and 67, 1024 on none and 5 rows on
// 16384 562 and 68, 256 on none and 24 x 5 rows on 8192 280 and 149.
static long group_steps_per_split(int n_kv, int n_servers, const int* gamma_host, const int* ctx_len_host, int group_tokens,
                                  long shortest, long max_steps) {
  constexpr long kPartialSteps = 7;
  // in units of 1 / (compute units x tokens of a group) steps
  auto cost = [&](long t) {
    long partial_tokens = 0;
    for_each_group(n_servers, gamma_host, ctx_len_host, group_tokens, [&](long st, long tokens) {
      const long n = (st + t - 1) / t;
      if (n > 1) partial_tokens += n * tokens;
    });
    return attention_busiest_cu(n_kv, n_servers, gamma_host, ctx_len_host, group_tokens, t, nullptr) * kComputeUnits * group_tokens +
           kPartialSteps * n_kv * partial_tokens;
  };
  const long unsplit = cost(max_steps);
  long best = unsplit, sps = max_steps;
  for (long k = 2; k <= 32 && (max_steps + k - 1) / k >= shortest; ++k) {
    const long t = (max_steps + k - 1) / k, c = cost(t);
    if (c < best && c < unsplit / 100 * 92) {
      best = c;
      sps = t;
    }
  }
  return sps;
}

// KV steps (32 keys) per split, and the resulting largest split count, for a batch of n_servers servers with
// the given draft lengths and contexts and blocks of at most max_block_tokens rows.  A group's steps
// are cut into ceil(steps / steps_per_split) splits of equal length up to one step.  All workgroups of the
// launch should be resident at once (they share the memory bandwidth; a second round starts with the chip
// half empty: measured on the 70B shape, 5.9 instead of 6.7 ms per step), which also keeps the partial
// results few; a floor on the steps per split bounds what the partial results cost on small batches.
// Prompt blocks whose unsplit groups already give every compute unit a workgroup: see group_steps_per_split.
void attention_plan(int n_kv, int group, long max_block_tokens, int n_servers, const int* gamma_host,
                    const int* ctx_len_host, int* steps_per_split, int* max_splits, int* key_groups) {
  int waves, group_tokens;
  attention_groups(group, max_block_tokens, &waves, &group_tokens);
  constexpr int kWavesPerCu = 12;    // by registers (three waves per SIMD)
  const int wgs_per_cu = kWavesPerCu / waves < 5 ? (kWavesPerCu / waves > 0 ? kWavesPerCu / waves : 1) : 5;   // 5 workgroups by LDS
  const long slots = (long)kComputeUnits * wgs_per_cu;
  long total_steps = 0, max_steps = 1, n_groups = 0;
  for_each_group(n_servers, gamma_host, ctx_len_host, group_tokens, [&](long st, long) {
    total_steps += st;
    max_steps = std::max(max_steps, st);
    n_groups += 1;
  });
  // workgroups of a launch with splits of at most t steps
  auto workgroups = [&](long t) {
    return attention_items(n_servers, gamma_host, ctx_len_host, group_tokens, (int)t) * n_kv;
  };
  long lo = (max_steps + 31) / 32;                        // at most 32 splits per group
  if (lo < 6) lo = 6;                                     // at least 6 steps per split (partial-result traffic)
  if (lo > max_steps) lo = max_steps;
  const long fit = slots - slots / 16;                    // all resident at once, with some slack for placement
  long sps;
  if (n_groups > n_servers && n_groups * n_kv >= kComputeUnits) {
    // (beyond 2^17 groups, hundreds per compute unit, a search would take longer than it gains)
    sps = n_groups > (1L << 17) ? max_steps
                                : group_steps_per_split(n_kv, n_servers, gamma_host, ctx_len_host, group_tokens, lo, max_steps);
  } else if (workgroups(max_steps) <= fit) {
    // the shortest splits whose workgroups are all resident at once ...
    long a = lo, b = max_steps;
    while (a < b) {
      const long mid = (a + b) / 2;
      if (workgroups(mid) <= fit) b = mid; else a = mid + 1;
    }
    sps = a;
    // ... unless splits up to half longer than the best so far load the busiest compute unit clearly less (a compute unit's
    // finishing time follows the steps it is dealt): 3 x 22 instead of 4 x 19 steps at the 70B shape with 16
    // servers (5.3 against 5.6 ms of attention per step).  Small differences do not pay for the workgroups that
    // are then missing per compute unit (8 servers at 2048 tokens: 2 x 9 steps on 512 workgroups took 17.1 us
    // per layer, 3 x 6 on 704 take 15.1), hence the margin of 8 %.
    const long stride = std::max(1L, sps / 1024);      // (at most a thousand candidates or so, however long the contexts)
    long best = attention_busiest_cu(n_kv, n_servers, gamma_host, ctx_len_host, group_tokens, sps, nullptr);
    for (long t = sps + 1; t <= sps + sps / 2 && t <= max_steps; t += stride) {
      const long l = attention_busiest_cu(n_kv, n_servers, gamma_host, ctx_len_host, group_tokens, t, nullptr);
      if (l * 100 < best * 92) {
        best = l;
        sps = t;
      }
    }
  } else {
    // more (group, KV head) pairs than slots: several rounds of workgroups anyway
    sps = (total_steps * n_kv + slots / 2 - 1) / (slots / 2);
    if (sps < lo) sps = lo;
    if (sps > max_steps) sps = max_steps;
  }
  *steps_per_split = (int)sps;
  *key_groups = waves == 1 && n_groups == n_servers && sps >= kKeyGroupSteps && workgroups(sps) <= kKeyGroupItems ? kKeyGroups
                : waves == kGroupWaves && n_groups > n_servers && std::min(sps, max_steps) >= kPromptKeyGroupSteps ? kPromptKeyGroups
                                                                                                                   : 1;
  // the split count is also the stride (in 512-byte partial rows) between the partial results of
  // neighbouring (row, head) pairs: kept odd, because a power-of-two stride sends all partial stores of a
  // workgroup to the same few memory channels (measured: 110 instead of 81 us per layer at a stride of 32)
  *max_splits = (int)((max_steps + sps - 1) / sps) | 1;
}

size_t attention_workspace_floats(int n_rows, int n_heads, int hd, int max_splits) {
  return (size_t)n_rows * n_heads * max_splits * (hd + 2);
}

template <int HD, int G>
static gs_status launch_mfma_g(const bf16_t* q, const bf16_t* k_pages, const bf16_t* v_pages, const int* block_table,
                               int max_blocks, const int* work, int n_work, int page_size,
                               int n_heads, int n_kv, int waves, int key_groups, int steps_per_split, int max_splits,
                               float* po, float* pml, bf16_t* attn_out, bool packed, hipStream_t stream) {
  dim3 grid((unsigned)n_work * (unsigned)n_kv);      // one workgroup per (entry, KV head) item, see item_of_workgroup
#define GS_RING(NW_) GS_RINGS(NW_, 1)
#define GS_RINGS(NW_, KW_)                                                                                        \
  attn_kernel<HD, G, NW_, KW_><<<grid, 64 * NW_ * KW_, 0, stream>>>(q, k_pages, v_pages, block_table, max_blocks, work,      \
                                                         n_work, page_size, n_heads, n_kv, steps_per_split, max_splits,   \
                                                         po, pml, attn_out, packed)
  if (key_groups > 1) {
    if (waves == 1) GS_RINGS(1, kKeyGroups);
    else GS_RINGS(kGroupWaves, kPromptKeyGroups);
    GS_LAUNCH_CHECK("attn");
    return GS_OK;
  }
  switch (waves) {
    case 1: GS_RING(1); break;
    case 2: GS_RING(2); break;
    case 3: GS_RING(3); break;
    case 4: GS_RING(4); break;
    case 5: GS_RING(5); break;
    case 6: GS_RING(6); break;
    case 7: GS_RING(7); break;
    default: GS_RING(8); break;
  }
#undef GS_RING
#undef GS_RINGS
  GS_LAUNCH_CHECK("attn");
  return GS_OK;
}

// Number of ints of a work list with room for `capacity` entries.
size_t attention_work_ints(int capacity) { return 8 + 8 * (size_t)capacity; }

// attn_out [R][H*hd] (storage type).  max_keys: the most keys any row sees.  scratch: attention_workspace_floats floats; work, n_work: the step's work
// list and its length as the host computes it from its copy of the batch geometry (bf16 path only).  waves: per
// workgroup (attention_groups).  split: whether any group has more than one split.  packed: bf16 result in
// fragment order (packed_index).
gs_status launch_attention(int dtype, const void* q, const void* k_pages, const void* v_pages,
                           const int* block_table, int max_blocks, const int* cu_rows, const int* ctx_len,
                           int n_servers, int n_rows, int max_keys, int page_size, int n_heads, int n_kv, int hd,
                           int waves, int key_groups, int steps_per_split, int max_splits, bool split, const void* row_info,
                           const int* work, int n_work, float* scratch, void* attn_out, bool packed, hipStream_t stream) {
  if (dtype == GS_F32) {
    dim3 grid(n_rows, n_heads);
    const float* qf = static_cast<const float*>(q);
    const float* kf = static_cast<const float*>(k_pages);
    const float* vf = static_cast<const float*>(v_pages);
    float* of = static_cast<float*>(attn_out);
    const bool vec = page_size % 4 == 0 && reinterpret_cast<uintptr_t>(k_pages) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(v_pages) % 16 == 0;
    // Looking ahead: 4 layers of 4 heads of 64 over 2, whole call, us without and with: 64 rows on 8000 keys 1268 and 980, 128 rows
    // 1425 and 1243 (1356 with a lane per key); 8 heads over 1, 256 rows on 8000 keys 3073 and 3577.  Up to 32 keys
    // there is nothing to wait for (8 layers, 8 servers on 8 keys 208 and 211, on 32 the same, on 60 217 and 212).
    const bool ahead = vec && (long)n_rows * n_heads <= kRowAheadItems && max_keys > 32;
#define GS_ROWWISE(HD_, VEC_, AHEAD_)                                                                             \
  attn_rowwise_kernel<HD_, VEC_, AHEAD_><<<grid, kRowThreads, 0, stream>>>(qf, kf, vf, block_table, max_blocks,           \
                                                                   static_cast<const int4*>(row_info), cu_rows, ctx_len, \
                                                                   page_size, n_heads, n_kv, of)
    if (hd == 64 && ahead) GS_ROWWISE(64, true, true);
    else if (hd == 64 && vec) GS_ROWWISE(64, true, false);
    else if (hd == 64) GS_ROWWISE(64, false, false);
    else if (ahead) GS_ROWWISE(128, true, true);
    else if (vec) GS_ROWWISE(128, true, false);
    else GS_ROWWISE(128, false, false);
#undef GS_ROWWISE
    GS_LAUNCH_CHECK("attn_rowwise");
    return GS_OK;
  }
  const bf16_t* qb = static_cast<const bf16_t*>(q);
  const bf16_t* kb = static_cast<const bf16_t*>(k_pages);
  const bf16_t* vb = static_cast<const bf16_t*>(v_pages);
  float* po = scratch;
  float* pml = scratch + (size_t)n_rows * n_heads * max_splits * hd;
  const int G = n_heads / n_kv;
  gs_status st = GS_OK;
#define GS_ATTN_CASE(HD_, G_)                                                                                     \
  if (hd == HD_ && G == G_)                                                                                       \
    st = launch_mfma_g<HD_, G_>(qb, kb, vb, block_table, max_blocks, work, n_work, page_size, n_heads, n_kv,     \
                                waves, key_groups, steps_per_split, max_splits, po, pml, static_cast<bf16_t*>(attn_out),       \
                                packed, stream);
  GS_ATTN_CASE(128, 1) GS_ATTN_CASE(128, 2) GS_ATTN_CASE(128, 4) GS_ATTN_CASE(128, 8)
  GS_ATTN_CASE(64, 1) GS_ATTN_CASE(64, 2) GS_ATTN_CASE(64, 4) GS_ATTN_CASE(64, 8)
#undef GS_ATTN_CASE
  if (st != GS_OK || !split) return st;
  const unsigned combine_grid = (unsigned)ceil_div(n_rows * n_heads, kCombineThreads * 4 / hd);
  if (hd == 128)
    attn_combine_kernel<128><<<combine_grid, kCombineThreads, 0, stream>>>(po, pml, max_splits, steps_per_split,
                                                                           static_cast<const int4*>(row_info), n_rows, n_heads,
                                                                           static_cast<bf16_t*>(attn_out), packed);
  else
    attn_combine_kernel<64><<<combine_grid, kCombineThreads, 0, stream>>>(po, pml, max_splits, steps_per_split,
                                                                          static_cast<const int4*>(row_info), n_rows, n_heads,
                                                                          static_cast<bf16_t*>(attn_out), packed);
  GS_LAUNCH_CHECK("attn_combine");
  return GS_OK;
}

}  // namespace gs
