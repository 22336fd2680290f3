// The attention work list: its entries (read by attn_kernel) and its construction (once per step, step_begin_kernel).
#pragma once
#include <hip/hip_runtime.h>

namespace gs {
namespace {

// Work list of a step: one entry per (server, query group, split) that has keys, so that the grid holds no workgroup
// that starts only to find its split empty (ragged contexts), and an entry carries all a workgroup needs
// before its first load, the pages of its first step included: start-up costs one dependent read instead
// of three.  list = int header[8] (header[0] = number of entries), then the entries.
// A query group is `group_tokens` consecutive tokens of a block (its last group may be shorter); n_tokens is the
// number of block tokens up to the end of the group, so ctx + n_tokens is the number of keys the group sees.
struct AttnWork {
  int srv, split, row0, n_tokens, ctx, page0, page1, tok0;
};
static_assert(sizeof(AttnWork) == 32, "entries are read as one 32-byte load");

// Work of one workgroup of kWorkThreads lanes.  The entries are written in the order of decreasing split length (counting sort over the
// lengths, which the splits of a group take only two of), because the hardware deals the workgroups of a
// launch to the compute units round robin by their linear index and a compute unit's finishing time follows
// the sum of the steps it was dealt: attn_kernel walks the sorted list in a serpentine (item_of_workgroup),
// so every compute unit gets one long, one medium, ... split instead of whatever the server order brings.
// Splits of kSortBins - 1 steps and more share a bin (any order).  A server's (group, split) pairs are dealt to
// 1024 / n_servers lanes (a power of two, at least one): one prompt block of 64 groups fills the workgroup, with many
// servers a lane takes one each.  Entries beyond the capacity are
// dropped (cannot happen when the host's copy of the batch geometry matches the device's).
constexpr int kSortBins = 1024;
constexpr int kWorkThreads = 1024;

// shared: 2 * kSortBins ints.
__device__ __forceinline__ void build_attention_work(const int* __restrict__ cu_rows, const int* __restrict__ ctx_len,
                                                     int n_servers, const int* __restrict__ block_table,
                                                     int max_blocks, int page_size, int steps_per_split,
                                                     int group_tokens, int capacity, int* __restrict__ list,
                                                     int* shared) {
  int* bin = shared;                  // entries per split length, then the next position of a length
  int* scan = shared + kSortBins;
  const int tid = threadIdx.x;
  int lanes = 1;                      // per server
  while (lanes * 2 * n_servers <= kWorkThreads) lanes *= 2;
  const int per_pass = kWorkThreads / lanes, sub = tid & (lanes - 1);
  bin[tid] = 0;
  __syncthreads();
  // f(row0, L, first token, block tokens up to the group's end, split, splits of the group, steps of the group)
  auto for_each_split = [&](int srv, auto f) {
    const int row0 = cu_rows[srv], T = cu_rows[srv + 1] - row0, L = ctx_len[srv];
    const int n_groups = (T + group_tokens - 1) / group_tokens;
    const int most = (((L + T + 31) >> 5) + steps_per_split - 1) / steps_per_split;      // splits of the last group
    for (int e = sub; e < n_groups * most; e += lanes) {
      const int g = e / most, sp = e - g * most;
      const int t_end = min(T, (g + 1) * group_tokens);
      const int steps = (L + t_end + 31) >> 5, count = (steps + steps_per_split - 1) / steps_per_split;
      if (sp < count) f(row0, L, g * group_tokens, t_end, sp, count, steps);
    }
  };
  // the steps of a group are dealt evenly to its splits: `rem` of base + 1 followed by count - rem of base steps
  auto bin_of = [&](int sp, int count, int steps) {
    const int base = steps / count, rem = steps - base * count;
    return kSortBins - 1 - min(kSortBins - 1, base + (sp < rem ? 1 : 0));      // longest first
  };
  for (int srv = tid / lanes; srv < n_servers; srv += per_pass)
    for_each_split(srv, [&](int, int, int, int, int sp, int count, int steps) { atomicAdd(&bin[bin_of(sp, count, steps)], 1); });
  __syncthreads();
  const int mine = bin[tid];
  scan[tid] = mine;
  __syncthreads();
  for (int off = 1; off < kSortBins; off <<= 1) {
    const int v = tid >= off ? scan[tid - off] : 0;
    __syncthreads();
    scan[tid] += v;
    __syncthreads();
  }
  bin[tid] = scan[tid] - mine;
  const int total = scan[kSortBins - 1];
  __syncthreads();
  AttnWork* entries = reinterpret_cast<AttnWork*>(list + 8);
  for (int srv = tid / lanes; srv < n_servers; srv += per_pass)
    for_each_split(srv, [&](int row0, int L, int tok0, int t_end, int sp, int count, int steps) {
      const int pos = atomicAdd(&bin[bin_of(sp, count, steps)], 1);
      if (pos >= capacity) return;
      const int base = steps / count, rem = steps - base * count;
      const int last_tile_key = ((L + t_end - 1) >> 4) << 4;
      const int key0 = min((sp * base + min(sp, rem)) * 32, last_tile_key), key1 = min(key0 + 16, last_tile_key);
      AttnWork w;
      w.srv = srv; w.split = sp; w.row0 = row0; w.n_tokens = t_end; w.ctx = L; w.tok0 = tok0;
      w.page0 = block_table[(size_t)srv * max_blocks + key0 / page_size];
      w.page1 = block_table[(size_t)srv * max_blocks + key1 / page_size];
      entries[pos] = w;
    });
  if (tid == 0) list[0] = min(total, capacity);
}
static_assert(kSortBins == kWorkThreads, "one lane per bin");

}  // namespace
}  // namespace gs
