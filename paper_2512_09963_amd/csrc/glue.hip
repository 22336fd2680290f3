// Row-wise kernels between the projections of the decoder: embedding gather,
// residual add + RMSNorm (also sums the split-K partials of the preceding projection),
// rotary embedding + KV-page append, SwiGLU.  All arithmetic is fp32; T is the storage
// type of the tensors fed to the next projection and of the KV pages (float or bf16).
#include "common.h"
#include "attn_work.h"
#include "device_types.h"
#include "gemm_common.h"

namespace gs {
namespace {

// Sum over the workgroup (any multiple of 64 threads up to 1024), fixed order.
__device__ __forceinline__ float block_sum(float v, float* sh /*[16]*/) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
  const int n_waves = blockDim.x >> 6;
  for (int w = 0; w < n_waves; ++w) t += sh[w];
  __syncthreads();
  return t;
}

// server that owns target row r: largest i with cu_rows[i] <= r
__device__ __forceinline__ int server_of_row(const int* __restrict__ cu_rows, int n_servers, int r) {
  int lo = 0, hi = n_servers;   // invariant: cu_rows[lo] <= r < cu_rows[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (cu_rows[mid] <= r) lo = mid; else hi = mid;
  }
  return lo;
}

// x[r] += sum_s partial[s][r] (if partial), then h[r] = x[r] * w / sqrt(mean(x[r]^2) + eps).
// One workgroup per row, one float4 per lane and pass; the loads of the S partials are
// independent, so they are issued back to back (d % 4 == 0).  The first two passes of a row (all of it for
// d <= 8192 at 1024 lanes) stay in registers between the sum of squares and the scaling, and the norm
// weights are fetched before the reduction, so the second phase touches no memory but its stores.
template <typename T>
__global__ __launch_bounds__(1024) void add_rmsnorm_kernel(float* __restrict__ x, const float* __restrict__ partial,
                                                           int n_splits, int n_rows, const float* __restrict__ w,
                                                           float eps, T* __restrict__ h, int d) {
  __shared__ float sh[16];
  const int r = blockIdx.x;
  float4* xr = reinterpret_cast<float4*>(x + (size_t)r * d);
  const int d4 = d >> 2;
  const size_t split_stride = (size_t)n_rows * d4;
  const float4* pr = reinterpret_cast<const float4*>(partial) + (size_t)r * d4;
  const float4* wr = reinterpret_cast<const float4*>(w);
  // element i of the row with the partial sums added (and stored back to the residual stream)
  auto fetch = [&](int i) {
    float4 v = xr[i];
    if (partial) {
      float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = a0;
      int s = 0;
      for (; s + 4 <= n_splits; s += 4) {
        const float4 p0 = pr[(size_t)s * split_stride + i], p1 = pr[(size_t)(s + 1) * split_stride + i];
        const float4 p2 = pr[(size_t)(s + 2) * split_stride + i], p3 = pr[(size_t)(s + 3) * split_stride + i];
        a0.x += p0.x + p1.x; a0.y += p0.y + p1.y; a0.z += p0.z + p1.z; a0.w += p0.w + p1.w;
        a1.x += p2.x + p3.x; a1.y += p2.y + p3.y; a1.z += p2.z + p3.z; a1.w += p2.w + p3.w;
      }
      for (; s < n_splits; ++s) {
        const float4 p0 = pr[(size_t)s * split_stride + i];
        a0.x += p0.x; a0.y += p0.y; a0.z += p0.z; a0.w += p0.w;
      }
      v.x += a0.x + a1.x; v.y += a0.y + a1.y; v.z += a0.z + a1.z; v.w += a0.w + a1.w;
      xr[i] = v;
    }
    return v;
  };
  auto squares = [](const float4& v) { return (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w); };
  auto emit = [&](int i, const float4& v, const float4& ww, float inv) {
    T* dst = h + (size_t)r * d + 4 * i;
    Storage<T>::store(dst + 0, v.x * inv * ww.x);
    Storage<T>::store(dst + 1, v.y * inv * ww.y);
    Storage<T>::store(dst + 2, v.z * inv * ww.z);
    Storage<T>::store(dst + 3, v.w * inv * ww.w);
  };
  const int bd = blockDim.x;
  const int i0 = threadIdx.x, i1 = threadIdx.x + bd;
  const bool has0 = i0 < d4, has1 = i1 < d4;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 v0 = zero, v1 = zero, w0 = zero, w1 = zero;
  float ss = 0.f;
  if (has0) {
    w0 = wr[i0];
    v0 = fetch(i0);
    ss += squares(v0);
  }
  if (has1) {
    w1 = wr[i1];
    v1 = fetch(i1);
    ss += squares(v1);
  }
  for (int i = i1 + bd; i < d4; i += bd) ss += squares(fetch(i));     // rows wider than two passes
  const float tot = block_sum(ss, sh);
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
  if (has0) emit(i0, v0, w0, inv);
  if (has1) emit(i1, v1, w1, inv);
  for (int i = i1 + bd; i < d4; i += bd) emit(i, xr[i], wr[i], inv);
}

// Everything of a step that precedes the first projection, in one launch (five dependent-looking launches of 3 to 17 us
// otherwise: 27 us of a 53-row step, 6 now; the roles are independent of each other).  Workgroups by index:
//   [0, R)       embedding row r into the residual stream (storage type -> fp32, 4 elements per lane and pass) and its
//                first RMSNorm h[r] = x[r] * w / sqrt(mean(x[r]^2) + eps), or x[r] * w and the row's sum of squares
//   [R, 2 R)     per-row facts that every layer shares: where the row's K/V go (page, slot), how many keys its attention
//                query group (group_tokens consecutive tokens of the block) sees, and the rotary sine/cosine of its
//                position, rope [R][hd/2] (cos, sin).  The angle pos * theta^(-2i/hd) reaches thousands of radians: it
//                is formed in double, so that the rotated values agree with a float64 evaluation to fp32 rounding.
//                Also draft_tokens[cu_rows[i] - i + j] = tokens[cu_rows[i] + 1 + j]: the drafts without the pending tokens.
//   2 R          the attention work list (bf16 models: the grid has this workgroup only then)
struct StepBegin {
  const void* embed;
  const int* tokens;
  float* x;
  const float* norm;
  void* h;
  const int* cu_rows;
  const int* ctx_len;
  const int* block_table;
  int4* row_slot;
  float2* rope;
  int* draft_tokens;
  int* attn_work;
  float* squares;      // or null: h complete
  double log2_theta;
  float eps;
  int n_rows, d, vocab, n_servers, max_blocks, page_size, hd, group_tokens, steps_per_split, work_capacity;
};

template <typename T>
__global__ __launch_bounds__(kWorkThreads) void step_begin_kernel(StepBegin a) {
  __shared__ int shared[2 * kSortBins];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < a.n_rows) {
    const int r = blockIdx.x;
    const int tok = min(max(a.tokens[r], 0), a.vocab - 1);      // an id outside the vocabulary is never used as an index
    const T* src = static_cast<const T*>(a.embed) + (size_t)tok * a.d;
    float4* xr = reinterpret_cast<float4*>(a.x + (size_t)r * a.d);
    const float4* wr = reinterpret_cast<const float4*>(a.norm);
    T* hr = static_cast<T*>(a.h) + (size_t)r * a.d;
    const int d4 = a.d >> 2;
    float ss = 0.f;
    float4 v0 = make_float4(0.f, 0.f, 0.f, 0.f), w0 = v0;      // the first pass stays in registers (all of a row to d = 4096)
    for (int i = tid; i < d4; i += kWorkThreads) {
      const float4 v = make_float4(Storage<T>::load(src + 4 * i), Storage<T>::load(src + 4 * i + 1),
                                   Storage<T>::load(src + 4 * i + 2), Storage<T>::load(src + 4 * i + 3));
      if (i == tid) {
        w0 = wr[i];
        v0 = v;
      }
      xr[i] = v;
      ss += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    }
    const float tot = block_sum(ss, reinterpret_cast<float*>(shared));
    float inv = 1.0f / sqrtf(tot / (float)a.d + a.eps);
    if (a.squares) {      // the row's factor is left to the projection that reads h (RowNorm)
      inv = 1.0f;
      for (int i = tid; i < a.d >> 4; i += kWorkThreads) a.squares[(size_t)r * (a.d >> 4) + i] = i == 0 ? tot : 0.f;
    }
    const bool packed = a.squares && sizeof(T) == 2;      // (bf16 rows in fragment order)
    for (int i = tid; i < d4; i += kWorkThreads) {
      const float4 v = i == tid ? v0 : xr[i], w = i == tid ? w0 : wr[i];
      T* dst = packed ? static_cast<T*>(a.h) + packed_index(r, 4 * i, a.d) : hr + 4 * i;
      Storage<T>::store(dst + 0, v.x * inv * w.x);
      Storage<T>::store(dst + 1, v.y * inv * w.y);
      Storage<T>::store(dst + 2, v.z * inv * w.z);
      Storage<T>::store(dst + 3, v.w * inv * w.w);
    }
  } else if ((int)blockIdx.x < 2 * a.n_rows) {
    if (tid >= 64) return;
    const int r = blockIdx.x - a.n_rows;
    const int srv = server_of_row(a.cu_rows, a.n_servers, r);
    const int row0 = a.cu_rows[srv], j = r - row0, pos = a.ctx_len[srv] + j;
    if (tid == 0) {
      a.row_slot[r] = make_int4(a.block_table[(size_t)srv * a.max_blocks + pos / a.page_size], pos % a.page_size,
                                a.ctx_len[srv] + min(a.cu_rows[srv + 1] - row0, (j / a.group_tokens + 1) * a.group_tokens),
                                srv);
      if (j > 0) a.draft_tokens[r - srv - 1] = a.tokens[r];
    }
    for (int i = tid; i < (a.hd >> 1); i += 64) {
      const double inv_freq = exp2(-2.0 * (double)i / (double)a.hd * a.log2_theta);
      double sn, cs;
      sincos((double)pos * inv_freq, &sn, &cs);
      a.rope[(size_t)r * (a.hd >> 1) + i] = make_float2((float)cs, (float)sn);
    }
  } else {
    build_attention_work(a.cu_rows, a.ctx_len, a.n_servers, a.block_table, a.max_blocks, a.page_size, a.steps_per_split,
                         a.group_tokens, a.work_capacity, a.attn_work, shared);
  }
}

// Sums the QKV partials and hands the element pair (i, i + hd/2) of a head to store_qkv_pair.
// grid (R, (H + 2 H_kv) * hd/2 / 256): a thread owns one pair.
template <typename T>
__global__ __launch_bounds__(256) void rope_append_kernel(const float* __restrict__ qkv, int n_splits, int n_rows, QkvOut out) {
  const int r = blockIdx.x;
  const int half = out.hd >> 1;
  const int item = blockIdx.y * 256 + threadIdx.x;
  const int head = item / half, i = item - head * half;
  if (head >= out.n_heads + 2 * out.n_kv) return;
  const int width = (out.n_heads + 2 * out.n_kv) * out.hd;
  const size_t split_stride = (size_t)n_rows * width;
  const float* src = qkv + (size_t)r * width + head * out.hd + i;
  float a = 0.f, b = 0.f;
  for (int s = 0; s < n_splits; ++s) {
    a += src[(size_t)s * split_stride];
    b += src[(size_t)s * split_stride + half];
  }
  const bool rotated = head < out.n_heads + out.n_kv;
  store_qkv_pair<T>(out, r, head, i, a, b, out.row_slot[r], rotated ? out.rope[(size_t)r * half + i] : make_float2(1.f, 0.f));
}

// act[r][f] = silu(gate) * up with gate = sum_s gu[s][r][f], up = sum_s gu[s][r][F + f].
// VEC: four features per lane (F % 4 == 0).
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void swiglu_kernel(const float* __restrict__ gu, int n_splits, int n_rows, int F,
                                                     T* __restrict__ act) {
  constexpr int W = VEC ? 4 : 1;
  const size_t idx = ((size_t)blockIdx.x * 256 + threadIdx.x) * W;
  if (idx >= (size_t)n_rows * F) return;
  const int r = (int)(idx / F), f = (int)(idx - (size_t)r * F);
  float gt[W], up[W];
#pragma unroll
  for (int k = 0; k < W; ++k) gt[k] = up[k] = 0.f;
  for (int s = 0; s < n_splits; ++s) {
    const float* row = gu + ((size_t)s * n_rows + r) * 2 * F;
    if constexpr (VEC) {
      const float4 g4 = *reinterpret_cast<const float4*>(row + f);
      const float4 u4 = *reinterpret_cast<const float4*>(row + F + f);
      gt[0] += g4.x; gt[1] += g4.y; gt[2] += g4.z; gt[3] += g4.w;
      up[0] += u4.x; up[1] += u4.y; up[2] += u4.z; up[3] += u4.w;
    } else {
      gt[0] += row[f];
      up[0] += row[F + f];
    }
  }
#pragma unroll
  for (int k = 0; k < W; ++k) Storage<T>::store(act + idx + k, gt[k] / (1.0f + expf(-gt[k])) * up[k]);
}

}  // namespace

#define GS_DISPATCH_T(dtype, ...)                 \
  if ((dtype) == GS_BF16) {                       \
    using T = bf16_t;                             \
    __VA_ARGS__                                   \
  } else {                                        \
    using T = float;                              \
    __VA_ARGS__                                   \
  }

// work_list: whether the step's attention needs its work list (bf16 models).
gs_status launch_step_begin(int dtype, const void* embed, const int* tokens, float* x, const float* norm, float eps, void* h,
                            int n_rows, int d, int vocab, const int* cu_rows, const int* ctx_len, int n_servers,
                            const int* block_table, int max_blocks, int page_size, int hd, float rope_theta,
                            int group_tokens, int steps_per_split, int work_capacity, bool work_list, void* row_slot,
                            void* rope, int* draft_tokens, int* attn_work, float* squares, hipStream_t stream) {
  const StepBegin a{embed, tokens, x, norm, h, cu_rows, ctx_len, block_table, static_cast<int4*>(row_slot),
                    static_cast<float2*>(rope), draft_tokens, attn_work, squares, log2((double)rope_theta), eps, n_rows, d, vocab,
                    n_servers, max_blocks, page_size, hd, group_tokens, steps_per_split, work_capacity};
  const unsigned grid = 2u * (unsigned)n_rows + (work_list ? 1u : 0u);
  GS_DISPATCH_T(dtype, step_begin_kernel<T><<<grid, kWorkThreads, 0, stream>>>(a);)
  GS_LAUNCH_CHECK("step_begin");
  return GS_OK;
}

gs_status launch_add_rmsnorm(int dtype, float* x, const float* partial, int n_splits, int n_rows, const float* w,
                             float eps, void* h, int d, hipStream_t stream) {
  int threads = ceil_div(d / 4, 64) * 64;
  if (threads > 1024) threads = 1024;
  GS_DISPATCH_T(dtype, add_rmsnorm_kernel<T><<<n_rows, threads, 0, stream>>>(x, partial, n_splits, n_rows, w, eps,
                                                                            static_cast<T*>(h), d);)
  GS_LAUNCH_CHECK("add_rmsnorm");
  return GS_OK;
}

gs_status launch_rope_append(int dtype, const float* qkv, int n_splits, int n_rows, const QkvOut& out, hipStream_t stream) {
  const dim3 grid(n_rows, ceil_div((out.n_heads + 2 * out.n_kv) * (out.hd / 2), 256));
  GS_DISPATCH_T(dtype, rope_append_kernel<T><<<grid, 256, 0, stream>>>(qkv, n_splits, n_rows, out);)
  GS_LAUNCH_CHECK("rope_append");
  return GS_OK;
}

gs_status launch_swiglu(int dtype, const float* gu, int n_splits, int n_rows, int F, void* act, hipStream_t stream) {
  const size_t total = (size_t)n_rows * F;
  if (F % 4 == 0) {
    const int blocks = (int)((total / 4 + 255) / 256);
    GS_DISPATCH_T(dtype, swiglu_kernel<T, true><<<blocks, 256, 0, stream>>>(gu, n_splits, n_rows, F, static_cast<T*>(act));)
  } else {
    const int blocks = (int)((total + 255) / 256);
    GS_DISPATCH_T(dtype, swiglu_kernel<T, false><<<blocks, 256, 0, stream>>>(gu, n_splits, n_rows, F, static_cast<T*>(act));)
  }
  GS_LAUNCH_CHECK("swiglu");
  return GS_OK;
}

}  // namespace gs
