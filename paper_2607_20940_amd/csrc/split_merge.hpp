// Merge of attention pieces for the kernels whose eight waves split the
// context of one 32-query item (attention_f32.hip, attention_fwd_small.hip).
// Each wave ends with an unnormalised output O (fp32), the running max m and
// the row sum l of the keys it saw; the waves meet in LDS, and when the
// context is also split over blocks (FwdArgs::key_splits > 1) each block's
// sum is a record in the workspace that combine_split_kernel merges.  Fixed
// orders (wave 0 first, split 0 first): the same bits on every run.
//
// Layout of O in LDS and in a record: V consecutive channels of one query are
// neighbours, the queries of one channel group next to each other: element
// (channel V i + j, query q) at (i * 32 + q) * V + j.
#pragma once

#include <hip/hip_runtime.h>

#include "kernel_args.hpp"

namespace mssa {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS of the merge: the waves' O, then m and l of every wave's 32 queries.
constexpr int split_lds_floats(int head_dim) { return kSplitWaves * 32 * (head_dim + 2); }

__device__ inline void split_stats(float* lds, int head_dim, int wave, int lane, float m, float l) {
  float* st = lds + kSplitWaves * 32 * head_dim + wave * 64;
  if (lane < 32) {
    st[lane] = m;
    st[32 + lane] = l;
  }
}

template <class T>
__device__ inline float split_exp(float x);  // the kernel's exponential: natural (fp32 plans) or base 2
template <>
__device__ inline float split_exp<float>(float x) { return expf(x); }
template <>
__device__ inline float split_exp<__bf16>(float x) { return __builtin_amdgcn_exp2f(x); }

// m + log l in natural units.
template <class T>
__device__ inline float split_lse(float m, float l);
template <>
__device__ inline float split_lse<float>(float m, float l) { return m + logf(l); }
template <>
__device__ inline float split_lse<__bf16>(float m, float l) { return (m + log2f(l)) * 0.6931471805599453f; }

// Weight of a piece (max m, sum l) in a sum with max mt.  A piece without
// keys, or whose scores are all -inf, has m = -inf and l = 0 and weighs 0
// whatever mt; l = NaN (a NaN score) stays.
template <class T>
__device__ inline float split_weight(float m, float l, float mt) {
  return m == -INFINITY ? l * 0.f : split_exp<T>(m - mt);
}

template <class T, int V>
__device__ inline void store_out(T* p, const float* x) {
  typedef T vecT __attribute__((ext_vector_type(V)));
  vecT v;
#pragma unroll
  for (int j = 0; j < V; ++j) v[j] = static_cast<T>(x[j]);
  *reinterpret_cast<vecT*>(p) = v;
}

// The block's waves -> the output (key_splits == 1) or record item * S + sp.
template <class T, int D, int V>
__device__ inline void merge_split(const FwdArgs& a, const float* lds, int item, int sp, int head, int q0, int q_end) {
  typedef float vec __attribute__((ext_vector_type(V)));
  const float* st = lds + kSplitWaves * 32 * D;
  const int q = threadIdx.x & 31;
  float mt = -INFINITY, lt = 0.f, w[kSplitWaves];
#pragma unroll
  for (int i = 0; i < kSplitWaves; ++i) mt = fmaxf(mt, st[i * 64 + q]);
#pragma unroll
  for (int i = 0; i < kSplitWaves; ++i) {
    w[i] = split_weight<T>(st[i * 64 + q], st[i * 64 + 32 + q], mt);
    lt += w[i] * st[i * 64 + 32 + q];
  }
  const bool whole = a.key_splits == 1;
  float* rec = whole ? nullptr : a.partial + (static_cast<int64_t>(item) * a.key_splits + sp) * split_record_floats(D);
  const float inv = 1.0f / lt;
  if (threadIdx.x < 32) {
    if (!whole) {
      rec[32 * D + q] = mt;
      rec[32 * D + 32 + q] = lt;
    } else if (a.lse && q0 + q < q_end) {
      a.lse[static_cast<int64_t>(head) * a.n_q + q0 + q] = split_lse<T>(mt, lt);
    }
  }
#pragma unroll
  for (int i0 = 0; i0 < 32 * D / V; i0 += kSplitThreads) {
    const int i = i0 + threadIdx.x;  // kSplitThreads is a multiple of 32: the query stays q
    vec s = vec{};
#pragma unroll
    for (int k = 0; k < kSplitWaves; ++k) s += w[k] * *reinterpret_cast<const vec*>(lds + k * 32 * D + i * V);
    if (!whole) {
      *reinterpret_cast<vec*>(rec + i * V) = s;
    } else if (q0 + q < q_end) {
      float x[V];
#pragma unroll
      for (int j = 0; j < V; ++j) x[j] = s[j] * inv;
      store_out<T, V>(static_cast<T*>(a.out) + static_cast<int64_t>(q0 + q) * a.ld + static_cast<int64_t>(head) * D +
                          (i >> 5) * V, x);
    }
  }
}

// One block per item: its key_splits records, split 0 first.
template <class T, int D, int V>
__global__ __launch_bounds__(kSplitThreads) void combine_split_kernel(FwdArgs a) {
  typedef float vec __attribute__((ext_vector_type(V)));
  const int item = blockIdx.x, S = a.key_splits;
  int g = 0, first = 0;  // first item of group g
  while (g + 1 < a.n_groups) {
    const int items = (a.groups[g].q_end - a.groups[g].q_begin + 31) / 32 * a.num_heads;
    if (item < first + items) break;
    first += items;
    ++g;
  }
  const FwdGroupArgs& G = a.groups[g];
  const int nt = (G.q_end - G.q_begin + 31) / 32;
  const int head = (item - first) / nt, q0 = G.q_begin + (item - first) % nt * 32;
  const int q = threadIdx.x & 31;
  const float* rec = a.partial + static_cast<int64_t>(item) * S * split_record_floats(D);
  float mt = -INFINITY, lt = 0.f;
  for (int s = 0; s < S; ++s) mt = fmaxf(mt, rec[s * split_record_floats(D) + 32 * D + q]);
  vec acc[32 * D / V / kSplitThreads];
#pragma unroll
  for (int i = 0; i < 32 * D / V / kSplitThreads; ++i) acc[i] = vec{};
  for (int s = 0; s < S; ++s) {
    const float* r = rec + s * split_record_floats(D);
    const float w = split_weight<T>(r[32 * D + q], r[32 * D + 32 + q], mt);
    lt += w * r[32 * D + 32 + q];
#pragma unroll
    for (int i = 0; i < 32 * D / V / kSplitThreads; ++i)
      acc[i] += w * *reinterpret_cast<const vec*>(r + (i * kSplitThreads + threadIdx.x) * V);
  }
  if (q0 + q >= G.q_end) return;
  const float inv = 1.0f / lt;
  if (a.lse && threadIdx.x < 32) a.lse[static_cast<int64_t>(head) * a.n_q + q0 + q] = split_lse<T>(mt, lt);
#pragma unroll
  for (int i = 0; i < 32 * D / V / kSplitThreads; ++i) {
    float x[V];
#pragma unroll
    for (int j = 0; j < V; ++j) x[j] = acc[i][j] * inv;
    store_out<T, V>(static_cast<T*>(a.out) + static_cast<int64_t>(q0 + q) * a.ld + static_cast<int64_t>(head) * D +
                        ((i * kSplitThreads + threadIdx.x) >> 5) * V, x);
  }
}

}  // namespace mssa
