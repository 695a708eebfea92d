// bf16 attention forward of small layers: the eight waves of a block split
// the context of one 32-query item (fwd_bf16_kernel in attention_fwd.hip
// gives each wave 32 queries of a 256-query item instead and streams the
// whole context past all of them).
//
// A layer with few 256-query items leaves that kernel either few blocks or
// many short pieces whose fp32 records (133 KB each) cost more than the
// attention; here an item is 32 queries, its pieces meet in LDS, and only
// where even these items are few does a context span several blocks
// (FwdArgs::key_splits).  Each wave streams its own 32-key tiles through 16 KB
// of LDS by direct transfers and waits for nothing but them: no barrier until
// the merge.  K of the next tile is in flight during softmax and P V, V during
// the scores; two waves share a SIMD and cover each other's waits.  The price
// is K/V read once per 32 queries instead of once per 256, so the L2 bounds it
// and the dispatch (forward_choice in plan.cpp) keeps it to small layers.
// Measured, pass: 2 heads of 128 on a 10 x 13 grid 55.9 -> 18.3 us, 6 heads of
// 64 on 17 x 23 79.8 -> 24.9 us (25.8 with the scale applied to every score
// before the maximum and the mask on every tile).
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "lds_stage.hpp"
#include "split_merge.hpp"
#include "xcd.hpp"

namespace mssa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

constexpr int kTileBytes = 32 * 256;  // 32 keys in the swizzled 256-byte rows of lds_stage.hpp
constexpr int kXfers = kTileBytes / 1024;
constexpr float kRescaleLog2 = 8.0f;  // as in attention_fwd.hip: m raised only past this, P <= 2^8

// s_waitcnt vmcnt(N) that LDS reads are not moved across.
template <int N>
__device__ inline void wait_transfers() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// This wave's LDS reads have returned: their tile may be overwritten.
__device__ inline void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int D>
__global__ __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fwd_small_kernel(FwdArgs a) {
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int kTiles = kSplitWaves * 2 * kTileBytes, kMerge = split_lds_floats(D) * 4;
  __shared__ __attribute__((aligned(16))) char lds[kTiles > kMerge ? kTiles : kMerge];

  const int S = a.key_splits;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int item = L / S, sp = L % S;
  int g = 0, first = 0;  // first item of group g
  while (g + 1 < a.n_groups) {
    const int items = (a.groups[g].q_end - a.groups[g].q_begin + 31) / 32 * a.num_heads;
    if (item < first + items) break;
    first += items;
    ++g;
  }
  const FwdGroupArgs& G = a.groups[g];
  const int nqt = (G.q_end - G.q_begin + 31) / 32;
  const int head = (item - first) / nqt, q0 = G.q_begin + (item - first) % nqt * 32;
  const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t ld = a.ld, hoff = static_cast<int64_t>(head) * D;
  const uint32_t rb = static_cast<uint32_t>(ld) * 2;
  const float c = a.scale_log2e;

  // Tiles of this wave: t, t + 8, .. below t1, each inside one run.
  int nt = 0;
  for (int r = 0; r < G.n_runs; ++r) nt += (G.runs[r].n_tok + 31) / 32;
  const int t1 = static_cast<int>(static_cast<int64_t>(nt) * (sp + 1) / S);
  int t = static_cast<int>(static_cast<int64_t>(nt) * sp / S) + wave;
  int run = 0, idx = t;  // tile idx of run `run`
  auto settle = [&]() {
    while (run < G.n_runs && idx >= (G.runs[run].n_tok + 31) / 32) {
      idx -= (G.runs[run].n_tok + 31) / 32;
      ++run;
    }
  };

  // Transfer i fills rows 4 i .. 4 i + 3 of a tile: the lane's row is
  // 4 i + lane / 16, its logical chunk lane % 16 ^ 4 (lane / 16) ^ (i % 4).
  // Rows past the run's end and chunks past D arrive as zeros.
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds)) + wave * 2 * kTileBytes;
  const int lc0 = (lane & 15) ^ ((lane >> 4) << 2);
  const uint32_t off0 = (lane >> 4) * rb + lc0 * 16;
  auto issue = [&](const void* src, int nv, uint32_t dst) {
    const i32x4 rs = rsrc_of(src, static_cast<uint32_t>(nv - 1) * rb + D * 2);
#pragma unroll
    for (int i = 0; i < kXfers; ++i) {
      const uint32_t vo = D / 8 >= 16 || (lc0 ^ (i & 3)) < D / 8 ? (off0 ^ ((i & 3) * 16)) + i * 4 * rb : kPastEnd;
      dma16(rs, vo, __builtin_amdgcn_readfirstlane(dst + i * 1024));
    }
  };
  int nv = 0;
  const __bf16* vp = nullptr;
  auto issue_k = [&]() {  // K of the tile (run, idx); its V is issued later
    const FwdRunArgs& R = G.runs[run];
    nv = min(32, R.n_tok - idx * 32);
    const int64_t off = static_cast<int64_t>(idx) * 32 * ld + hoff;
    vp = static_cast<const __bf16*>(R.v) + off;
    issue(static_cast<const __bf16*>(R.k) + off, nv, lds0);
  };

  bf16x8 qf[KS];
  {
    const bool ok = q0 + n < G.q_end;
    const __bf16* qp = static_cast<const __bf16*>(a.q) + static_cast<int64_t>(ok ? q0 + n : q0) * ld + hoff + hh * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
      qf[ks] = ok ? v : bf16x8{};
    }
  }
  // complete before the first transfer, which the compiler does not count
  wait_transfers<0>();
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));

  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = f32x16{};
  float m = -INFINITY, l = 0.f;  // running max (base 2, both half-waves), this lane's share of the sum

  const __bf16* Ks = reinterpret_cast<const __bf16*>(lds + wave * 2 * kTileBytes);
  const __bf16* Vs = Ks + kTileBytes / 2;
  const int k_rd = swz256(n, hh * 8);
  const int t_row = 4 * (lane >> 5) + ((lane & 15) >> 2);
  const int t_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

  if (t < t1) {
    settle();
    issue_k();
    issue(vp, nv, lds0 + kTileBytes);
  }
  while (t < t1) {
    wait_transfers<kXfers>();  // K here, V may be on its way
    f32x16 s = f32x16{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(Ks + (k_rd ^ (ks * 16))), qf[ks], s, 0, 0, 0);
    wait_lds_reads();
    const int valid = nv;
    t += kSplitWaves;
    idx += kSplitWaves;
    const bool more = t < t1;
    if (more) {
      settle();
      issue_k();
    }
    if (valid < 32) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + 4 * hh + (e & 3) >= valid) s[e] = -INFINITY;
    }
    float mx = fmaxf(s[0], s[1]);
#pragma unroll
    for (int e = 2; e < 16; e += 2) mx = fmaxf(fmaxf(mx, s[e]), s[e + 1]);
    mx = fmaxf(mx, other_half(mx)) * c;  // the scale is positive
    if (__any(mx > m + kRescaleLog2 || (m == -INFINITY && mx > m))) {
      const float mn = fmaxf(m, mx);
      const float alpha = mn == m ? 1.f : __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] *= alpha;
    }
    const float ms = m == -INFINITY ? 0.f : m;
    bf16x8 pb[2];
    float ls[2] = {0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c, -ms));
      ls[e & 1] += p;
      pb[e >> 3][e & 7] = static_cast<__bf16>(p);
    }
    l += ls[0] + ls[1];
    if (more)
      wait_transfers<kXfers>();  // V here, the next K may be on its way
    else
      wait_transfers<0>();
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const __bf16* r0 = Vs + cc * 16 * 128;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(r0 + swz256(t_row, db * 32 + t_col)));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(r0 + swz256(t_row + 8, db * 32 + t_col)));
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7), pb[cc],
                                                        o[db], 0, 0, 0);
      }
    if (more) {
      wait_lds_reads();
      issue(vp, nv, lds0 + kTileBytes);
    }
  }
  l += other_half(l);
  __syncthreads();  // every wave's transfers have arrived and been read
  // channels 32 db + 8 j + 4 hh .. + 3 of query n: channel group 8 db + 2 j + hh
  float* O = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = o[db][4 * j + i];
      *reinterpret_cast<f32x4*>(O + wave * 32 * D + ((8 * db + 2 * j + hh) * 32 + n) * 4) = v;
    }
  split_stats(O, D, wave, lane, m, l);
  __syncthreads();
  merge_split<__bf16, D, 4>(a, O, item, sp, head, q0, G.q_end);
}

}  // namespace

hipError_t launch_forward_small(const FwdArgs& a, int head_dim, hipStream_t stream) {
  int64_t items = 0;
  for (int g = 0; g < a.n_groups; ++g)
    items += static_cast<int64_t>((a.groups[g].q_end - a.groups[g].q_begin + 31) / 32) * a.num_heads;
  const int64_t blocks = items * a.key_splits;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff || (a.key_splits > 1 && !a.partial)) return hipErrorInvalidValue;
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kSplitThreads);
  if (head_dim == 128)
    hipLaunchKernelGGL(fwd_small_kernel<128>, grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL(fwd_small_kernel<64>, grid, block, 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.key_splits == 1) return e;
  const dim3 cgrid(static_cast<uint32_t>(items));
  if (head_dim == 128)
    hipLaunchKernelGGL((combine_split_kernel<__bf16, 128, 4>), cgrid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((combine_split_kernel<__bf16, 64, 4>), cgrid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace mssa
