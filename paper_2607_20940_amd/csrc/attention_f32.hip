// Multi-scale self-attention of fp32 plans, forward and backward, on the fp32
// matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums).
//
// Every block takes 32 rows of one operand (32 queries of one head: forward
// and dQ; 32 context keys: dK, dV) and its eight waves take turns over the
// 32-row tiles of the other one, each wave with accumulators of its own that
// meet in LDS at the end, in wave order.  A product of two row-major operands
// X Y^T has its A operand from rows of X (lane = row, 16 bytes of every 32;
// the two half-waves next to each other) and its B operand from rows of Y
// held in LDS; its result leaves lane n the column n.  That result, after the
// exponential, is the B operand of the accumulating product as it stands: 16
// pairs of rows, one MFMA each, whose A operand is a row of the other tensor
// read as it lies (32 lanes x 16 bytes).  So nothing is transposed and only
// the block's own rows pass through LDS.
//
// Bound: the matrix cores (64 cycles per MFMA of 4096 operations, 157 TFLOP/s)
// and, for the small layers fp32 plans are used on, the number of blocks: the
// forward splits the context of an item over key_splits blocks when the items
// alone leave CUs idle (merged by combine_split_kernel), and the backward runs
// its two kinds of blocks in one launch.
// Measured (2 heads of 128, 1095 queries, 725 and 1485 keys; 1.4 GFLOP
// forward): forward 30 + 5 us, dQ + dK/dV 90 us; with one lane per query or
// key and plain FMAs 4.1 ms and 9.5 ms.  Errors against 64 bits are smaller
// (6.0e-7 after 9.6e-7: shorter chains of sums).
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "split_merge.hpp"
#include "xcd.hpp"

namespace mssa {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWaves = kSplitWaves;

// Row of element e of a 32x32 accumulator in half-wave hh.
__device__ inline int acc_row(int e, int hh) { return 8 * (e >> 2) + 4 * hh + (e & 3); }

// One 32-row tile of a run: rows [base, base + 32 ld), nv of them valid.
struct Tile {
  const float *k, *v;
  int nv;
};

__device__ inline Tile tile_at(const FwdRunArgs* runs, int64_t ld, int64_t hoff, int t) {
  int r = 0;
  while (t >= (runs[r].n_tok + 31) / 32) {
    t -= (runs[r].n_tok + 31) / 32;
    ++r;
  }
  const int64_t off = static_cast<int64_t>(t) * 32 * ld + hoff;
  return {static_cast<const float*>(runs[r].k) + off, static_cast<const float*>(runs[r].v) + off,
          min(32, runs[r].n_tok - t * 32)};
}

__device__ inline int run_tiles(const FwdRunArgs* runs, int n_runs) {
  int t = 0;
  for (int r = 0; r < n_runs; ++r) t += (runs[r].n_tok + 31) / 32;
  return t;
}

// Rows [0, nv) of a 32-row tile as a buffer: loads past them are zeros.
__device__ inline __amdgpu_buffer_rsrc_t tile_buffer(const float* p, int64_t ld, int nv, int D) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, static_cast<int>(((nv - 1) * ld + D) * 4), 0x00020000);
}

// Operands stream from memory in batches of kBatch vectors, two
// batches in registers: the next one is in flight during the 16 MFMAs (1024
// cycles) of the current one.  prefetch() starts the first batch; the caller
// places it before the work that precedes the product.  Whole tiles in
// registers (64 + 64 beside the accumulators) spilled; like this the backward
// for head_dim 128 alone does, five registers.
constexpr int kBatch = 4;

// A operand of a row product: lane's row l % 32, 16 bytes at 8 j + 4 hh.
template <int D>
struct Rows {
  static constexpr int N = D / 8;
  __amdgpu_buffer_rsrc_t buf;
  uint32_t off;
  f32x4 x[2][kBatch];
  __device__ inline void fetch(int b) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
      x[b & 1][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, off + (b * kBatch + i) * 32, 0, 0));
  }
  __device__ inline void prefetch(const float* p, int64_t ld, int nv, int n, int hh) {
    buf = tile_buffer(p, ld, nv, D);
    off = (n * static_cast<uint32_t>(ld) + 4 * hh) * 4;
    fetch(0);
  }
};

// A operand of an accumulating product: for accumulator element e, the row
// acc_row(e, hh), D / 32 consecutive columns per lane.
template <int D>
struct Cols {
  typedef float vec __attribute__((ext_vector_type(D / 32)));
  __amdgpu_buffer_rsrc_t buf;
  uint32_t off, rb;  // lane's first row (4 hh) and columns; bytes per row
  vec x[2][kBatch];
  __device__ inline void fetch(int b) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const uint32_t o = off + (8 * b + i) * rb;  // element 4 b + i: row 8 b + 4 hh + i
      if constexpr (D == 128)
        x[b & 1][i] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(buf, o, 0, 0));
      else
        x[b & 1][i] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(buf, o, 0, 0));
    }
  }
  __device__ inline void prefetch(const float* p, int64_t ld, int nv, int n, int hh) {
    buf = tile_buffer(p, ld, nv, D);
    rb = static_cast<uint32_t>(ld) * 4;
    off = 4 * hh * rb + (D / 32) * 4 * n;
    fetch(0);
  }
};
static_assert(kBatch == 4, "a batch of Cols is one group of four accumulator elements");

// LDS copy of a block's 32 rows: rows of D + 4 floats, so that the 16-byte
// reads of 16 consecutive rows fall in distinct banks.
template <int D>
constexpr int kRowStr = D + 4;

template <int D>
__device__ inline void stage_row(float* dst, int i, const float* row) {  // i: 16-byte piece of the 32 rows
  const int r = i / (D / 4), c = i % (D / 4);
  *reinterpret_cast<f32x4*>(dst + r * kRowStr<D> + 4 * c) =
      row ? *reinterpret_cast<const f32x4*>(row + 4 * c) : f32x4{};
}

// X Y^T: A from the stream, B from the LDS rows of Y.
template <int D>
__device__ inline f32x16 row_product(Rows<D>& a, const float* y, int n, int hh) {
  f32x16 s = f32x16{};
  const float* b = y + n * kRowStr<D> + 4 * hh;
#pragma unroll
  for (int t = 0; t < Rows<D>::N / kBatch; ++t) {
    if (t + 1 < Rows<D>::N / kBatch) a.fetch(t + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const f32x4 bv = *reinterpret_cast<const f32x4*>(b + 8 * (t * kBatch + j));
#pragma unroll
      for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x[t & 1][j][i], bv[i], s, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return s;
}

template <int D>
__device__ inline void acc_product(f32x16 (&acc)[D / 32], Cols<D>& a, const f32x16& w) {
#pragma unroll
  for (int t = 0; t < 16 / kBatch; ++t) {
    if (t + 1 < 16 / kBatch) a.fetch(t + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x[t & 1][i][db], w[t * kBatch + i], acc[db], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// acc element (db, e) is column (D / 32) acc_row(e, hh) + db of row n: the
// D / 32 elements of one e are neighbours, stored at (acc_row * 32 + n).
template <int D>
__device__ inline void acc_to_lds(float* dst, const f32x16 (&acc)[D / 32], int n, int hh) {
  typedef float vec __attribute__((ext_vector_type(D / 32)));
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    vec v;
#pragma unroll
    for (int db = 0; db < D / 32; ++db) v[db] = acc[db][e];
    *reinterpret_cast<vec*>(dst + (acc_row(e, hh) * 32 + n) * (D / 32)) = v;
  }
}

// ------------------------------------------------------------------ forward

template <int D>
__global__ __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fwd_f32_kernel(FwdArgs a) {
  __shared__ __attribute__((aligned(16))) float lds[split_lds_floats(D)];
  const int S = a.key_splits;
  const int L = xcd_remap(blockIdx.x, a.n_blocks * S);
  const int item = L / S, sp = L % S;
  int g = 0;
  while (g + 1 < a.n_groups && item >= a.groups[g + 1].block_begin) ++g;
  const FwdGroupArgs& G = a.groups[g];
  const int head = (item - G.block_begin) / G.n_qtiles, qt = (item - G.block_begin) % G.n_qtiles;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q0 = G.q_begin + qt * 32;
  const int64_t ld = a.ld, hoff = static_cast<int64_t>(head) * D;

  for (int i = tid; i < 32 * D / 4; i += kSplitThreads) {
    const int row = q0 + i / (D / 4);
    stage_row<D>(lds, i, row < G.q_end ? static_cast<const float*>(a.q) + row * ld + hoff : nullptr);
  }
  const int nt = run_tiles(G.runs, G.n_runs);
  const int t1 = static_cast<int>(static_cast<int64_t>(nt) * (sp + 1) / S);
  int t = static_cast<int>(static_cast<int64_t>(nt) * sp / S) + wave;
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) o[db] = f32x16{};
  float m = -INFINITY, l = 0.f;  // running max (both half-waves the same) and this lane's share of the sum
  Rows<D> kx;
  Cols<D> vx;
  Tile T{};
  if (t < t1) {
    T = tile_at(G.runs, ld, hoff, t);
    kx.prefetch(T.k, ld, T.nv, n, hh);
  }
  __syncthreads();
  while (t < t1) {
    vx.prefetch(T.v, ld, T.nv, n, hh);
    f32x16 s = row_product<D>(kx, lds, n, hh);
    const int nv = T.nv;
    t += kWaves;
    if (t < t1) {
      T = tile_at(G.runs, ld, hoff, t);
      kx.prefetch(T.k, ld, T.nv, n, hh);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = acc_row(e, hh) < nv ? s[e] * a.scale : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (__any(mx > m)) {
      const float mn = fmaxf(m, mx);
      const float alpha = mn == m ? 1.f : expf(m - mn);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) o[db] *= alpha;
    }
    const float ms = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = expf(s[e] - ms);
      l += s[e];
    }
    acc_product<D>(o, vx, s);
  }
  l += __shfl_xor(l, 32);
  __syncthreads();  // the query rows are no longer read
  acc_to_lds<D>(lds + wave * 32 * D, o, n, hh);
  split_stats(lds, D, wave, lane, m, l);
  __syncthreads();
  merge_split<float, D, D / 32>(a, lds, item, sp, head, q0, G.q_end);
}

// ------------------------------------------------------------------ backward

// Context token j of group G -> its K (or V) row, head 0.
__device__ inline const float* ctx_row(const BwdGroupArgs& G, int j, bool v, int64_t ld) {
  int r = 0;
  while (r + 1 < G.n_runs && j >= G.runs[r].n_tok) {
    j -= G.runs[r].n_tok;
    ++r;
  }
  return static_cast<const float*>(v ? G.runs[r].v : G.runs[r].k) + static_cast<int64_t>(j) * ld;
}

// Sum of the waves' accumulators (wave order) times scale, to rows of dst:
// row r of the block at dst_row(r) (null: not stored).
template <int D, class Row>
__device__ inline void merge_rows(const float* lds, float scale, Row dst_row) {
  constexpr int V = D / 32;
  typedef float vec __attribute__((ext_vector_type(V)));
  for (int i = threadIdx.x; i < 32 * 32; i += kSplitThreads) {
    vec s = vec{};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += *reinterpret_cast<const vec*>(lds + w * 32 * D + i * V);
    float* row = dst_row(i % 32);
    if (row) *reinterpret_cast<vec*>(row + (i / 32) * V) = s * scale;
  }
}

// dK, dV of 32 context keys: waves over the query tiles.
template <int D>
__device__ __forceinline__ void dkdv_f32_block(const BwdArgs& a, int b, float* lds) {
  int g = 0;
  while (g + 1 < a.n_groups && b >= a.groups[g + 1].kv_block_begin) ++g;
  const BwdGroupArgs& G = a.groups[g];
  const int head = (b - G.kv_block_begin) / G.n_kblocks, k0 = (b - G.kv_block_begin) % G.n_kblocks * 32;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ld = a.ld, hoff = static_cast<int64_t>(head) * D;
  float* Ks = lds;
  float* Vs = lds + 32 * kRowStr<D>;
  for (int i = tid; i < 32 * D / 4; i += kSplitThreads) {
    const int key = k0 + i / (D / 4);
    const bool ok = key < G.n_kv;
    stage_row<D>(Ks, i, ok ? ctx_row(G, key, false, ld) + hoff : nullptr);
    stage_row<D>(Vs, i, ok ? ctx_row(G, key, true, ld) + hoff : nullptr);
  }
  __syncthreads();
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) dk[db] = dv[db] = f32x16{};
  const int nq = G.q_end - G.q_begin;
  const float* lse = a.lse + static_cast<int64_t>(head) * a.n_q + G.q_begin;
  const float* dsum = a.dsum + static_cast<int64_t>(head) * a.n_q + G.q_begin;
  for (int t = wave; t * 32 < nq; t += kWaves) {
    const int nv = min(32, nq - t * 32);
    const int64_t off = static_cast<int64_t>(G.q_begin + t * 32) * ld + hoff;
    const float* q = static_cast<const float*>(a.q) + off;
    const float* go = static_cast<const float*>(a.d_out) + off;
    // statistics of the tile's rows (zeros past nv)
    const auto lse_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lse + t * 32), 0, nv * 4, 0x00020000);
    const auto dsum_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(dsum + t * 32), 0, nv * 4, 0x00020000);
    auto stat = [&](__amdgpu_buffer_rsrc_t buf, int e) {
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(buf, 16 * hh + 4 * acc_row(e, 0), 0, 0));
    };
    // the next operand's first batch is requested before each product
    Rows<D> qr, gr;
    Cols<D> gc, qc;
    qr.prefetch(q, ld, nv, n, hh);
    gc.prefetch(go, ld, nv, n, hh);
    f32x16 p = row_product<D>(qr, Ks, n, hh);
    gr.prefetch(go, ld, nv, n, hh);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = acc_row(e, hh);
      p[e] = r < nv ? expf(p[e] * a.scale - stat(lse_buf, e)) : 0.f;
    }
    acc_product<D>(dv, gc, p);
    qc.prefetch(q, ld, nv, n, hh);
    const f32x16 dp = row_product<D>(gr, Vs, n, hh);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = acc_row(e, hh);
      p[e] = r < nv ? p[e] * (dp[e] + stat(dsum_buf, e)) : 0.f;
    }
    acc_product<D>(dk, qc, p);
  }
  __syncthreads();
  acc_to_lds<D>(lds + wave * 32 * D, dk, n, hh);
  __syncthreads();
  merge_rows<D>(lds, a.scale, [&](int r) {
    return k0 + r < G.n_kv ? G.dk_ctx + static_cast<int64_t>(k0 + r) * ld + hoff : nullptr;
  });
  __syncthreads();
  acc_to_lds<D>(lds + wave * 32 * D, dv, n, hh);
  __syncthreads();
  merge_rows<D>(lds, 1.f, [&](int r) {
    return k0 + r < G.n_kv ? G.dv_ctx + static_cast<int64_t>(k0 + r) * ld + hoff : nullptr;
  });
}

// dQ of 32 queries: waves over the context tiles.
template <int D>
__device__ __forceinline__ void dq_f32_block(const BwdArgs& a, int b, float* lds) {
  int g = 0;
  while (g + 1 < a.n_groups && b >= a.groups[g + 1].dq_block_begin) ++g;
  const BwdGroupArgs& G = a.groups[g];
  const int head = (b - G.dq_block_begin) / G.n_qblocks;
  const int q0 = G.q_begin + (b - G.dq_block_begin) % G.n_qblocks * 32;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ld = a.ld, hoff = static_cast<int64_t>(head) * D;
  float* Qs = lds;
  float* Gs = lds + 32 * kRowStr<D>;
  for (int i = tid; i < 32 * D / 4; i += kSplitThreads) {
    const int row = q0 + i / (D / 4);
    const int64_t off = row * ld + hoff;
    const bool ok = row < G.q_end;
    stage_row<D>(Qs, i, ok ? static_cast<const float*>(a.q) + off : nullptr);
    stage_row<D>(Gs, i, ok ? static_cast<const float*>(a.d_out) + off : nullptr);
  }
  __syncthreads();
  f32x16 acc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) acc[db] = f32x16{};
  const int64_t stat = static_cast<int64_t>(head) * a.n_q + min(q0 + n, G.q_end - 1);
  const float ls = a.lse[stat], ds = a.dsum[stat];
  const int nt = run_tiles(G.runs, G.n_runs);
  for (int t = wave; t < nt; t += kWaves) {
    const Tile T = tile_at(G.runs, ld, hoff, t);
    Rows<D> kr, vr;
    Cols<D> kc;
    kr.prefetch(T.k, ld, T.nv, n, hh);
    vr.prefetch(T.v, ld, T.nv, n, hh);
    f32x16 p = row_product<D>(kr, Qs, n, hh);
    kc.prefetch(T.k, ld, T.nv, n, hh);
#pragma unroll
    for (int e = 0; e < 16; ++e) p[e] = acc_row(e, hh) < T.nv ? expf(p[e] * a.scale - ls) : 0.f;
    const f32x16 dp = row_product<D>(vr, Gs, n, hh);
#pragma unroll
    for (int e = 0; e < 16; ++e) p[e] = acc_row(e, hh) < T.nv ? p[e] * (dp[e] + ds) : 0.f;
    acc_product<D>(acc, kc, p);
  }
  __syncthreads();
  acc_to_lds<D>(lds + wave * 32 * D, acc, n, hh);
  __syncthreads();
  merge_rows<D>(lds, a.scale, [&](int r) {
    return q0 + r < G.q_end ? static_cast<float*>(a.dq) + (q0 + r) * ld + hoff : nullptr;
  });
}

// The dK/dV blocks and the dQ blocks of one call in one launch: they depend on
// the same inputs only, and a small layer has too few of either for the chip.
template <int D>
__global__ __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_f32_kernel(BwdArgs a, int kv_blocks) {
  static_assert(2 * 32 * kRowStr<D> <= split_lds_floats(D), "operand rows fit the merge area");
  __shared__ __attribute__((aligned(16))) float lds[split_lds_floats(D)];
  const int b = blockIdx.x;
  if (b < kv_blocks)
    dkdv_f32_block<D>(a, b, lds);
  else
    dq_f32_block<D>(a, b - kv_blocks, lds);
}

}  // namespace

hipError_t launch_forward_f32(const FwdArgs& a, int head_dim, hipStream_t stream) {
  if (a.n_blocks <= 0) return hipSuccess;
  const int64_t blocks = static_cast<int64_t>(a.n_blocks) * a.key_splits;
  if (a.key_splits < 1 || blocks > 0x7fffffff || (a.key_splits > 1 && !a.partial)) return hipErrorInvalidValue;
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kSplitThreads);
  if (head_dim == 128)
    hipLaunchKernelGGL(fwd_f32_kernel<128>, grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL(fwd_f32_kernel<64>, grid, block, 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.key_splits == 1) return e;
  const dim3 cgrid(a.n_blocks);
  if (head_dim == 128)
    hipLaunchKernelGGL((combine_split_kernel<float, 128, 4>), cgrid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((combine_split_kernel<float, 64, 2>), cgrid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_bwd_f32(const BwdArgs& a, int dq_blocks, int kv_blocks, int head_dim, hipStream_t stream) {
  const int64_t blocks = static_cast<int64_t>(dq_blocks) + kv_blocks;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kSplitThreads);
  if (head_dim == 128)
    hipLaunchKernelGGL(bwd_f32_kernel<128>, grid, block, 0, stream, a, kv_blocks);
  else
    hipLaunchKernelGGL(bwd_f32_kernel<64>, grid, block, 0, stream, a, kv_blocks);
  return hipGetLastError();
}

}  // namespace mssa
