// Multi-scale self-attention backward: the chain rule through Eq. 4 of Ms.
// Forcing (Sec. 4.1), whose rolling-window training (Sec. 3.1, Alg. 1)
// differentiates the attention of every window state.  For each head and
// query scale s, with P = softmax(scale q k_s^T) over the context of s and dO
// the gradient of the output:
//   dV_s = P^T dO,  dS = P * (dO V_s^T - rowsum(dO * O)),
//   dQ = scale dS K_s,  dK_s = scale dS^T Q.
// The statistics come from the forward: the log of each row's softmax
// denominator (lse), and rowsum(dO * O) (dot_kernel, which stores both
// negated in the units the kernels use).  Context gradients are kept per
// query scale in fp32; scatter_kernel then sums, for every sink, history and
// window token, the gradients of the context rows made from it (the adjoint
// of the resampling: the block mean hands g / c to each of its c cells, the
// strided pick g to the block's first cell).  Fixed summation orders and no
// atomics: the result is the same bits on every run.
//
// bf16 path (gfx950 matrix cores, v_mfma_f32_32x32x16_bf16, fp32
// accumulation), five products in two kernels so that no gradient needs
// atomics:
//   dkdv_kernel  64 or 32 context keys per wave, one wave per SIMD; queries stream in
//                32-query stages: S = Q K^T, P (lane = key), dV^T += dO^T P, dP =
//                dO V^T, dS = P (dP - rowsum), dK^T += Q^T dS, with dO^T, Q^T
//                from transposing reads, and dS (bf16, the value its own
//                product uses) to a tile in HBM.
//   dq_kernel    dQ^T += K^T dS^T over the context, 32 queries per wave, K
//                rows and the wave's dS tiles streamed through LDS and read
//                transposed; it reads each dS element once from HBM instead
//                of recomputing S and dP.
// One XOR-swizzled copy of each staged K / Q / dO tile serves both read
// patterns without bank conflicts; stages arrive by direct global -> LDS
// transfers (no staging registers).  Rows past the end of a context or query
// range are zero-filled and add nothing to any gradient.
//
// fp32 plans take the dQ, dK and dV kernels of attention_f32.hip; the rowsum
// and scatter kernels here serve both.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "kernels.hpp"
#include "lds_stage.hpp"
#include "xcd.hpp"

namespace mssa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// Context token j of group G -> its K (or V) row, head 0; nullptr past the end.
template <typename T>
__device__ inline const T* ctx_row(const BwdGroupArgs& G, int j, bool v, int64_t ld) {
  if (j >= G.n_kv) return nullptr;
  int r = 0;
  while (r + 1 < G.n_runs && j >= G.runs[r].n_tok) {
    j -= G.runs[r].n_tok;
    ++r;
  }
  return static_cast<const T*>(v ? G.runs[r].v : G.runs[r].k) + static_cast<int64_t>(j) * ld;
}

// Operand shapes of both bf16 kernels: a 32-row block is read as the A
// operand of a 32x32x16 MFMA (lane n takes row n and the 8 columns of its
// half-wave), or, through the transposing read, as X^T[d][row] of a 32-wide d
// block and 16 rows in the row order in which a 32x32 accumulator's lane holds
// its 16 values, so that the accumulator packed to bf16 is the matching B
// operand.
template <int D>
struct Lay {
  static constexpr int KS = D / 16, DB = D / 32;
};

// ------------------------------------------------------------------ rowsum(dO * O)

// One row (query, head) per group of L = head_dim * sizeof(T) / 16 lanes (8,
// 16 or 32; rows are contiguous, so a wave reads 1-2 KB in one piece), each
// lane 16 bytes of O and dO; the group's partial sums meet by lane
// exchanges in a fixed order.
template <typename T>
__global__ __launch_bounds__(kDotThreads) void dot_kernel(DotArgs a) {
  constexpr int N = 16 / sizeof(T);
  typedef T vecT __attribute__((ext_vector_type(N)));
  const int L = a.head_dim / N;
  const int64_t gt = static_cast<int64_t>(blockIdx.x) * kDotThreads + threadIdx.x;
  const int64_t r = gt / L, rows = static_cast<int64_t>(a.n_q) * a.num_heads;
  const int c = static_cast<int>(gt % L);
  float acc = 0.f;
  if (r < rows) {
    // rows are contiguous: row r = (query r / heads, head r % heads) at r * head_dim
    const int64_t off = r * a.head_dim + c * N;
    const vecT ov = *reinterpret_cast<const vecT*>(static_cast<const T*>(a.out) + off);
    const vecT gv = *reinterpret_cast<const vecT*>(static_cast<const T*>(a.d_out) + off);
#pragma unroll
    for (int e = 0; e < N; ++e) acc = __builtin_fmaf(static_cast<float>(ov[e]), static_cast<float>(gv[e]), acc);
  }
  for (int m = L >> 1; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
  if (r < rows && c == 0) {
    const int q = static_cast<int>(r / a.num_heads), h = static_cast<int>(r % a.num_heads);
    // Both statistics are stored negated, as the dK/dV kernel's accumulator
    // inputs: -rowsum, and -lse / scale (the row's log-sum-exp in units of the
    // unscaled scores q k^T).
    a.dsum[static_cast<int64_t>(h) * a.n_q + q] = -acc;
    if (a.lse) a.lse2[static_cast<int64_t>(h) * a.n_q + q] = -a.lse[static_cast<int64_t>(h) * a.n_q + q] * a.inv_scale;
  }
}

// ------------------------------------------------------------------ bf16 kernels

// Stage rows: one copy per tensor in the 256-byte swizzled layout of
// lds_stage.hpp (row reads and transposing reads both conflict-free), filled
// by direct transfers.
__device__ inline int swz(int row, int col) { return swz256(row, col); }

// ------------------------------------------------------------------ bf16: dQ

// dQ = scale dS K, from the dS tiles the dK/dV kernel wrote.  A block owns
// 256 queries, eight waves of 32 (two per SIMD).  The context streams through
// LDS in 64-key stages inside one run at a time, cut as the tiles were: the
// stage's K rows (one swizzled copy for the block) and each wave's own 4 KB
// dS tile arrive by direct transfers into three stage buffers (the one read
// and two in flight: the tiles come from HBM once, and HBM latency needs that
// depth).  Rows past a run's end arrive as zeros in both, so they add
// nothing.  Each wave accumulates dQ^T += K^T dS^T with both operands from
// transposing reads: K^T from the K rows, dS^T from the tile's 64-byte rows
// (keys) of 32 query positions, which become the accumulator's columns.
// Position p of a tile row holds query 8 ((p % 16) / 4) + 4 (p / 16) + p % 4
// of the 32-query block: the order in which the dK/dV kernel's lanes hold
// them.  A block's chain of stages is bound by their latency (about 0.85 us
// each), so where the blocks leave CUs idle the context is split over
// dq_splits of them (6 heads of 64 on 17 x 23: 36 blocks, 45 us; with 7 splits
// 14 us and 6 us for the sum).  A split's sum (fp32) takes the place of the dS
// tiles its wave has read, which no one else reads: D / 32 tiles' bytes, so a
// split has at least as many stages (dq_splits of its group, 1: no split).
template <int D>
__global__ __launch_bounds__(kBwdQThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dq_kernel(BwdArgs a) {
  constexpr int DB = Lay<D>::DB;
  constexpr int BN = kBwdKS;                       // keys per stage
  constexpr int NW = kBwdQThreads / 64;            // waves of 32 queries
  constexpr int KT = BN * 256;                     // bytes of the stage's K rows (256-byte swizzled rows)
  constexpr int DT = BN * 64;                      // bytes of one wave's dS tile
  // The tile's LDS footprint: its second half sits 128 bytes further on, so
  // that the two halves' rows a transposing read takes together fall in
  // different banks.
  constexpr int DTL = DT + 128;
  constexpr int STB = KT + NW * DTL;
  constexpr int NK = KT / 1024 / NW;               // 1 KB K transfers per wave and stage
  constexpr int NDS = DT / 1024;                   // 1 KB dS transfers per wave and stage
  static_assert(NK * 1024 * NW == KT && NW * 32 == kBwdQ && BN % 32 == 0 && NDS % 2 == 0, "stage shape");
  __shared__ __attribute__((aligned(16))) char lds[3 * STB];

  // block b takes context split b / dq_blocks, if its group has that many
  const int sp = blockIdx.x / a.dq_blocks, b = blockIdx.x - sp * a.dq_blocks;
  int g = 0;
  while (g + 1 < a.n_groups && b >= a.groups[g + 1].dq_block_begin) ++g;
  const BwdGroupArgs& G = a.groups[g];
  if (sp >= G.dq_splits) return;
  const int idx = xcd_remap(b - G.dq_block_begin, G.n_qblocks * a.num_heads);
  const int hl = idx / G.n_qblocks, qt = idx % G.n_qblocks;  // head of the launch
  const int head = a.head0 + hl;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hh = lane >> 5;
  const int qb = qt * NW + wave;                   // the wave's 32-query block of the group
  const bool wave_ok = G.q_begin + qb * 32 < G.q_end;
  const int q_row = G.q_begin + qb * 32 + 8 * ((n & 15) >> 2) + 4 * (n >> 4) + (n & 3);
  const int64_t ld = a.ld, hoff = static_cast<int64_t>(head) * D;

  f32x16 acc[DB];  // dQ^T: lane n holds tile position n's query
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x16{};

  const int nr = G.n_runs;
  int nst = 0;
  for (int r = 0; r < nr; ++r) nst += (G.runs[r].n_tok + BN - 1) / BN;
  const int st0 = static_cast<int>(static_cast<int64_t>(nst) * sp / G.dq_splits);  // this split's first stage
  nst = static_cast<int>(static_cast<int64_t>(nst) * (sp + 1) / G.dq_splits) - st0;
  struct Stream {
    const __bf16* k;
    int left;  // tokens of the current run from k on
    int r;
  };
  const int64_t tile_step = static_cast<int64_t>(BN) * ld;
  auto seek = [&](Stream& s, int r) {
    while (r < nr && G.runs[r].n_tok == 0) ++r;
    s.r = r;
    if (r < nr) {
      s.k = static_cast<const __bf16*>(G.runs[r].k) + hoff;
      s.left = G.runs[r].n_tok;
    }
  };
  auto step = [&](Stream& s) {
    s.left -= BN;
    s.k += tile_step;
    if (s.left <= 0) seek(s, s.r + 1);
  };

  // Per-lane global offsets of this wave's K transfers (the same every
  // stage): transfer t = wave NK + i covers bytes 1024 t of the K rows,
  // logical chunk of the fixed LDS slot, zero past D.  The dS tile is copied
  // as it lies, 1 KB per transfer, non-temporal (each element is read once;
  // -1 % against plain loads, K rows keep their L2 lines).
  const uint32_t row_bytes = static_cast<uint32_t>(ld) * 2;
  uint32_t voff[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const int p = (wave * NK + i) * 1024 + 16 * lane;
    const int row = p >> 8, phys = (p >> 4) & 15;
    const int lc = unswz256(row, phys);
    voff[i] = lc < D / 8 ? row * row_bytes + lc * 16 : kPastEnd;
  }
  __bf16* const ds_wave = static_cast<__bf16*>(G.ds) +
      ((static_cast<int64_t>(hl) * G.ds_qblocks + (wave_ok ? qb : 0)) * G.ds_stages + st0) * (BN * 32);
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  auto issue = [&](const Stream& s, int st, int buf) {
    const int nv = min(s.left, BN);
    const i32x4 rk = rsrc_of(s.k, static_cast<uint32_t>(nv - 1) * row_bytes + D * 2);
    const uint32_t base = lds0 + buf * STB;
#pragma unroll
    for (int i = 0; i < NK; ++i) dma16(rk, voff[i], __builtin_amdgcn_readfirstlane(base + (wave * NK + i) * 1024));
    if (wave_ok) {
      // the tile's two halves (positions 16 hh + 8 j + e of every slot, j = 0, 1)
      // each hold 32 bytes per slot; slots past the run's end read as zeros
      const __bf16* tile = ds_wave + static_cast<int64_t>(st) * (BN * 32);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const i32x4 rd = rsrc_of(tile + j * (BN * 16), static_cast<uint32_t>(nv) * 32);
#pragma unroll
        for (int i = 0; i < NDS / 2; ++i)
          dma16_nt(rd, i * 1024 + 16 * lane,
                   __builtin_amdgcn_readfirstlane(base + KT + wave * DTL + j * (DT / 2 + 128) + i * 1024));
      }
    }
  };
  // all of this wave's transfers but the last stage's
  auto wait_but_one = [&]() {
    if (wave_ok)
      wait_vmcnt<NK + NDS>();
    else
      wait_vmcnt<NK>();
  };
  // Transposing reads: rows R + t_lane (+ 8 for the upper half), R a
  // multiple of 16; K at columns 32 db + t_col (swizzled rows), dS at t_col.
  const int t_lane = 4 * (lane >> 5) + ((lane & 15) >> 2);
  const int t_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  int k_rd[DB][2], d_rd[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    d_rd[h] = ((t_col >> 3) & 1) * (BN * 16 + 64) + (t_lane + 8 * h) * 16 + (t_col >> 4) * 8 + (t_col & 7);
#pragma unroll
    for (int db = 0; db < DB; ++db) k_rd[db][h] = swz(t_lane + 8 * h, db * 32 + t_col);
  }
  auto tr = [](const __bf16* p0, int o0, int o1) {
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p0 + o0));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p0 + o1));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto stage = [&](int buf) {
    const __bf16* Ks = reinterpret_cast<const __bf16*>(lds + buf * STB);
    const __bf16* Ds = reinterpret_cast<const __bf16*>(lds + buf * STB + KT + wave * DTL);
#pragma unroll
    for (int rb = 0; rb < BN / 16; ++rb) {
      const bf16x8 dst = tr(Ds + rb * 16 * 16, d_rd[0], d_rd[1]);
#pragma unroll
      for (int db = 0; db < DB; ++db)
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr(Ks + rb * 16 * 128, k_rd[db][0], k_rd[db][1]), dst,
                                                          acc[db], 0, 0, 0);
    }
  };

  Stream ls;
  {
    int r = 0, skip = st0;
    while (r < nr && skip >= (G.runs[r].n_tok + BN - 1) / BN) {
      skip -= (G.runs[r].n_tok + BN - 1) / BN;
      ++r;
    }
    seek(ls, r);
    ls.k += skip * tile_step;
    ls.left -= skip * BN;
  }
  if (nst > 0) issue(ls, 0, 0);
  if (nst > 1) {
    step(ls);
    issue(ls, 1, 1);
    wait_but_one();
  } else {
    wait_vmcnt<0>();
  }
  __syncthreads();
  for (int it = 0; it < nst; ++it) {
    if (it + 2 < nst) {
      step(ls);
      issue(ls, it + 2, (it + 2) % 3);
    }
    if (wave_ok) stage(it % 3);
    if (it + 2 < nst)
      wait_but_one();
    else
      wait_vmcnt<0>();
    __syncthreads();
  }

  if (G.dq_splits > 1) {
    // this split's sum where dq_sum_kernel finds it; the last stage's wait and
    // barrier have passed, so the wave's tiles are read
    if (wave_ok) {
      f32x4* op = reinterpret_cast<f32x4*>(ds_wave) + lane;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          f32x4 v;
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = acc[db][4 * jj + i];
          op[(db * 4 + jj) * 64] = v;
        }
    }
    return;
  }
  if (wave_ok && q_row < G.q_end) {
    __bf16* op = static_cast<__bf16*>(a.dq) + static_cast<int64_t>(q_row) * ld + hoff + 4 * hh;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = static_cast<__bf16>(acc[db][4 * jj + i] * a.scale);
        *reinterpret_cast<bf16x4*>(op + db * 32 + 8 * jj) = v;
      }
  }
}

// dQ from the fp32 sums of the context splits, split 0 first.  A block per
// 32-query block and head, a wave per 32 channels, lanes as in dq_kernel.
template <int D>
__global__ __launch_bounds__(2 * D) void dq_sum_kernel(BwdArgs a) {
  static_assert(2 * D == 64 * Lay<D>::DB, "a wave per 32 channels");
  int g = 0, b = blockIdx.x;
  for (; g + 1 < a.n_groups; ++g) {
    const int n = a.groups[g].dq_splits > 1 ? (a.groups[g].q_end - a.groups[g].q_begin + 31) / 32 * a.num_heads : 0;
    if (b < n) break;
    b -= n;
  }
  const BwdGroupArgs& G = a.groups[g];
  const int nqb = (G.q_end - G.q_begin + 31) / 32, hl = b / nqb, qb = b % nqb;
  const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5, db = threadIdx.x >> 6;
  const __bf16* tiles = static_cast<const __bf16*>(G.ds) +
                        (static_cast<int64_t>(hl) * G.ds_qblocks + qb) * G.ds_stages * (kBwdKS * 32);
  f32x4 s[4] = {};
  auto add = [&](auto n_c, int k0) {  // splits k0 .. k0 + n - 1, their loads in flight together
    constexpr int N = decltype(n_c)::value;
    f32x4 v[N][4];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int64_t st0 = static_cast<int64_t>(G.ds_stages) * (k0 + k) / G.dq_splits;
      const f32x4* p = reinterpret_cast<const f32x4*>(tiles + st0 * (kBwdKS * 32)) + db * 256 + lane;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) v[k][jj] = p[jj * 64];
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) s[jj] += v[k][jj];
  };
  int k = 0;
  for (; k + 4 <= G.dq_splits; k += 4) add(std::integral_constant<int, 4>{}, k);
  if (k + 2 <= G.dq_splits) {
    add(std::integral_constant<int, 2>{}, k);
    k += 2;
  }
  if (k < G.dq_splits) add(std::integral_constant<int, 1>{}, k);
  const int q_row = G.q_begin + qb * 32 + 8 * ((n & 15) >> 2) + 4 * (n >> 4) + (n & 3);
  if (q_row >= G.q_end) return;
  __bf16* op = static_cast<__bf16*>(a.dq) + static_cast<int64_t>(q_row) * a.ld +
               static_cast<int64_t>(a.head0 + hl) * D + 4 * hh + db * 32;
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    bf16x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = static_cast<__bf16>(s[jj][i] * a.scale);
    *reinterpret_cast<bf16x4*>(op + 8 * jj) = v;
  }
}

// ------------------------------------------------------------------ bf16: dK, dV

// d += a b, with d in ordinary registers (read by VALU instructions later) or
// in accumulation registers.  Of the 512 registers of a lone wave half are
// accumulation registers, which VALU instructions cannot read; left to itself
// the compiler put every product's result there and copied S, dP and their
// starting values back and forth (264 copies per 64 MFMAs).  It does not see
// these as matrix instructions, so the waits it would put around one are the
// kernel's to keep:
// - a VALU or memory instruction that touches d comes two MFMAs or 19 cycles of
//   s_nop later (mfma_done ties the reads of d to that place);
// - an MFMA comes two instructions after a VALU instruction that writes one of
//   its operands (mfma_operands where the compiler may have put a copy);
// - a VALU instruction that writes a register of the first product's c comes an
//   MFMA or 16 cycles later (mfma_read keeps c until there; its last registers are
//   read late).
// tests/test_matrix_core_waits.py checks both in the emitted code.
// kAccB: b lies in accumulation registers.
template <bool kAccB = false>
__device__ inline void mfma_v(f32x16& d, bf16x8 a, bf16x8 b) {
  if constexpr (kAccB)
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ inline void mfma_a(f32x16& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}

__device__ inline void mfma_done(f32x16& d) { asm volatile("" : "+v"(d)); }
__device__ inline void mfma_read(const f32x16& c) { asm volatile("" ::"v"(c)); }
__device__ inline void mfma_operands() { asm volatile("s_nop 1"); }

// f(I) for I = 0 .. N - 1 as constants (integral_constant), unrolled by the
// front end: the unroller gives up on the dK/dV kernel's step.
template <class F, int... I>
__device__ __forceinline__ void for_constants(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// d = c + a b, the first product of a chain.
template <bool kAccB = false>
__device__ inline void mfma_first(f32x16& d, bf16x8 a, bf16x8 b, const f32x16& c) {
  if constexpr (kAccB)
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "a"(b), "v"(c));
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "v"(b), "v"(c));
}

// dK/dV: a block owns 128 KB context keys, four waves (one per SIMD, 512
// registers) of KB 32-key blocks each: with KB = 2 every operand read from LDS
// feeds two MFMAs, with KB = 1 a layer of few blocks has twice as many and a
// step is shorter (kv_block_keys in plan.cpp chooses).  Queries stream in
// 32-query stages t; a step is
//   A  S_t  = Q_t K^T                (K fragments in registers)
//   B  dK^T += Q_{t-1}^T dS_{t-1}
//   C  dP_t = dO_t V^T               (KB = 2: V from the block's 64 KB of LDS;
//                                     KB = 1: V fragments in registers)
//   D  dV^T += dO_t^T P_t
// of N = D / 16 chunks each: one operand (row read or transposing read, kLead
// chunks ahead of its use) and its KB MFMAs.  What else there is to do is cut
// into pieces of about four instructions, one behind every MFMA: P_t =
// exp2(c S_t) during B and C, dS_t = P_t dP_t during D, its stores and the
// transfers during A.  A wave alone on its SIMD issues one instruction at a
// time, and an MFMA waits at issue until the one before has left the core (32
// cycles), so the order within the stream is what keeps the matrix core fed;
// scheduling barriers hold it.  The loop is unrolled over the stage buffers,
// which makes every LDS address a lane offset plus an immediate.  Nothing is
// handed between waves and there is one barrier per step, between C and D.
// Stage t's Q, dO and row statistics live in LDS buffer t % 4.  Stage t + 2 is
// requested during A of step t into the buffer of stage t - 2 (last read in B
// of step t - 1, before that step's barrier); the wait for stage t + 1 comes
// before the barrier of step t, and D of step t may already read it.  Memory
// operations complete in order: the wait leaves the younger ones in flight.
// The row products start from the stage's negated row statistics (-lse / scale,
// -rowsum), so that S arrives as S - lse / scale (P = exp2(c S'); kQS, queries
// pre-scaled: c = 1) and dP as dP - rowsum.  dS (bf16, the value the dK product
// uses) goes to its tile in HBM by range-checked stores at a per-lane offset
// fixed for the whole kernel.
// Measured (12 heads of 128, 9360 + 3510 queries on 26910 and 12870 keys, KB = 2):
// 3.0 - 3.3 ms, matrix cores busy two thirds of the cycles (a wave is there nine
// tenths of them: the grid's end), LDS 30 %, the clock (1.6 GHz) set by power;
// pairs of waves sharing a SIMD, one on the matrix core and one on the softmax,
// handing P over through LDS behind two barriers per 64 queries: 4.24 - 4.43 ms,
// 44 %.
// Vector, scalar and LDS instructions per MFMA: 3.5, with the pairs 6.8.
// Whole backward of small layers with those pairs of waves, KB = 2 and KB = 1: 13
// heads of 128, 108 queries on 489 keys and two coarser groups 40.1, 53.3 and
// 41.3 us; 3 heads of 64, 1275 on 5341 and two groups 114, 80.3 and 66.8.
template <int D, bool kQS, int KB>
__global__ __launch_bounds__(kBwdKVThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void dkdv_kernel(BwdArgs a) {
  using L = Lay<D>;
  constexpr int N = L::KS, DB = L::DB;                  // chunks per phase, 32-channel blocks
  static_assert(N == 2 * DB, "row and transposing phases have the same chunks");
  constexpr int BQ = kBwdStage;                         // queries per stage
  constexpr int BK = KB * kBwdKVKeys;                   // keys per block
  constexpr int QT = BQ * 256;                          // bytes of one swizzled tile (256-byte rows)
  constexpr int STB = 2 * QT;                           // Q | dO
  constexpr int kStat = 1024;                           // -lse / scale | unused | -rowsum | unused (256 bytes each, 128 used)
  constexpr int NBUF = 4;
  constexpr int NDMA = 2 * QT / 1024 / 4;               // 1 KB transfers per wave and stage
  constexpr int kStat0 = NBUF * STB, kV0 = kStat0 + NBUF * kStat;  // the stages' statistics, the block's V rows
  constexpr int kDump = kV0 + (KB == 2 ? BK * 256 : 0); // 1 KB that nothing reads
  constexpr int kLead = 4;                              // chunks an operand is read ahead
  static_assert(BQ == 32 && NDMA == 4 && kBwdKVKeys == 128 && (KB == 1 || KB == 2) && 4 * N % kLead == 0, "stage shape");
  __shared__ __attribute__((aligned(16))) char lds[kDump + 1024];

  const int b = blockIdx.x;
  int g = 0;
  while (g + 1 < a.n_groups && b >= a.groups[g + 1].kv_block_begin) ++g;
  const BwdGroupArgs& G = a.groups[g];
  // an eighth of every group per XCD, not of the grid: the groups' blocks differ
  // in length (293 and 110 stages on the 1.3B layer), and contiguous eighths of
  // the grid left the XCDs with the short group idle for 30 % of the kernel
  const int idx = xcd_remap(b - G.kv_block_begin, G.n_kblocks * a.num_heads);
  const int hl = idx / G.n_kblocks, kt = idx % G.n_kblocks;  // head of the launch
  const int head = a.head0 + hl;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hh = lane >> 5;
  const int64_t ld = a.ld, hoff = static_cast<int64_t>(head) * D;
  const float c = a.scale_log2e;
  const int key0 = kt * BK + wave * 32 * KB + n;  // this lane's keys: key0 + 32 kb

  // Byte offset, in the tiles of a 32-query block, of the lane's dS of each
  // key: the key's 64-key stage (its run's stages, as the dQ kernel walks
  // them), slot and the lane's 8 queries of each tile half.  Keys past the
  // context point past the range: the range check drops their stores.
  uint32_t ds_voff[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int key = key0 + kb * 32;
    const bool ok = key < G.n_kv;
    int j = ok ? key : 0, st = 0, r = 0;
    while (r + 1 < G.n_runs && j >= G.runs[r].n_tok) {
      st += (G.runs[r].n_tok + kBwdKS - 1) / kBwdKS;
      j -= G.runs[r].n_tok;
      ++r;
    }
    ds_voff[kb] = ok ? static_cast<uint32_t>((st + j / kBwdKS) * (kBwdKS * 64) + (j % kBwdKS) * 32 + 16 * hh) : kPastEnd;
  }
  const uint32_t ds_qbytes = static_cast<uint32_t>(G.ds_stages) * (kBwdKS * 64);  // one 32-query block's tiles
  const char* const ds_head = static_cast<const char*>(G.ds) + static_cast<int64_t>(hl) * G.ds_qblocks * ds_qbytes;

  // This wave's transfers of a stage: 1 KB (4 rows) each, rows 4 (4 (wave & 1)
  // + i) + lane / 16 of the Q (waves 0, 1) or dO (waves 2, 3) tile, and a row
  // statistic (waves 0, 2; lanes past the 32 queries read zeros).  Rows past
  // the range's end arrive as zeros with zero statistics: their P = 1 meets
  // zero dO rows and dS = 1 (0 - 0) = 0.
  const uint32_t row_bytes = static_cast<uint32_t>(ld) * 2;
  // Transfer i's offset is that of transfer 0 with its chunk XORed with i, 4 i
  // rows on (three registers less than one offset per transfer: the kernel
  // uses all 256).
  const int row0 = 16 * (wave & 1) + (lane >> 4), lc0 = unswz256(row0, lane & 15);
  const uint32_t voff0 = lc0 < D / 8 ? row0 * row_bytes + lc0 * 16 : kPastEnd;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int q_begin = G.q_begin, nq = G.q_end - G.q_begin, nst = (nq + BQ - 1) / BQ;
  const __bf16* const x_head =
      static_cast<const __bf16*>(wave < 2 ? a.q : a.d_out) + hoff + static_cast<int64_t>(q_begin) * ld;
  const float* const s_head = (wave == 0 ? a.lse2 : a.dsum) + static_cast<int64_t>(head) * a.n_q + q_begin;
  // Past the last stage dO and -rowsum are zeros, and the queries and their
  // -lse / scale stay those of the buffer's previous stage (the transfers'
  // zeros go to kDump): a finite P whatever K holds, where a row of zeros
  // would be NaN against an infinite key.  Bringing the last stage again
  // instead cost its time: 2 of 38 us where 25 stages fill 28.
  auto issue = [&](int ts, int t, int i) {  // transfer i of stage ts into buffer t % 4 (i == NDMA: the statistic)
    const int nv = max(0, min(BQ, nq - ts * BQ));
    const bool keep = wave < 2 && nv == 0;
    if (i < NDMA) {
      const i32x4 rs = rsrc_of(x_head + static_cast<int64_t>(ts) * BQ * ld, nv > 0 ? static_cast<uint32_t>(nv - 1) * row_bytes + D * 2 : 0u);
      const uint32_t dst = (t & (NBUF - 1)) * STB + (wave * NDMA + i) * 1024;
      dma16(rs, (voff0 ^ (i * 16)) + i * 4 * row_bytes, __builtin_amdgcn_readfirstlane(lds0 + (keep ? kDump : dst)));
    } else {
      // waves 1 and 3 fill unused parts: every wave counts the same transfers
      const uint32_t dst = kStat0 + (t & (NBUF - 1)) * kStat + wave * 256;
      dma4(rsrc_of(s_head + ts * BQ, static_cast<uint32_t>(nv) * 4), 4 * lane,
           __builtin_amdgcn_readfirstlane(lds0 + (keep ? kDump : dst)));
    }
  };

  // Everything a block starts with is requested at once: the first two stages,
  // the K fragments and the V rows (zeros past the context), kept in registers
  // until they are all there.
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i <= NDMA; ++i) issue(t, t, i);
  // fewer stages than buffers: the others hold the last stage's queries
  if (KB == 2 && wave < 2)
    for (int t = nst; t < NBUF; ++t)
#pragma unroll
      for (int i = 0; i <= NDMA; ++i) issue(nst - 1, t, i);
  bf16x8 kf[KB][N], vf[KB == 1 ? N : 1];  // KB = 1: V fragments too, in accumulation registers
  {
    constexpr int CH = D / 8, RP = kBwdKVThreads / CH, NV = BK / RP;  // 16-byte chunks per row, rows per pass, passes
    bf16x8 vrow[NV];
    if constexpr (KB == 1) {
      const __bf16* vp = ctx_row<__bf16>(G, key0, true, ld);
#pragma unroll
      for (int ks = 0; ks < N; ++ks)
        vf[ks] = vp ? *reinterpret_cast<const bf16x8*>(vp + hoff + hh * 8 + ks * 16) : bf16x8{};
    }
#pragma unroll
    for (int i = 0; i < NV && KB == 2; ++i) {
      const __bf16* vp = ctx_row<__bf16>(G, kt * BK + i * RP + tid / CH, true, ld);
      vrow[i] = vp ? *reinterpret_cast<const bf16x8*>(vp + hoff + tid % CH * 8) : bf16x8{};
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const __bf16* kp = ctx_row<__bf16>(G, key0 + kb * 32, false, ld);
#pragma unroll
      for (int ks = 0; ks < N; ++ks)
        kf[kb][ks] = kp ? *reinterpret_cast<const bf16x8*>(kp + hoff + hh * 8 + ks * 16) : bf16x8{};
    }
    // the queries of stage -1 (multiplied by dS = 0 in the first step)
    for (int i = KB == 2 && nst < NBUF ? QT / 16 : tid; i < QT / 16; i += kBwdKVThreads)
      reinterpret_cast<bf16x8*>(lds + (NBUF - 1) * STB)[i] = bf16x8{};
#pragma unroll
    for (int i = 0; i < NV && KB == 2; ++i)
      *reinterpret_cast<bf16x8*>(reinterpret_cast<__bf16*>(lds + kV0) + swz(i * RP + tid / CH, tid % CH * 8)) = vrow[i];
  }
  wait_vmcnt<0>();  // the transfers too, which the compiler does not count
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int ks = 0; ks < N; ++ks) {
      asm volatile("" : "+v"(kf[kb][ks]));
      if (KB == 1) asm volatile("" : "+a"(vf[ks]));
    }
  __syncthreads();

  // Lane offsets (elements) of row reads and of transposing reads.
  const int r_rd = swz(n, hh * 8);
  const int t_lane = 4 * (lane >> 5) + ((lane & 15) >> 2);
  const int t_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  int t_rd[DB][2];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int h = 0; h < 2; ++h) t_rd[db][h] = swz(t_lane + 8 * h, db * 32 + t_col);
  const __bf16* const Vw = reinterpret_cast<const __bf16*>(lds + kV0) + wave * 32 * KB * 128;
  auto tile = [&](int buf, int which) { return reinterpret_cast<const __bf16*>(lds + buf * STB + which * QT); };  // 0: Q, 1: dO
  auto row_op = [&](const __bf16* x, int ks) { return *reinterpret_cast<const bf16x8*>(x + (r_rd ^ (ks * 16))); };
  auto tr_op = [&](const __bf16* x, int i) {  // i = (16-row half, channel block)
    const __bf16* r0 = x + (i / DB) * 16 * 128;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(r0 + t_rd[i % DB][0]));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(r0 + t_rd[i % DB][1]));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  f32x16 dk[DB][KB], dv[DB][KB], s[KB], dp[KB], stat;
  i32x4 pw[KB][2], ds[KB][2];  // P_t and dS packed as B operands, [key block][16-query half]
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
    for (int db = 0; db < DB; ++db) dk[db][kb] = dv[db][kb] = f32x16{};
    ds[kb][0] = ds[kb][1] = i32x4{};
  }
  auto load_stat = [&](int buf, int which) {  // element e: query 8 (e / 4) + 4 hh + e % 4
    const float* p = reinterpret_cast<const float*>(lds + kStat0 + buf * kStat) + which * 64;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(p + 8 * j + 4 * hh);
#pragma unroll
      for (int i = 0; i < 4; ++i) stat[4 * j + i] = v[i];
    }
  };
  auto pack = [](float x, float y) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(int, bf16x2{static_cast<__bf16>(x), static_cast<__bf16>(y)});
  };
  // Pair x (of 8 KB) of the lane's elements: key block x / 8, elements e, e + 1.
  // P stays in s in fp32 for dS.
  auto p_pair = [&](int x) {
    const int kb = x >> 3, e = (x & 7) * 2;
    s[kb][e] = __builtin_amdgcn_exp2f(kQS ? s[kb][e] : s[kb][e] * c);
    s[kb][e + 1] = __builtin_amdgcn_exp2f(kQS ? s[kb][e + 1] : s[kb][e + 1] * c);
    pw[kb][e >> 3][(e & 7) >> 1] = pack(s[kb][e], s[kb][e + 1]);
  };
  auto ds_pair = [&](int x) {
    const int kb = x >> 3, e = (x & 7) * 2;
    ds[kb][e >> 3][(e & 7) >> 1] = pack(s[kb][e] * dp[kb][e], s[kb][e + 1] * dp[kb][e + 1]);
  };
  auto ds_store = [&](int t, int kb, int h) {  // stage t's dS of one key block and tile half
    const i32x4 rd = rsrc_of(ds_head + static_cast<int64_t>(max(t, 0)) * ds_qbytes, t >= 0 && t < nst ? ds_qbytes : 0u);
    if (h == 0)
      bstore16_nt<0>(ds[kb][0], rd, ds_voff[kb], 0);
    else
      bstore16_nt<kBwdKS * 32>(ds[kb][1], rd, ds_voff[kb], 0);
  };
  // Runs f(x) for the pairs x that slot j of n (of which the first does
  // nothing: the pairs' inputs may still be in the matrix core) has to do.
  auto spread = [](auto J, auto n_c, auto pairs_c, auto&& f) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value, n = decltype(n_c)::value, pairs = decltype(pairs_c)::value;
    if constexpr (j > 0) {
      constexpr int x0 = ((j - 1) * pairs + n - 2) / (n - 1), x1 = (j * pairs + n - 2) / (n - 1);
      if constexpr (x0 < x1) f(x0);
      if constexpr (x0 + 1 < x1) f(x0 + 1);
      if constexpr (x0 + 2 < x1) f(x0 + 2);
      static_assert(x1 - x0 <= 3, "pairs per slot");
    }
  };

  bf16x8 ring[kLead], vring[2][KB];
  // Operand of chunk i (0 .. 4 N - 1; 4 N .. : the next step's) of a step on buffer B.
  auto operand = [&](auto B, int i) {
    constexpr int cur = decltype(B)::value, prev = (cur + NBUF - 1) % NBUF, next = (cur + 1) % NBUF;
    if (i < N) return row_op(tile(cur, 0), i);
    if (i < 2 * N) return tr_op(tile(prev, 0), i - N);
    if (i < 3 * N) return row_op(tile(cur, 1), i - 2 * N);
    if (i < 4 * N) return tr_op(tile(cur, 1), i - 3 * N);
    return row_op(tile(next, 0), i - 4 * N);
  };
  auto v_op = [&](int ks, int kb) { return row_op(Vw + kb * 32 * 128, ks); };

  auto step = [&](auto B, int t) __attribute__((always_inline)) {
    constexpr int cur = decltype(B)::value, next = (cur + 1) % NBUF;
    for_constants(std::make_integer_sequence<int, 4 * N>{}, [&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value, ph = i / N, j = i % N;
      if (i == 3 * N) {
        // stage t + 1 has arrived: younger than its transfers (in A of the
        // previous step) are that step's 2 KB stores, stage t + 2's transfers
        // and this step's 2 KB stores
        // (operand reads stay in flight across the barrier: no buffer they
        // read is overwritten before the next one)
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NDMA + 1 + 4 * KB) : "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i == 0) mfma_operands();
      const bf16x8 av = ring[i % kLead];
      for_constants(std::make_integer_sequence<int, KB>{}, [&](auto KBI) __attribute__((always_inline)) {
        constexpr int kb = decltype(KBI)::value, sl = KB * j + kb;  // slot sl of the phase's KB N
        if constexpr (ph == 0 && j == 0)
          mfma_first(s[kb], av, kf[kb][0], stat);
        else if constexpr (ph == 0)
          mfma_v(s[kb], av, kf[kb][j]);
        else if constexpr (ph == 1)
          mfma_a(dk[j % DB][kb], av, __builtin_bit_cast(bf16x8, ds[kb][j / DB]));
        else if constexpr (ph == 2 && j == 0)
          mfma_first<KB == 1>(dp[kb], av, KB == 1 ? vf[0] : vring[0][kb], stat);
        else if constexpr (ph == 2)
          mfma_v<KB == 1>(dp[kb], av, KB == 1 ? vf[KB == 1 ? j : 0] : vring[j & 1][kb]);
        else
          mfma_a(dv[j % DB][kb], av, __builtin_bit_cast(bf16x8, pw[kb][j / DB]));
        if constexpr ((ph == 0 || ph == 2) && sl == KB) mfma_read(stat);
        if constexpr ((ph == 1 || ph == 3) && sl == 1) {  // two MFMAs behind S's, dP's last
#pragma unroll
          for (int b = 0; b < KB; ++b) mfma_done(ph == 1 ? s[b] : dp[b]);
        }
        if (kb == 0) {
          // operands ahead: the last chunks of a step read the next step's
          // stage, after the barrier
          ring[i % kLead] = operand(B, i + kLead);
        }
        if (KB == 2 && i >= 2 * N - 2 && i < 3 * N - 2) vring[i & 1][kb] = v_op(i + 2 - 2 * N, kb);
        if (kb == KB - 1) {
          if (ph == 1 && j == N - 2) load_stat(cur, 2);
          if (ph == 3 && j == N - 2) load_stat(next, 0);
        }
        if constexpr (ph == 0 && KB == 1) {
          // the pieces in this order, spread over the slots
          constexpr int kPieces = NDMA + 3;
          for_constants(std::make_integer_sequence<int, kPieces>{}, [&](auto P) __attribute__((always_inline)) {
            constexpr int p = decltype(P)::value;
            if constexpr (p * N / kPieces == sl) {
              if (p <= NDMA)
                issue(t + 2, t + 2, p);
              else
                ds_store(t - 1, 0, p - NDMA - 1);
            }
          });
        } else if constexpr (ph == 0) {
          if (sl <= NDMA) issue(t + 2, t + 2, sl);  // before the stores: the wait above counts on it
          if (N == 4 && sl == 2 * N - 2) {
            ds_store(t - 1, 0, 0);
            ds_store(t - 1, 0, 1);
          }
          if (N == 4 && sl == 2 * N - 1) {
            ds_store(t - 1, 1, 0);
            ds_store(t - 1, 1, 1);
          }
          if (N > 4 && sl >= 2 * N - 8 && sl % 2 == 0) ds_store(t - 1, (sl - (2 * N - 8)) / 4, (sl - (2 * N - 8)) / 2 % 2);
        } else if constexpr (ph == 3) {
          spread(std::integral_constant<int, sl>{}, std::integral_constant<int, KB * N>{}, std::integral_constant<int, 8 * KB>{}, ds_pair);
        } else {
          spread(std::integral_constant<int, (ph - 1) * KB * N + sl>{}, std::integral_constant<int, 2 * KB * N>{},
                 std::integral_constant<int, 8 * KB>{}, p_pair);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    // dS is due here, not in the next step's block
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int h = 0; h < 2; ++h) asm volatile("" : "+v"(ds[kb][h]));
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  load_stat(0, 0);
#pragma unroll
  for (int i = 0; i < kLead; ++i) ring[i] = operand(I0{}, i);
  // KB = 2: stages past the last one, which fill the round, add nothing (a way
  // out between the steps made the compiler move the accumulators about, which
  // take all the registers there).
  int t = 0;
  while (true) {  // a group has queries
    step(I0{}, t++);
    if (KB == 1 && t >= nst) break;
    step(I1{}, t++);
    if (KB == 1 && t >= nst) break;
    step(I2{}, t++);
    if (KB == 1 && t >= nst) break;
    step(I3{}, t++);
    if (t >= nst) break;
  }
  // dS of the last stage, and its dK
  const int last = KB == 1 ? (t - 1) & (NBUF - 1) : NBUF - 1;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int h = 0; h < 2; ++h) ds_store(t - 1, kb, h);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bf16x8 av = tr_op(tile(last, 0), i);
    mfma_operands();
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) mfma_a(dk[i % DB][kb], av, __builtin_bit_cast(bf16x8, ds[kb][i / DB]));
  }
  wait_vmcnt<0>();  // no transfer into this block's LDS outlives it
  // the last products have left the matrix core before the accumulators are
  // read, and each read is tied to its wait
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      asm volatile("s_nop 15" : "+a"(dk[db][kb]));
      asm volatile("s_nop 15" : "+a"(dv[db][kb]));
    }

#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int key = key0 + kb * 32;
    if (key < G.n_kv) {
      const int64_t off = static_cast<int64_t>(key) * ld + hoff + 4 * hh;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          f32x4 k4, v4;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            k4[i] = dk[db][kb][4 * jj + i] * a.scale;
            v4[i] = dv[db][kb][4 * jj + i];
          }
          *reinterpret_cast<f32x4*>(G.dk_ctx + off + db * 32 + 8 * jj) = k4;
          *reinterpret_cast<f32x4*>(G.dv_ctx + off + db * 32 + 8 * jj) = v4;
        }
    }
  }
}

// ------------------------------------------------------------------ scatter to the sources

// One thread per 16-byte output chunk of a source token; it adds, in group
// order, the context gradient of the row each group made from this token.
template <typename T>
__global__ __launch_bounds__(kPoolThreads) void scatter_kernel(ScatterArgs a) {
  constexpr int N = 16 / sizeof(T);
  typedef T vecT __attribute__((ext_vector_type(N)));
  const int b = blockIdx.x;
  int jn = 0;
  while (jn + 1 < a.n_jobs && b >= a.jobs[jn + 1].block_begin) ++jn;
  const ScatterJobArgs& J = a.jobs[jn];
  const int64_t cpt = a.chunks_per_tok;
  const int64_t ftok = static_cast<int64_t>(J.gh) * J.gw;
  const int64_t idx = static_cast<int64_t>(b - J.block_begin) * kPoolThreads + threadIdx.x;
  if (idx >= J.n_frames * ftok * cpt) return;
  const int64_t chunk = idx % cpt;
  const int64_t t = idx / cpt;
  const int x = static_cast<int>(t % J.gw);
  const int y = static_cast<int>((t / J.gw) % J.gh);
  const int64_t fr = t / ftok;
  const bool is_v = blockIdx.y != 0;
  float acc[N];
#pragma unroll
  for (int e = 0; e < N; ++e) acc[e] = 0.f;
  for (int g = 0; g < a.n_groups; ++g) {
    const ScatterGroupArgs& S = J.g[g];
    const int f = S.factor;
    if (a.pick_first && f > 1 && ((y % f) != 0 || (x % f) != 0)) continue;
    const int Y = y / f, X = x / f;
    const int ow = (J.gw + f - 1) / f;
    const float cnt = a.pick_first ? 1.f : static_cast<float>(min(f, J.gh - f * Y) * min(f, J.gw - f * X));
    const float* src = (is_v ? a.ctx_v[g] : a.ctx_k[g]) +
                       (S.ctx_begin + fr * S.frame_stride + static_cast<int64_t>(Y) * ow + X) * a.ld + chunk * N;
#pragma unroll
    for (int e = 0; e < N; e += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + e);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[e + i] += v[i] / cnt;
    }
  }
  vecT o;
#pragma unroll
  for (int e = 0; e < N; ++e) o[e] = static_cast<T>(acc[e]);
  T* dst = static_cast<T*>(is_v ? J.dst_v : J.dst_k);
  *reinterpret_cast<vecT*>(dst + (fr * ftok + static_cast<int64_t>(y) * J.gw + x) * a.ld + chunk * N) = o;
}

}  // namespace

hipError_t launch_bwd_dot(const DotArgs& a, bool bf16, hipStream_t stream) {
  const int64_t rows = static_cast<int64_t>(a.n_q) * a.num_heads;
  if (rows == 0) return hipSuccess;
  if (a.ld != static_cast<int64_t>(a.num_heads) * a.head_dim) return hipErrorInvalidValue;
  const int64_t threads = rows * (a.head_dim * (bf16 ? 2 : 4) / 16);
  if ((threads + kDotThreads - 1) / kDotThreads > 0x7fffffff) return hipErrorInvalidValue;
  const int blocks = static_cast<int>((threads + kDotThreads - 1) / kDotThreads);
  if (bf16)
    hipLaunchKernelGGL(dot_kernel<__bf16>, dim3(blocks), dim3(kDotThreads), 0, stream, a);
  else
    hipLaunchKernelGGL(dot_kernel<float>, dim3(blocks), dim3(kDotThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_bwd(const BwdArgs& a, int dq_blocks, int kv_blocks, int head_dim, bool bf16,
                      hipStream_t stream) {
  if (!bf16) return launch_bwd_f32(a, dq_blocks, kv_blocks, head_dim, stream);
  // dK/dV first: it writes the dS tiles the dQ kernel reads.
  if (kv_blocks > 0) {
    auto go = [&](auto d, auto qs, auto kb) {
      hipLaunchKernelGGL((dkdv_kernel<decltype(d)::value, decltype(qs)::value, decltype(kb)::value>), dim3(kv_blocks),
                         dim3(kBwdKVThreads), 0, stream, a);
    };
    auto pick = [&](auto d, auto qs) {
      if (a.kv_keys == kBwdKVKeys)
        go(d, qs, std::integral_constant<int, 1>{});
      else
        go(d, qs, std::integral_constant<int, 2>{});
    };
    if (a.kv_keys != kBwdKVKeys && a.kv_keys != 2 * kBwdKVKeys) return hipErrorInvalidValue;
    if (head_dim == 128 && a.q_prescaled)
      pick(std::integral_constant<int, 128>{}, std::true_type{});
    else if (head_dim == 128)
      pick(std::integral_constant<int, 128>{}, std::false_type{});
    else if (a.q_prescaled)
      pick(std::integral_constant<int, 64>{}, std::true_type{});
    else
      pick(std::integral_constant<int, 64>{}, std::false_type{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (dq_blocks > 0) {
    BwdArgs d = a;
    d.dq_blocks = dq_blocks;
    int splits = 1;
    int64_t sums = 0;
    for (int g = 0; g < d.n_groups; ++g) {
      const BwdGroupArgs& G = d.groups[g];
      // a split's sum lies in the dS tiles of its stages
      if (G.dq_splits < 1 || (G.dq_splits > 1 && G.ds_stages / G.dq_splits < head_dim / 32)) return hipErrorInvalidValue;
      splits = G.dq_splits > splits ? G.dq_splits : splits;
      if (G.dq_splits > 1) sums += static_cast<int64_t>((G.q_end - G.q_begin + 31) / 32) * d.num_heads;
    }
    const int64_t grid = static_cast<int64_t>(dq_blocks) * splits;
    if (grid > 0x7fffffff || sums > 0x7fffffff) return hipErrorInvalidValue;
    if (head_dim == 128)
      hipLaunchKernelGGL(dq_kernel<128>, dim3(static_cast<uint32_t>(grid)), dim3(kBwdQThreads), 0, stream, d);
    else
      hipLaunchKernelGGL(dq_kernel<64>, dim3(static_cast<uint32_t>(grid)), dim3(kBwdQThreads), 0, stream, d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || sums == 0) return e;
    if (head_dim == 128)
      hipLaunchKernelGGL(dq_sum_kernel<128>, dim3(static_cast<uint32_t>(sums)), dim3(256), 0, stream, d);
    else
      hipLaunchKernelGGL(dq_sum_kernel<64>, dim3(static_cast<uint32_t>(sums)), dim3(128), 0, stream, d);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t launch_scatter(const ScatterArgs& a, int n_blocks, bool bf16, hipStream_t stream) {
  if (n_blocks <= 0) return hipSuccess;
  const dim3 grid(n_blocks, 2), block(kPoolThreads);
  if (bf16)
    hipLaunchKernelGGL(scatter_kernel<__bf16>, grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL(scatter_kernel<float>, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace mssa
