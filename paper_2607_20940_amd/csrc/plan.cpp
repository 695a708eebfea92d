// Static MSSA plan (host).  Every table follows Sec. 4.1 of Ms. Forcing:
// MSP grids from Eq. 3 (ceil grid when a scale does not divide the native
// grid), query groups per distinct scale, and the Eq. 4 context of each
// query scale s:
//   sink frames        native, never resampled;
//   history frames     native, pooled by s;
//   window frame of b  at max(s, p_b), pooled by max(1, s / p_b);
// in the order sink, history (oldest first), window (state 1..T).
#include "plan.hpp"

#include "kernel_args.hpp"

#include <algorithm>
#include <cmath>
#include <limits>
#include <map>

namespace mssa {
namespace {

bool is_pow2(int32_t x) { return x > 0 && (x & (x - 1)) == 0; }

int32_t ceil_div(int32_t a, int32_t b) { return (a + b - 1) / b; }

int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

// Partial records and range table of n tile ranges of the persistent forward.
int64_t range_records(const Plan& p, int64_t n) {
  return n > 1 ? align256(2 * n * partial_record_floats(p.desc.head_dim) * 4) + align256((n + 1) * 8) : 0;
}

// 32-query items, and the records of s blocks for each of them.
int64_t items_32q(const Plan& p) {
  int64_t n = 0;
  for (const QGroup& g : p.groups) n += int64_t{ceil_div(g.q_end - g.q_begin, kFwdF32BM)} * p.desc.num_heads;
  return n;
}
int64_t split_records(const Plan& p, int64_t s) {
  return s > 1 ? align256(items_32q(p) * s * split_record_floats(p.desc.head_dim) * 4) : 0;
}

// Blocks of one cost (microseconds), and the time of blocks dealt out in this
// order over an XCD's CUs, one at a time on each.
constexpr int64_t kXcds = 8;
struct BlockRun {
  int64_t n;
  double cost;
};
double dealt_out(const std::vector<BlockRun>& runs, int64_t cus) {
  cus = std::max<int64_t>(1, cus);
  std::map<double, int64_t> busy{{0.0, cus}};  // CUs by the time they are free
  double rounds = 0;                           // of whole rounds, on top of it
  for (const BlockRun& r : runs) {
    int64_t left = r.n;
    if (left >= 2 * cus) {
      rounds += r.cost * static_cast<double>(left / cus - 1);
      left = left % cus + cus;
    }
    while (left > 0) {
      const auto [t, free] = *busy.begin();
      const int64_t k = std::min(left, free);
      busy.erase(busy.begin());
      if (free > k) busy[t] += free - k;
      busy[t + r.cost] += k;
      left -= k;
    }
  }
  return rounds + busy.rbegin()->first;
}

// Blocks of a grid of which every XCD has a contiguous eighth: the slowest XCD.
double dealt_in_eighths(const std::vector<BlockRun>& runs, int64_t cus) {
  int64_t blocks = 0;
  for (const BlockRun& r : runs) blocks += r.n;
  double worst = 0;
  for (int64_t x = 0; x < kXcds; ++x) {
    const int64_t lo = blocks * x / kXcds, hi = blocks * (x + 1) / kXcds;
    std::vector<BlockRun> mine;
    int64_t first = 0;
    for (const BlockRun& r : runs) {
      mine.push_back({std::min(hi, first + r.n) - std::max(lo, first), r.cost});
      first += r.n;
    }
    worst = std::max(worst, dealt_out(mine, cus / kXcds));
  }
  return worst;
}

// How a bf16 forward runs when the caller does not say: `splits` blocks per
// 32-query item of fwd_small_kernel, or 0 for the persistent 256-query kernel
// on `ranges` tile ranges.
struct FwdChoice {
  int32_t splits;
  int64_t ranges;
};

// The fastest of three schedules by times fitted on an MI355X (microseconds,
// forward alone) over 310 layers of 1 to 57 heads of 64 and 128 and 2e8 to 4e11
// FLOP: 5 to 7 % rms off each schedule's time, the choice 0.14 % above the best
// of all schedules on average and 7 % at worst.
// - Small kernel: blocks of c0 + c1 per step of eight 32-key tiles, dealt out
//   longest first, c1 up by cx where every CU streams K/V; merging S blocks of
//   an item adds m0 + m1 S.
// - Persistent kernel, one range per CU of two tiles at least: p0, pr for the
//   records of a range per CU, p1 per tile of a range and p2 per piece of the
//   longest item.
// - Persistent kernel, whole items, no records and no merge, where the items
//   are equally long and no more than the CUs: u0 and, per tile, u1 + u2 items
//   (the clock falls as CUs fill).
// - A merge is one more launch, 3.4 us of the host, and below some length a
//   program that launches pass by pass (here through the Python binding) is bound
//   by the host: a merging schedule counts as no shorter than `host` + 3.4 (the
//   shorter of two such on the device is taken).  That leaves out splits that save
//   less than the launch costs (3 heads of 64, 588 queries on 2352 keys, streamed:
//   16.3 us a layer, 18.9 split in four).  Of 148 small layers launched so the
//   choice is 0.2 % (passes) and 0.4 % (streamed) above the best split on average,
//   15 % and 11 % at worst; without this 1.4, 3.7, 17 and 20 %.
// A schedule has to be better than those before it by 3 %.
// Measured, small S = 1, 2, 4 / one range per CU / whole items: 2 heads of 128
// on 270 queries and 4372 keys (and fewer at 2x and 4x) 23.8, 19.7, 16.4 /
// 41.3 / 74.9 us; 1 head of 64 on 792 and 14256 58.4, 36.0, 24.2 / 48.1 / 181;
// 18 heads of 128 on 3168 and 3520 166, 205, 264 / 111 / 95.8; 39 heads of 128
// on 1500 and 1875 111, 153, 228 / 76.2 / 59.9; 50 heads of 128 on 768 and 3072
// (150 items) - / 78.6 / 74.5, on 768 and 6144 - / 123 / 131.
// fits: may a schedule's records of that many bytes be had?
template <class Fits>
FwdChoice forward_choice(const Plan& p, const std::vector<std::vector<int64_t>>& run_tok, const Schedule& sc,
                         int64_t n_items, int64_t cus, Fits&& fits) {
  struct Fit {
    double a, c0, c1, cx, m0, m1, p0, pr, p1, p2, u0, u1, u2;
  };
  const Fit f = p.desc.head_dim == 128
                    ? Fit{2.1, 4.6, 1.04, 0.25, 3.1, 0.59, 14.0, 12.6, 1.745, 0.44, 15.0, 0.96, 0.0023}
                    : Fit{2.6, 3.25, 0.89, 0.08, 2.3, 0.46, 9.6, 10.6, 1.14, 0.40, 11.7, 0.91, 0.0005};
  constexpr double kLaunch = 3.4;
  const double host = p.head_ring ? 15.0 : p.hist_ring ? 20.0 : 12.5;
  const double n_cus = static_cast<double>(cus);
  const int32_t longest = *std::max_element(sc.tiles_per_item.begin(), sc.tiles_per_item.end());
  const bool equal = *std::min_element(sc.tiles_per_item.begin(), sc.tiles_per_item.end()) == longest;
  FwdChoice best{0, std::min<int64_t>(cus, std::max<int64_t>(n_items, sc.total_tiles / 2))};
  if (!fits(range_records(p, std::min(best.ranges, sc.total_tiles)))) best.ranges = std::min<int64_t>(cus, n_items);
  const double ranges = static_cast<double>(std::max<int64_t>(1, std::min(best.ranges, sc.total_tiles)));
  const double share = std::max(1.0, static_cast<double>(sc.total_tiles) / ranges);  // tiles of a range
  double on_device = f.p0 + f.pr * ranges / n_cus + f.p1 * share + f.p2 * longest / share;
  double t_best = std::max(on_device, host + kLaunch);
  bool merges = true;
  if (equal && n_items <= cus) {
    const double t = f.u0 + longest * (f.u1 + f.u2 * static_cast<double>(n_items));
    if (t < t_best) {
      best.ranges = n_items;
      t_best = on_device = t;
      merges = false;
    }
  }
  for (int32_t s = 1; s <= 8; s *= 2) {
    if (!fits(split_records(p, s))) break;
    std::vector<BlockRun> runs;
    double blocks = 0, sum = 0;
    for (int g : p.order)
      runs.push_back({int64_t{ceil_div(p.groups[g].q_end - p.groups[g].q_begin, kFwdF32BM)} * p.desc.num_heads * s, 0.0});
    for (const BlockRun& r : runs) blocks += static_cast<double>(r.n);
    const double step = f.c1 * (1.0 + f.cx * std::min(1.0, blocks / n_cus));
    for (size_t i = 0; i < runs.size(); ++i) {
      int64_t tiles = 0;
      for (int64_t n : run_tok[p.order[i]]) tiles += (n + 31) / 32;
      runs[i].cost = f.c0 + step * static_cast<double>((tiles + kSplitWaves * s - 1) / (kSplitWaves * s));
      sum += static_cast<double>(runs[i].n) * runs[i].cost;
    }
    const double fixed = f.a + (s > 1 ? f.m0 + f.m1 * s : 0.0);
    if (fixed + sum / n_cus >= t_best) continue;  // (also keeps the dealing short)
    const double dealt = fixed + dealt_in_eighths(runs, cus), t = s > 1 ? std::max(dealt, host + kLaunch) : dealt;
    if (1.03 * t < t_best || (merges && t <= t_best && 1.03 * dealt < on_device)) {
      best.splits = s;
      t_best = t;
      on_device = dealt;
      merges = s > 1;
    }
  }
  return best;
}

// Keys per block of the bf16 dK/dV kernel: 128 (32 a wave) where there are few
// blocks or few queries, else 256 (64 a wave: two MFMAs per operand read).  The
// faster one by times fitted on an MI355X over 150 layers of 1 to 40 heads and
// 1e8 to 1.5e12 FLOP: a block costs its start and its 32-query steps, which with
// 64 keys a wave run in fours; each XCD has an eighth of every group's blocks.
// Backward with 128 / 256 keys: 13 heads of 128, 108 queries on 489 keys and two
// small groups 41.3 / 53.3 us; 3 heads of 64, 1275 on 5341 and two groups 66.8 /
// 80.3; 14 heads of 64, 832 on 4160 87.4 / 81.4; 3 heads of 128, 6048 on 11088
// 401 / 336.  The choice was 2.4 % above the better one at worst.
int32_t kv_block_keys(const Plan& p, int64_t cus) {
  const bool d128 = p.desc.head_dim == 128;
  double best = 0;
  int32_t keys = 0;
  for (int32_t kb = 1; kb <= 2; ++kb) {
    const double start = kb == 1 ? (d128 ? 8.0 : 4.4) : (d128 ? 16.9 : 9.1);
    const double step = kb == 1 ? (d128 ? 0.59 : 0.435) : (d128 ? 0.96 : 0.657);
    std::vector<BlockRun> runs;
    for (int g : p.order) {
      const int64_t n = (p.groups[g].n_kv + kb * kBwdKVKeys - 1) / (kb * kBwdKVKeys) * p.bwd_ds_heads;
      int64_t steps = ceil_div(p.groups[g].q_end - p.groups[g].q_begin, kBwdStage);
      if (kb == 2) steps = (steps + 3) / 4 * 4;
      runs.push_back({(n + kXcds - 1) / kXcds, start + step * static_cast<double>(steps)});
    }
    const double t = dealt_out(runs, cus / kXcds);
    if (keys == 0 || t < best) {
      best = t;
      keys = kb * kBwdKVKeys;
    }
  }
  return keys;
}

}  // namespace

mssa_status build_plan(const mssa_plan_desc& d, int slots, int attention_blocks, Plan& p, std::string& err) {
  const int32_t T = d.num_states;
  if (T < 1 || T > MSSA_MAX_STATES) {
    err = "num_states must be in [1, " + std::to_string(MSSA_MAX_STATES) + "]";
    return MSSA_ERR_INVALID_ARG;
  }
  if (d.grid_h < 1 || d.grid_w < 1 || d.grid_h > 65536 || d.grid_w > 65536) {
    err = "grid_h and grid_w must be in [1, 65536]";
    return MSSA_ERR_INVALID_ARG;
  }
  if (d.frames_per_state < 1 || d.sink_frames < 0 || d.hist_frames < 0) {
    err = "frames_per_state must be >= 1, sink_frames and hist_frames >= 0";
    return MSSA_ERR_INVALID_ARG;
  }
  if (d.num_heads < 1) {
    err = "num_heads must be >= 1";
    return MSSA_ERR_INVALID_ARG;
  }
  if (d.dtype != MSSA_BF16 && d.dtype != MSSA_F32) {
    err = "dtype must be MSSA_BF16 or MSSA_F32";
    return MSSA_ERR_INVALID_ARG;
  }
  if (!std::isfinite(d.softmax_scale)) {
    err = "softmax_scale must be finite";
    return MSSA_ERR_INVALID_ARG;
  }
  if ((d.flags & ~(MSSA_PLAN_POOLED_HIST_RING | MSSA_PLAN_STRIDED_SUBSAMPLE | MSSA_PLAN_HEAD_IN_RING |
                   MSSA_PLAN_Q_PRESCALED)) != 0) {
    err = "unknown plan flags";
    return MSSA_ERR_INVALID_ARG;
  }
  for (int l = 0; l < T; ++l) {
    if (!is_pow2(d.scales[l]) || d.scales[l] > 64) {
      err = "scales must be powers of two in [1, 64]";
      return MSSA_ERR_UNSUPPORTED;
    }
    if (l > 0 && d.scales[l] < d.scales[l - 1]) {
      err = "scales must be nondecreasing (coarser patches for noisier states)";
      return MSSA_ERR_UNSUPPORTED;
    }
  }
  if (d.head_dim != 64 && d.head_dim != 128) {
    err = "head_dim must be 64 or 128";
    return MSSA_ERR_UNSUPPORTED;
  }
  if ((d.flags & MSSA_PLAN_HEAD_IN_RING) &&
      (!(d.flags & MSSA_PLAN_POOLED_HIST_RING) || d.scales[0] != 1 || d.dtype != MSSA_BF16)) {
    err = "MSSA_PLAN_HEAD_IN_RING needs MSSA_PLAN_POOLED_HIST_RING, a native head state (scales[0] == 1) and bf16";
    return MSSA_ERR_UNSUPPORTED;
  }

  p = Plan{};
  p.desc = d;
  p.hist_ring = (d.flags & MSSA_PLAN_POOLED_HIST_RING) != 0;
  p.head_ring = (d.flags & MSSA_PLAN_HEAD_IN_RING) != 0;
  p.strided = (d.flags & MSSA_PLAN_STRIDED_SUBSAMPLE) != 0;
  p.q_prescaled = (d.flags & MSSA_PLAN_Q_PRESCALED) != 0;
  p.softmax_scale = d.softmax_scale > 0.f ? d.softmax_scale
                                          : 1.0f / std::sqrt(static_cast<float>(d.head_dim));
  const int32_t F = d.frames_per_state;
  auto tok_at = [&](int32_t s) {
    return static_cast<int64_t>(ceil_div(d.grid_h, s)) * ceil_div(d.grid_w, s);
  };
  p.tok1 = tok_at(1);
  p.ld = static_cast<int64_t>(d.num_heads) * d.head_dim;
  p.elem_bytes = d.dtype == MSSA_BF16 ? 2 : 4;
  p.n_sink_tok = p.tok1 * d.sink_frames;
  p.n_hist_tok = p.tok1 * d.hist_frames;
  p.win_shift = p.head_ring ? p.tok1 * F : 0;

  // GRID: native scale plus every scheduled scale, ascending.
  std::vector<int32_t> sc{1};
  for (int l = 0; l < T; ++l) sc.push_back(d.scales[l]);
  std::sort(sc.begin(), sc.end());
  sc.erase(std::unique(sc.begin(), sc.end()), sc.end());
  for (int32_t s : sc)
    p.grids.push_back({s, ceil_div(d.grid_h, s), ceil_div(d.grid_w, s), static_cast<int32_t>(tok_at(s))});

  // Window frames in token order and the query groups (contiguous per scale
  // because the schedule is nondecreasing).
  struct WinFrame { int32_t w, p; int64_t first, n; };
  std::vector<WinFrame> wf;
  int64_t pos = 0;
  for (int l = 0; l < T; ++l)
    for (int f = 0; f < F; ++f) {
      const int64_t n = tok_at(d.scales[l]);
      wf.push_back({l * F + f, d.scales[l], pos, n});
      pos += n;
    }
  p.n_q = pos;
  for (const WinFrame& w : wf) {
    if (!p.groups.empty() && p.groups.back().scale == w.p)
      p.groups.back().q_end = static_cast<int32_t>(w.first + w.n);
    else
      p.groups.push_back({w.p, static_cast<int32_t>(w.first), static_cast<int32_t>(w.first + w.n), 0});
  }

  const int64_t kIdxMax = std::numeric_limits<int32_t>::max();
  if (p.n_q > kIdxMax || p.n_sink_tok > kIdxMax || p.n_hist_tok > kIdxMax) {
    err = "token counts exceed 32-bit indexing";
    return MSSA_ERR_UNSUPPORTED;
  }

  // SEG rows per group, their placement, runs and pool jobs.
  const int G = static_cast<int>(p.groups.size());
  p.runs.assign(G, {});
  p.pooled_tokens.assign(G, 0);
  p.pooled_k_off.assign(G, 0);
  p.pooled_v_off.assign(G, 0);
  p.pairs_per_head = 0;
  int64_t ws = 0;
  std::vector<char> win_read(wf.size(), 0);
  bool hist_read = false;

  for (int g = 0; g < G; ++g) {
    QGroup& grp = p.groups[g];
    const int32_t s = grp.scale;
    int64_t kv = 0, pooled = 0;
    std::vector<SegRow> rows;
    for (int f = 0; f < d.sink_frames; ++f)
      rows.push_back({s, kSink, f, 1, 1, 1, static_cast<int32_t>(p.tok1), 0, kBufSink, f * p.tok1});
    for (int f = 0; f < d.hist_frames; ++f) {
      SegRow r{s, kHist, f, 1, s, s, static_cast<int32_t>(tok_at(s)), 0, kBufHist, f * p.tok1};
      if (s > 1 && p.hist_ring) {
        r.buffer = kBufHistPooled;
        r.tok_offset = f * r.n_tok;
      } else if (s > 1) {
        r.buffer = kBufPooled;
        r.tok_offset = pooled;
        pooled += r.n_tok;
        hist_read = true;
      }
      rows.push_back(r);
    }
    for (size_t i = 0; i < wf.size(); ++i) {
      const WinFrame& w = wf[i];
      const int32_t eff = std::max(s, w.p);
      const int32_t fac = std::max(1, s / w.p);
      SegRow r{s, kWin, w.w, w.p, eff, fac, static_cast<int32_t>(tok_at(eff)), 0, kBufWin, w.first - p.win_shift};
      if (p.head_ring && w.w < F) {
        // state 1 lives in the spare ring slots, pooled there by pool_kv
        r.buffer = kBufRingHead;
        r.tok_offset = w.w * r.n_tok;
      } else if (fac > 1) {
        r.buffer = kBufPooled;
        r.tok_offset = pooled;
        pooled += r.n_tok;
        win_read[i] = 1;
      }
      rows.push_back(r);
    }
    for (SegRow& r : rows) { r.kv_begin = kv; kv += r.n_tok; }
    if (kv > kIdxMax) {
      err = "context length exceeds 32-bit indexing";
      return MSSA_ERR_UNSUPPORTED;
    }
    grp.n_kv = kv;
    p.pairs_per_head += static_cast<int64_t>(grp.q_end - grp.q_begin) * kv;

    // Runs: merge rows that are contiguous in one buffer.
    for (const SegRow& r : rows) {
      std::vector<Run>& rs = p.runs[g];
      if (!rs.empty() && rs.back().buffer == r.buffer &&
          rs.back().tok_offset + rs.back().n_tok == r.tok_offset)
        rs.back().n_tok += r.n_tok;
      else
        rs.push_back({r.buffer, r.tok_offset, r.n_tok});
    }

    // Pool jobs: merge consecutive pooled rows of one source kind, source
    // scale and factor whose source and destination frames are contiguous.
    for (const SegRow& r : rows) {
      if (r.buffer != kBufPooled) continue;
      const int32_t src_buf = r.kind == kHist ? kBufHist : kBufWin;
      int64_t src_tok;
      int64_t src_n;
      if (r.kind == kHist) {
        src_tok = r.frame * p.tok1;
        src_n = p.tok1;
      } else {
        src_tok = wf[r.frame].first - p.win_shift;
        src_n = wf[r.frame].n;
      }
      const int32_t sgh = ceil_div(d.grid_h, r.src_scale), sgw = ceil_div(d.grid_w, r.src_scale);
      if (!p.pool_jobs.empty()) {
        PoolJob& j = p.pool_jobs.back();
        const int64_t jsrc_n = static_cast<int64_t>(j.src_gh) * j.src_gw;
        const int64_t jdst_n = static_cast<int64_t>(j.dst_gh) * j.dst_gw;
        if (j.group == g && j.buffer == src_buf && j.factor == r.factor && j.src_gh == sgh &&
            j.src_gw == sgw && j.src_tok + j.n_frames * jsrc_n == src_tok &&
            j.dst_tok + j.n_frames * jdst_n == r.tok_offset) {
          j.n_frames += 1;
          continue;
        }
      }
      (void)src_n;
      p.pool_jobs.push_back({g, src_buf, src_tok, sgh, sgw, r.factor, 1,
                             ceil_div(sgh, r.factor), ceil_div(sgw, r.factor), r.tok_offset});
    }

    p.pooled_tokens[g] = pooled;
    if (pooled > 0) {
      const int64_t bytes = align256(pooled * p.ld * p.elem_bytes);
      p.pooled_k_off[g] = ws;
      ws += bytes;
      p.pooled_v_off[g] = ws;
      ws += bytes;
    }
    for (SegRow& r : rows) p.segs.push_back(r);
  }
  // Persistent attention schedule: items (group, head, query tile) in launch
  // order, each a sequence of 64-key tiles over the group's runs.
  for (int g = 0; g < G; ++g) p.order.push_back(g);
  std::stable_sort(p.order.begin(), p.order.end(),
                   [&](int x, int y) { return p.groups[x].n_kv > p.groups[y].n_kv; });
  std::vector<std::vector<int64_t>> run_tok(G);
  int64_t n_items = 0;
  for (int g = 0; g < G; ++g) {
    for (const Run& r : p.runs[g]) run_tok[g].push_back(r.n_tok);
    n_items += static_cast<int64_t>((p.groups[g].q_end - p.groups[g].q_begin + kFwdBM - 1) / kFwdBM) * d.num_heads;
  }
  p.n_ranges = 1;
  const Schedule whole = make_schedule(p, run_tok);
  const int64_t total = whole.total_tiles;
  if (slots <= 0) slots = 512;
  // Workspace after the pooled blocks.  Where there is a choice of schedule,
  // one whose records would push a plan past the scratch of the entry point
  // without allocations is passed over if another one fits.
  const int64_t room = MSSA_NOALLOC_SCRATCH_BYTES - ws;
  auto fits = [&](int64_t bytes) { return room < 0 || bytes <= room; };
  p.partial_off = ws;
  p.range_table_off = 0;
  if (d.dtype == MSSA_F32) {
    // The eight waves of a block take 32-key tiles in turn; a context is
    // split over several blocks while that leaves every wave a tile and the
    // items alone leave CUs idle.
    int64_t tiles = 0;
    for (int g = 0; g < G; ++g) {
      int64_t t = 0;
      for (const Run& r : p.runs[g]) t += (r.n_tok + 31) / 32;
      tiles = std::max(tiles, t);
    }
    int64_t s = std::max<int64_t>(1, std::min(slots / items_32q(p), (tiles + kSplitWaves - 1) / kSplitWaves));
    if (!fits(split_records(p, s))) s = 1;
    p.key_splits = static_cast<int32_t>(s);
    p.partial_bytes = split_records(p, s);
  } else {
    FwdChoice c{0, attention_blocks};
    if (attention_blocks <= 0) c = forward_choice(p, run_tok, whole, n_items, slots, fits);
    p.key_splits = c.splits;
    p.n_ranges = c.splits > 0 ? 1 : static_cast<int32_t>(std::max<int64_t>(1, std::min(c.ranges, total)));
    p.partial_bytes = c.splits > 0 ? split_records(p, c.splits) : range_records(p, p.n_ranges);
    if (p.n_ranges > 1) p.range_table_off = ws + p.partial_bytes - align256((static_cast<int64_t>(p.n_ranges) + 1) * 8);
  }
  p.sched = make_schedule(p, run_tok);
  ws += p.partial_bytes;
  p.workspace_bytes = ws;

  // Backward workspace and the scatter of context gradients to the sources.
  // dS of whole heads per launch within the budget, at least one head.
  p.bwd_ds_stages.assign(G, 0);
  p.bwd_ds_qblocks.assign(G, 0);
  p.bwd_dq_splits.assign(G, 1);
  p.bwd_ds_heads = d.num_heads;
  if (d.dtype == MSSA_BF16) {
    int64_t per_head = 0, longest = 0;
    for (int g = 0; g < G; ++g) {
      int64_t stages = 0;
      for (const Run& r : p.runs[g]) stages += (r.n_tok + kBwdKS - 1) / kBwdKS;
      const int64_t nq = p.groups[g].q_end - p.groups[g].q_begin;
      const int64_t qblocks = 2 * ((nq + kBwdQS - 1) / kBwdQS);
      // the dK/dV kernel addresses the tiles of a 32-query block by buffer
      // offsets, and points what it does not store past their range
      if (stages * kBwdKS * 64 > int64_t{kPastEnd} || qblocks > 0x7fffffff) {
        err = "backward dS buffer too large";
        return MSSA_ERR_UNSUPPORTED;
      }
      p.bwd_ds_stages[g] = static_cast<int32_t>(stages);
      p.bwd_ds_qblocks[g] = static_cast<int32_t>(qblocks);
      per_head += qblocks * stages * kBwdKS * 32 * 2;
      longest = std::max(longest, stages);
    }
    p.bwd_ds_heads = static_cast<int32_t>(
        std::max<int64_t>(1, std::min<int64_t>(d.num_heads, kBwdDsBudget / std::max<int64_t>(1, per_head))));
    p.bwd_kv_keys = kv_block_keys(p, slots);
    // dQ of a layer with few 256-query blocks: splits of at least six 64-key
    // stages of the longest context, and of enough stages of the group's own
    // for a split's sum to lie in their dS tiles.
    const int64_t splits = std::max<int64_t>(1, std::min({slots / n_items, longest / 6, int64_t{8}}));
    for (int g = 0; g < G; ++g)
      p.bwd_dq_splits[g] = static_cast<int32_t>(
          std::max<int64_t>(1, std::min<int64_t>(splits, p.bwd_ds_stages[g] / (d.head_dim / 32))));
  }
  ws = align256(ws);
  p.bwd_dsum_off = ws;
  ws += align256(static_cast<int64_t>(d.num_heads) * p.n_q * 4);
  p.bwd_lse2_off = ws;
  ws += align256(static_cast<int64_t>(d.num_heads) * p.n_q * 4);
  p.bwd_dk_off.assign(G, 0);
  p.bwd_dv_off.assign(G, 0);
  for (int g = 0; g < G; ++g) {
    const int64_t bytes = align256(p.groups[g].n_kv * p.ld * 4);
    p.bwd_dk_off[g] = ws;
    ws += bytes;
    p.bwd_dv_off[g] = ws;
    ws += bytes;
  }
  p.bwd_ds_off.assign(G, 0);
  if (d.dtype == MSSA_BF16)
    for (int g = 0; g < G; ++g) {
      p.bwd_ds_off[g] = ws;
      ws += align256(static_cast<int64_t>(p.bwd_ds_heads) * p.bwd_ds_qblocks[g] * p.bwd_ds_stages[g] * kBwdKS * 32 * 2);
    }
  p.bwd_workspace_bytes = ws;
  auto seg_of = [&](int g, int32_t kind, int32_t frame) -> const SegRow& {
    for (const SegRow& r : p.segs)
      if (r.q_scale == p.groups[g].scale && r.kind == kind && r.frame == frame) return r;
    return p.segs.front();  // unreachable: every source frame is in every context
  };
  bool scatter_ok = true;
  auto add_job = [&](int32_t buffer, int32_t kind, int32_t frame0, int64_t src_tok, int32_t n_frames,
                     int32_t src_scale) {
    ScatterJob j;
    j.buffer = buffer;
    j.src_tok = src_tok;
    j.n_frames = n_frames;
    j.gh = ceil_div(d.grid_h, src_scale);
    j.gw = ceil_div(d.grid_w, src_scale);
    for (int g = 0; g < G; ++g) {
      const SegRow& r = seg_of(g, kind, frame0);
      j.ctx_begin.push_back(r.kv_begin);
      j.frame_stride.push_back(r.n_tok);
      j.factor.push_back(r.factor);
      // a resampled frame has ceil(gh / f) x ceil(gw / f) tokens, and the
      // job's frames lie inside the context
      scatter_ok &= r.kind == kind && r.frame == frame0 &&
                    static_cast<int64_t>(ceil_div(j.gh, r.factor)) * ceil_div(j.gw, r.factor) == r.n_tok &&
                    r.kv_begin + static_cast<int64_t>(n_frames) * r.n_tok <= p.groups[g].n_kv;
    }
    p.scatter_jobs.push_back(j);
  };
  if (d.sink_frames > 0) add_job(kBufSink, kSink, 0, 0, d.sink_frames, 1);
  if (d.hist_frames > 0) add_job(kBufHist, kHist, 0, 0, d.hist_frames, 1);
  for (size_t i = 0; i < wf.size();) {
    size_t e = i;
    while (e < wf.size() && wf[e].p == wf[i].p) ++e;
    add_job(kBufWin, kWin, wf[i].w, wf[i].first, static_cast<int32_t>(e - i), wf[i].p);
    i = e;
  }
  if (!scatter_ok) {
    err = "internal: inconsistent gradient scatter tables";
    return MSSA_ERR_UNSUPPORTED;
  }

  // Algorithmic pool traffic, K and V: block mean, each pooled source frame
  // read once and each pooled frame written once; stride, each pooled token
  // reads the one source token it copies.
  int64_t write_tok = 0;
  for (int64_t t : p.pooled_tokens) write_tok += t;
  int64_t read_tok = hist_read ? p.n_hist_tok : 0;
  for (size_t i = 0; i < wf.size(); ++i)
    if (win_read[i]) read_tok += wf[i].n;
  if (p.head_ring) {
    // state 1's frames, read once from the ring and written pooled to every
    // coarser query scale's ring
    bool any = false;
    for (const QGroup& g : p.groups)
      if (g.scale > 1) {
        write_tok += F * tok_at(g.scale);
        any = true;
      }
    if (any) read_tok += F * p.tok1;
  }
  if (p.strided) read_tok = write_tok;
  p.pool_bytes_alg = 2 * (read_tok + write_tok) * p.ld * p.elem_bytes;
  return MSSA_OK;
}

Schedule make_schedule(const Plan& p, const std::vector<std::vector<int64_t>>& n_tok) {
  const int G = static_cast<int>(p.groups.size());
  Schedule sc;
  sc.tiles_per_item.assign(G, 0);
  sc.tile_begin.assign(G, 0);
  int64_t n_items = 0, t_max = 0;
  std::vector<int64_t> item_first(G, 0);
  for (int g : p.order) {
    int64_t tiles = 0;
    for (int64_t n : n_tok[g]) tiles += (n + kFwdBN - 1) / kFwdBN;
    sc.tiles_per_item[g] = static_cast<int32_t>(tiles);
    sc.tile_begin[g] = sc.total_tiles;
    item_first[g] = n_items;
    const int64_t items =
        static_cast<int64_t>((p.groups[g].q_end - p.groups[g].q_begin + kFwdBM - 1) / kFwdBM) * p.desc.num_heads;
    n_items += items;
    sc.total_tiles += items * tiles;
    t_max = std::max(t_max, tiles);
  }
  const int64_t ranges = p.n_ranges;
  // Whole-item rounds: as many as fit without any block exceeding its even
  // share total_tiles / ranges; the rest is split into per-block tail ranges
  // sized to make every block's total equal.
  sc.dp_rounds = static_cast<int32_t>(
      std::min<int64_t>(n_items / ranges, (sc.total_tiles / ranges) / std::max<int64_t>(1, t_max)));
  const int64_t i = static_cast<int64_t>(sc.dp_rounds) * ranges;  // first tail item
  int gl = p.order.front();
  for (int g : p.order)
    if (i >= item_first[g]) gl = g;
  sc.tail_begin = sc.tile_begin[gl] + (i - item_first[gl]) * sc.tiles_per_item[gl];
  return sc;
}

std::vector<int64_t> export_tables(const Plan& p) {
  std::vector<int64_t> t;
  t.push_back(static_cast<int64_t>(p.grids.size()));
  t.push_back(static_cast<int64_t>(p.groups.size()));
  t.push_back(static_cast<int64_t>(p.segs.size()));
  for (const GridRow& g : p.grids) t.insert(t.end(), {g.scale, g.gh, g.gw, g.tok});
  for (const QGroup& g : p.groups) t.insert(t.end(), {g.scale, g.q_begin, g.q_end, g.n_kv});
  for (const SegRow& r : p.segs)
    t.insert(t.end(), {r.q_scale, r.kind, r.frame, r.src_scale, r.eff_scale, r.factor, r.n_tok, r.kv_begin});
  t.push_back(p.n_q);
  t.push_back(p.pairs_per_head);
  return t;
}


// K slices of a narrow GEMM (launch_gemm_split): enough blocks for two per
// CU at most, each slice at least three stages; 1 when the output tiles alone
// fill 256 CUs or K does not split into such slices.
int gemm_k_splits(int32_t M, int32_t N, int32_t K) {
  if (M <= 0 || N <= 0 || K % kGemmStage != 0) return 1;
  const int64_t tiles = static_cast<int64_t>((M + kGemmTile - 1) / kGemmTile) * ((N + kGemmTile - 1) / kGemmTile);
  if (tiles >= 256) return 1;
  const int stages = K / kGemmStage;
  int best = 1;
  for (int s = 2; s <= stages; ++s)
    if (stages % s == 0 && stages / s >= 3 && tiles * s <= 512) best = s;
  return best;
}

int64_t gemm_split_bytes(int32_t M, int32_t N, int32_t K) {
  const int s = gemm_k_splits(M, N, K);
  if (s <= 1) return 0;
  const int64_t tiles = static_cast<int64_t>((M + kGemmTile - 1) / kGemmTile) * ((N + kGemmTile - 1) / kGemmTile);
  return s * tiles * kGemmTile * kGemmTile * 4;
}

// Fused tiers move pixels in pairs (even patch rows on an even frame width) and
// take K in whole 64-element stages with 16-byte rows.  The embedding holds a
// block's patch rows in LDS, K <= 256 of them.  The de-embedding takes 64 x 64
// tiles: while the output is narrow (N <= 256) or has so few tiles that a
// 128 x 128 tile would leave the chip idle.
bool tier_fused(const TierProblem& t, bool embed) {
  const PatchArgs& p = t.patch;
  const bool pairs = p.P % 2 == 0 && p.W % 2 == 0 && (p.frame0 + p.n_frames) * p.C * p.H * p.W <= 0x7fffffff;
  auto at = [](const void* q, uintptr_t n) { return (reinterpret_cast<uintptr_t>(q) & (n - 1)) == 0; };
  if (!pairs || t.K % kGemmStage != 0) return false;
  if (embed) return t.K <= kEmbedMaxK && t.N % 8 == 0 && at(t.bias, 8) && at(t.y, 16);
  const int64_t tiles = int64_t{ceil_div(t.M, kUnembedTile)} * ceil_div(t.N, kUnembedTile);
  return (t.N <= 256 || tiles <= 512) && at(t.bias, 2);
}

// One launch for all these tiers, or patches and GEMM tier by tier?  Measured on
// an MI355X over 660 (embedding) and 430 (de-embedding) random sets of tiers of 8
// to 48 channels and hidden sizes of 384 to 6400, each both ways.
// Embedding: the separate passes cost two launches a tier and read the patches
// twice, but their 256 x 256 tiles read W less often.  Several tiers: one launch
// up to 1.2e8 output elements (9.3e7 + 2.4e7 in hidden 4928 93.7 -> 75.9 us, but
// 1.1e8 + 2.8e7 in 4352 136.5 -> 147.6).  A lone tier: always for K = 64; K = 128
// up to 4e7 (3.7e7 38.0 -> 30.2, 5.8e7 50.4 -> 50.9), 192 up to 2e7 (1.9e7 31.2 ->
// 27.8, 4.4e7 47.0 -> 56.9), 256 up to 3.5e6 (3.1e6 12.2 -> 10.7, 4.6e6 13.1 ->
// 15.5).  370 other sets: 0.84 of the separate passes' time on average, 1.15 at
// worst (lone tiers of K = 128 and 192 scatter by a tenth either way).
// De-embedding: the separate passes may split a long K over the chip, the fused
// kernel walks it.  The better one by fitted times (0.2 % above the better one on
// average, 5 % slower than the separate passes at worst): one tier of 210 tokens
// on hidden 4928 13.9 us apart and 20.6 in one launch, of 396 tokens and 128
// features on 5632 17.3 and 23.1, the two tiers of the 1.3B window 46 and 20.
bool tiers_pay(const TierArgs& a, bool embed) {
  if (embed) {
    double outputs = 0;
    for (int i = 0; i < a.n; ++i) outputs += static_cast<double>(a.g[i].M) * a.g[i].N;
    if (a.n != 1) return a.n > 1 && outputs <= 1.2e8;
    const int32_t k = a.g[0].K;
    return k <= 64 || outputs <= (k <= 128 ? 4e7 : k <= 192 ? 2e7 : 3.5e6);
  }
  double apart = 0, together = 5.88, walked = 0;
  int64_t tiles = 0, stages = 0;
  for (int i = 0; i < a.n; ++i) {
    const TierProblem& t = a.g[i];
    const double m = t.M, n = t.N, k = t.K, st = k / kGemmStage;
    const int64_t t128 = int64_t{ceil_div(t.M, kGemmTile)} * ceil_div(t.N, kGemmTile);
    const int splits = gemm_k_splits(t.M, t.N, t.K);
    apart += 6.22 + 1e-6 * (5.4 * m * n + 0.13 * m * k + 0.56 * n * k);
    if (splits > 1)  // a third launch, a slice's stages, the partial tiles
      apart += 2.92 + 0.435 * st / splits + 0.25e-6 * 4 * splits * static_cast<double>(t128) * kGemmTile * kGemmTile;
    else
      apart += 0.548 * st * std::max(1.0, static_cast<double>(t128) / 512);
    const int64_t cols = ceil_div(t.N, kUnembedTile);
    tiles += ceil_div(t.M, kUnembedTile) * cols;
    stages = std::max<int64_t>(stages, t.K / kGemmStage);
    together += 1e-6 * (0.80 * m * n + 0.038 * m * k);
    walked += 0.125e-6 * m * k * static_cast<double>(cols);  // the tokens once per 64 features
  }
  const double chain = static_cast<double>(stages);
  together += tiles <= 256 ? 0.189 * chain : 0.27 * chain * static_cast<double>((tiles + 511) / 512) + walked;
  return together < apart;
}

int64_t tier_blocks(TierArgs& a, bool embed) {
  const int bm = embed ? kEmbedTile : kUnembedTile;
  // Embedding: quads of feature steps (one for each of a block's four waves)
  // per block so that at most 512 blocks, two per CU and so one round, share
  // the work; a step costs its K stages and its stores (about 1.5 stages).
  // Rounding up tier by tier may leave more blocks than that, and the long ones
  // of the last tier in a second round: the shares of several tiers grow until
  // they fit, or a block has a whole row of steps (14508 tokens of 64 pixels and
  // 3720 of 256 in hidden 1664: 631 blocks; such pairs 12 % faster on average).
  auto step = [](const TierProblem& t) { return t.K / kGemmStage + 1.5; };
  double share = 0;
  for (int i = 0; i < a.n; ++i)
    share += 1.0 * ceil_div(a.g[i].M, bm) * ceil_div(a.g[i].N, bm) * step(a.g[i]) / 512;
  for (;; share *= 1.125) {
    int64_t blocks = 0;
    bool whole_rows = true;
    for (int i = 0; i < a.n; ++i) {
      TierProblem& t = a.g[i];
      t.block_begin = static_cast<int32_t>(std::min<int64_t>(blocks, 0x7fffffff));
      t.tiles_per_block = 1;
      int64_t cols = ceil_div(t.N, bm);
      if (embed) {
        const int64_t quads = (cols + 3) / 4;
        const int64_t most = std::max<int64_t>(1, static_cast<int64_t>(std::ceil(share / step(t) / 4)));
        const int64_t chunks = (quads + most - 1) / most;
        t.tiles_per_block = static_cast<int32_t>(4 * ((quads + chunks - 1) / chunks));
        cols = (cols + t.tiles_per_block - 1) / t.tiles_per_block;
        whole_rows = whole_rows && chunks == 1;
      }
      blocks += ceil_div(t.M, bm) * cols;
    }
    if (!embed || a.n < 2 || blocks <= 512 || whole_rows) return blocks;
  }
}

}  // namespace mssa
