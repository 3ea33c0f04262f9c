// Host-side launch planner: turns per-sequence lengths into workgroup slots.
// Pure host code (no HIP calls) so it can be tested without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "common.h"

namespace medha {

// Geometry of one kernel instantiation.
struct ModeShape {
  int rows_per_wg;  // query rows a workgroup owns
  int tile_keys;    // keys staged per loop iteration (the KV split granule)
};

struct LaunchPlan {
  std::vector<SeqDesc> descs;
  std::vector<int32_t> seq_index;  // position of each descriptor in the caller's batch
  ModeShape shape{0, 0};
  int q_blocks = 1;   // 32-row blocks per wavefront (row-split mode)
  int n_slots = 0;    // grid size
  int total_rows = 0; // token rows of the launch
  bool any_split = false;
};

struct Plan {
  LaunchPlan rows;  // row-split mode: sequences with more than 32 (token, head-in-group) rows
  LaunchPlan keys;  // key-split mode: decodes and other tiny chunks
  int64_t part_rows = 0;  // token rows of split-KV partials (both launches)
  // workspace layout (byte offsets, 256-aligned)
  size_t off_part_o = 0, off_part_lse = 0, bytes = 0;
  // partials of the plan with the least scratch: what a caller has to bring at least
  int64_t min_part_rows = 0;
  size_t min_bytes = 0;
  // what callers are told to bring: enough for this plan and for any smaller choice
  size_t workspace_bytes() const { return std::max(bytes, min_bytes); }
};

struct SeqInput {
  int64_t pt_off;
  int32_t q_row, out_row, chunk_len, prefix_len;
  int32_t kv_len = -1;  // keys in the page-table slice; -1: prefix_len + chunk_len
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace for `rows` token rows of partials: outputs, then LSEs.
inline size_t partial_o_bytes(int64_t rows, int h_q, int head_dim) {
  return align256((size_t)rows * h_q * head_dim * sizeof(float));
}
inline size_t partial_bytes(int64_t rows, int h_q, int head_dim) {
  return std::max<size_t>(256, align256(partial_o_bytes(rows, h_q, head_dim) +
                                        (size_t)rows * h_q * sizeof(float)));
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// What a workgroup of a row-split launch costs, in microseconds (MI355X): one KV tile of its
// walk, and everything outside the walk (descriptor, Q, the ring's first fill, the epilogue).
// Only the ratios matter: they weigh more, shorter KV ranges against fewer, longer ones.
struct WalkCost {
  double tile_us, fixed_us;
  int wgs_per_cu;  // workgroups a compute unit holds at a time
};

// (measured; the small workgroups of head dim 64 share a compute unit in pairs, where one's
// start and end hide behind the other's walk, at the price of a second copy of the K/V loads)
inline WalkCost walk_cost(int head_dim, int q_blocks) {
  if (head_dim == 128) return q_blocks == 2 ? WalkCost{1.64, 10.0, 1} : WalkCost{1.2, 10.0, 1};
  return q_blocks == 2 ? WalkCost{0.9, 11.0, 1} : WalkCost{0.91, 9.0, 2};
}

// The merge of a launch's partials: a launch, then bytes at the rate the merge kernel reads
// them (31 MB in 8 us).  Writing them hides behind the walks of other workgroups.
constexpr double kMergeLaunchUs = 3.0, kMergeBytesPerUs = 4.5e6;
// Partials beyond this are not worth their memory (a split that needs more is not considered).
constexpr int64_t kMaxPartialBytes = (int64_t)128 << 20;
constexpr int kMaxPlannedSeqs = 16;  // launches of more sequences keep the simple rule
constexpr int kMaxWaves = 8;         // rounds of workgroups per compute unit worth considering

// Workgroups of one length on the fullest accelerator die.
struct WalkGroup {
  double us;
  int64_t count;
};

// When the last workgroup ends if `machines` slots take the groups in descending length, each
// workgroup going to the slot that is free first.  Slots free at the same time are kept as one
// entry, so equal walks cost one step per round of the device.
inline double makespan(std::vector<WalkGroup>& groups, int64_t machines) {
  std::sort(groups.begin(), groups.end(),
            [](const WalkGroup& a, const WalkGroup& b) { return a.us > b.us; });
  std::vector<WalkGroup> free_at{{0.0, machines}};  // (time, slots), ascending
  double end = 0.0;
  for (WalkGroup g : groups)
    while (g.count > 0) {
      WalkGroup& first = free_at.front();
      const int64_t n = std::min(g.count, first.count);
      const double t = first.us + g.us;
      end = std::max(end, t);
      g.count -= n;
      first.count -= n;
      if (first.count == 0) free_at.erase(free_at.begin());
      auto at = std::lower_bound(free_at.begin(), free_at.end(), t,
                                 [](const WalkGroup& a, double v) { return a.us < v; });
      if (at != free_at.end() && at->us == t)
        at->count += n;
      else
        free_at.insert(at, WalkGroup{t, n});
    }
  return end;
}

inline int64_t kv_tiles_of(const SeqDesc& sd, int tile_keys) {
  return std::max<int64_t>(1, ceil_div((int64_t)sd.kv_len, tile_keys));
}

// Tiles that row tile rt of a sequence walks.
inline int64_t tiles_at(const SeqDesc& sd, const ModeShape& sh, int gqa, int64_t rt) {
  const int64_t last_tok =
      (std::min((int64_t)sd.chunk_len * gqa, (rt + 1) * sh.rows_per_wg) - 1) / gqa;
  const int64_t keys = std::min<int64_t>(sd.kv_len, (int64_t)sd.prefix_len + last_tok + 1);
  return ceil_div(std::max<int64_t>(0, keys), sh.tile_keys);
}

// Whether the causal triangle makes the walks of its row tiles differ by more than a sixteenth.
inline bool uneven_walks(const SeqDesc& sd, const ModeShape& sh, int gqa) {
  const int64_t t_last = tiles_at(sd, sh, gqa, sd.n_row_tiles - 1);
  return t_last - tiles_at(sd, sh, gqa, 0) > t_last / 16;
}

// KV ranges of a sequence when no range is longer than `steps` tiles nor shorter than min_tiles.
inline void split_by_steps(const SeqDesc& sd, int tile_keys, int64_t steps, int min_tiles,
                           int64_t& n_split, int64_t& tps) {
  const int64_t kv_tiles = kv_tiles_of(sd, tile_keys);
  n_split = ceil_div(kv_tiles, steps);
  n_split = std::min(n_split, std::max<int64_t>(1, kv_tiles / min_tiles));
  n_split = std::max<int64_t>(1, n_split);
  tps = ceil_div(kv_tiles, n_split);
  n_split = ceil_div(kv_tiles, tps);
}

// Partial token rows of a launch split by `steps`.
inline int64_t partial_rows(const LaunchPlan& lp, int64_t steps, int min_tiles) {
  int64_t rows = 0, n_split, tps;
  for (const SeqDesc& sd : lp.descs) {
    split_by_steps(sd, lp.shape.tile_keys, steps, min_tiles, n_split, tps);
    if (n_split > 1) rows += n_split * sd.chunk_len;
  }
  return rows;
}

// Workgroup slots of a launch split by `steps`.
inline int64_t workgroups(const LaunchPlan& lp, int h_kv, int64_t steps, int min_tiles) {
  int64_t n = 0, n_split, tps;
  for (const SeqDesc& sd : lp.descs) {
    split_by_steps(sd, lp.shape.tile_keys, steps, min_tiles, n_split, tps);
    n += kXcds * ceil_div((int64_t)h_kv * sd.n_row_tiles * n_split, kXcds);
  }
  return n;
}

// Estimated time of a row-split launch whose KV ranges are at most `steps` tiles long.
inline double launch_us(const LaunchPlan& lp, int h_kv, int gqa, int num_cus, const WalkCost& wc,
                        int64_t steps, int min_tiles, int64_t row_bytes) {
  const ModeShape sh = lp.shape;
  std::vector<WalkGroup> groups;
  int64_t part = 0;
  for (const SeqDesc& sd : lp.descs) {
    int64_t n_split, tps;
    split_by_steps(sd, sh.tile_keys, steps, min_tiles, n_split, tps);
    if (n_split > 1) part += n_split * sd.chunk_len;
    // up to 8 classes of row tiles stand for a causal triangle
    const int64_t n_rt = sd.n_row_tiles;
    const int64_t t_last = tiles_at(sd, sh, gqa, n_rt - 1);
    const int64_t classes = uneven_walks(sd, sh, gqa) ? std::min<int64_t>(n_rt, 8) : 1;
    // Workgroups of the fullest die (see decode_slot_dealt): its whole groups, one of every 8, and an
    // eighth, rounded up, of what the others hold.
    const int64_t all = h_kv * n_split, dealt = all / kXcds;
    int64_t before = 0;
    auto add = [&](int64_t tiles, int64_t count, bool whole) {
      if (tiles <= 0) return;
      int64_t n = count;
      if (!whole) {
        n = ceil_div(before + count, kXcds) - ceil_div(before, kXcds);
        before += count;
      }
      if (n > 0) groups.push_back(WalkGroup{wc.fixed_us + (double)tiles * wc.tile_us, n});
    };
    if (classes == 1) {
      if (t_last >= tps) add(tps, n_rt * h_kv * (t_last / tps), false);
      add(t_last % tps, n_rt * h_kv, false);
      continue;
    }
    for (int64_t c = classes; c-- > 0;) {
      const int64_t lo = c * n_rt / classes, hi = (c + 1) * n_rt / classes;
      const int64_t t = tiles_at(sd, sh, gqa, (lo + hi) / 2);
      for (int64_t g = 0; g < dealt && (g * kXcds / h_kv) * tps < t; ++g)
        add(std::min(tps, t - (g * kXcds / h_kv) * tps), hi - lo, true);
      const int64_t from = dealt * kXcds;  // the other groups: (split, heads of it)
      for (int64_t sp = from / h_kv; sp < n_split && sp * tps < t; ++sp)
        add(std::min(tps, t - sp * tps), (hi - lo) * (h_kv - std::max<int64_t>(0, from - sp * h_kv)),
            false);
    }
  }
  const int64_t machines = std::max<int64_t>(1, num_cus / kXcds) * wc.wgs_per_cu;
  double us = makespan(groups, machines);
  if (part > 0) us += kMergeLaunchUs + (double)(part * row_bytes) / kMergeBytesPerUs;
  return us;
}

// Longest KV range (in tiles) of a row-split launch.  The simple rule (one round of workgroups
// over the device, rounded up) can leave a second round nearly empty: 47 row tiles in 6 ranges
// are 282 workgroups on 256 compute units and take twice the time of 256.  So the ranges that
// fill 1, 2, ... whole rounds as well as possible are compared with it by estimated time: more
// rounds waste less of the last one, but pay a workgroup's fixed cost each and write more
// partials.  `base` is the simple rule's answer; it is always allowed, others only if their
// partials fit `max_rows` token rows.
inline int64_t choose_steps(const LaunchPlan& lp, int h_kv, int gqa, int num_cus,
                            const WalkCost& wc, int64_t base, int min_tiles, int64_t row_bytes,
                            int64_t max_rows, double& best_us) {
  best_us = launch_us(lp, h_kv, gqa, num_cus, wc, base, min_tiles, row_bytes);
  int64_t longest = 1, unsplit = 0;
  for (const SeqDesc& sd : lp.descs) {
    longest = std::max(longest, kv_tiles_of(sd, lp.shape.tile_keys));
    unsplit += (int64_t)h_kv * sd.n_row_tiles;
  }
  const int64_t slots = (int64_t)num_cus * wc.wgs_per_cu;
  if (unsplit >= kMaxWaves * slots || longest <= min_tiles) return base;
  const int64_t allowed = std::min(max_rows, kMaxPartialBytes / row_bytes);
  int64_t best = base, prev = base;
  auto consider = [&](int64_t steps) {
    if (steps == prev || partial_rows(lp, steps, min_tiles) > allowed) return;
    prev = steps;
    const double us = launch_us(lp, h_kv, gqa, num_cus, wc, steps, min_tiles, row_bytes);
    // A few idle compute units are not all loss: the part is power-limited, the others clock
    // higher.  (47 row tiles, 4712 tiles: 16 ranges in 3 rounds, 2 % of them empty, are estimated
    // at 0.97 of 5 ranges in one round with 8 % empty, and measure the same within 2 %.)
    if (us < 0.97 * best_us) {
      best = steps;
      best_us = us;
    }
  };
  consider(longest);  // no split at all
  for (int waves = 1; waves <= kMaxWaves; ++waves) {
    if (workgroups(lp, h_kv, longest, min_tiles) > waves * slots) continue;
    int64_t lo = min_tiles, hi = longest;  // the shortest ranges that fit `waves` rounds
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      if (workgroups(lp, h_kv, mid, min_tiles) <= waves * slots) hi = mid; else lo = mid + 1;
    }
    consider(lo);
    if (lo <= min_tiles) break;
  }
  return best;
}

// Cuts the KV axis of each sequence into ranges of at most `steps` tiles (never below
// `min_tiles`), orders the sequences and hands out workgroup slots and partial rows.
inline void plan_launch(LaunchPlan& lp, int h_kv, int gqa, int64_t steps, int min_tiles,
                        int64_t& part_rows) {
  const ModeShape sh = lp.shape;
  for (SeqDesc& sd : lp.descs) {
    int64_t n_split, tps;
    split_by_steps(sd, sh.tile_keys, steps, min_tiles, n_split, tps);
    sd.n_split = (int)n_split;
    sd.tiles_per_split = (int)tps;
    sd.dealt = sd.n_row_tiles > 1 && uneven_walks(sd, sh, gqa);
  }
  // Longest workgroups first: the hardware hands workgroups out in slot order, so the short
  // ones fill the launch's tail instead of a long one starting last (the order of the
  // sequences inside a launch is free: every descriptor carries its own rows).
  {
    std::vector<int> order(lp.descs.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
    auto walk = [&](int i) {
      const SeqDesc& sd = lp.descs[i];
      return std::min<int64_t>(sd.tiles_per_split, ceil_div((int64_t)sd.kv_len, sh.tile_keys));
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return walk(a) > walk(b); });
    std::vector<SeqDesc> descs(order.size());
    std::vector<int32_t> index(order.size());
    for (size_t i = 0; i < order.size(); ++i) {
      descs[i] = lp.descs[order[i]];
      index[i] = lp.seq_index[order[i]];
    }
    lp.descs.swap(descs);
    lp.seq_index.swap(index);
  }
  int slot = 0, rank = 0;
  for (SeqDesc& sd : lp.descs) {
    sd.work_start = slot;
    sd.row_rank = rank;
    sd.part_row = 0;
    if (sd.n_split > 1) {
      sd.part_row = (int32_t)part_rows;
      part_rows += (int64_t)sd.n_split * sd.chunk_len;
      lp.any_split = true;
    }
    const int64_t items = (int64_t)h_kv * sd.n_split * sd.n_row_tiles;
    slot += (int)(kXcds * ceil_div(items, kXcds));
    rank += sd.chunk_len;
  }
  lp.n_slots = slot;
  lp.total_rows = rank;
}

inline void set_row_tiles(LaunchPlan& lp, int gqa) {
  for (SeqDesc& sd : lp.descs)
    sd.n_row_tiles = (int)ceil_div((int64_t)sd.chunk_len * gqa, lp.shape.rows_per_wg);
}

// The simple rule: ranges short enough for about `target_wgs` equally long workgroups, no
// split where the row tiles alone are as many.  Also sets the row tiles.
inline int64_t simple_steps(LaunchPlan& lp, int h_kv, int gqa, int target_wgs) {
  int64_t unsplit_wgs = 0, total_steps = 0, longest = 1;
  set_row_tiles(lp, gqa);
  for (const SeqDesc& sd : lp.descs) {
    const int64_t kv_tiles = ceil_div((int64_t)sd.kv_len, lp.shape.tile_keys);
    unsplit_wgs += (int64_t)h_kv * sd.n_row_tiles;
    total_steps += (int64_t)h_kv * sd.n_row_tiles * kv_tiles;
    longest = std::max(longest, kv_tiles);
  }
  return unsplit_wgs < target_wgs ? std::max<int64_t>(1, ceil_div(total_steps, target_wgs))
                                  : longest;
}

// Plans a batch.  `budget` is the size of the workspace at hand: the plan takes the KV ranges
// that are expected to be fastest among those whose partials fit it; the simple rule's need
// (`min_bytes`) is the least a call has to bring.
inline Plan make_plan(const SeqInput* seqs, int batch, int h_q, int h_kv, int head_dim,
                      int num_cus, size_t budget = SIZE_MAX) {
  Plan plan;
  const int gqa = h_q / h_kv;
  int max_rows = 0;
  for (int b = 0; b < batch; ++b) {
    SeqDesc sd{};
    sd.pt_off = seqs[b].pt_off;
    sd.q_row = seqs[b].q_row;
    sd.out_row = seqs[b].out_row;
    sd.chunk_len = seqs[b].chunk_len;
    sd.prefix_len = seqs[b].prefix_len;
    sd.kv_len = seqs[b].kv_len >= 0 ? seqs[b].kv_len : sd.prefix_len + sd.chunk_len;
    const int64_t n_rows = (int64_t)sd.chunk_len * gqa;
    LaunchPlan& lp = n_rows <= 32 ? plan.keys : plan.rows;
    lp.descs.push_back(sd);
    lp.seq_index.push_back(b);
    if (n_rows > 32) max_rows = std::max(max_rows, (int)std::min<int64_t>(n_rows, 1 << 30));
  }
  // Row-split mode: 4 wavefronts x (32 * q_blocks) rows, 64-key tiles.
  plan.rows.q_blocks = max_rows >= 256 ? 2 : 1;
  plan.rows.shape = ModeShape{kWaves * 32 * plan.rows.q_blocks, 64};
  // Key-split mode: one 32-row block, 128-key tiles (32 per wavefront).
  plan.keys.q_blocks = 1;
  plan.keys.shape = ModeShape{32, 32 * kWaves};
  constexpr int kMinTiles = 4;
  const int64_t row_bytes = (int64_t)h_q * (head_dim + 1) * sizeof(float);
  int64_t keys_steps = 1, rows_steps = 1, min_rows = 0;
  if (!plan.keys.descs.empty()) {
    keys_steps = simple_steps(plan.keys, h_kv, gqa, num_cus * 8);
    min_rows += partial_rows(plan.keys, keys_steps, kMinTiles);
  }
  if (!plan.rows.descs.empty()) {
    rows_steps = simple_steps(plan.rows, h_kv, gqa, num_cus);
    const int64_t keys_rows = min_rows;
    min_rows += partial_rows(plan.rows, rows_steps, kMinTiles);
    // token rows of partials that fit the budget (the workspace's two arrays are rounded up to
    // 256 bytes each, which can cost the last rows)
    int64_t fit = (int64_t)(std::min<size_t>(budget, (size_t)1 << 60) / row_bytes);
    while (fit > 0 && partial_bytes(fit, h_q, head_dim) > budget) --fit;
    if ((int)plan.rows.descs.size() <= kMaxPlannedSeqs) {
      double us, small_us;
      rows_steps = choose_steps(plan.rows, h_kv, gqa, num_cus,
                                walk_cost(head_dim, plan.rows.q_blocks), rows_steps, kMinTiles,
                                row_bytes, fit - keys_rows, us);
      // At head dim 64 the small workgroups are the alternative: half the granule, short walks
      // overlapped (777 tokens at 20K, 32/8 heads: 164 -> 155 us; 14 prompts, 24 tiles
      // on average: 174 -> 163 us; 12 prompts, 14 tiles: 226 -> 215 us; but 1 % longer at 96 and
      // 288 tiles where both fill the device).  At 128 two of their rings do not fit a unit.
      if (head_dim == 64 && plan.rows.q_blocks == 2) {
        LaunchPlan small = plan.rows;
        small.q_blocks = 1;
        small.shape.rows_per_wg = kWaves * 32;
        set_row_tiles(small, gqa);
        const int64_t steps = choose_steps(small, h_kv, gqa, num_cus, walk_cost(head_dim, 1),
                                           INT32_MAX, kMinTiles, row_bytes, fit - keys_rows,
                                           small_us);
        if (small_us < 0.97 * us &&
            workgroups(small, h_kv, steps, kMinTiles) > num_cus) {  // else nothing pairs up
          plan.rows = small;
          rows_steps = steps;
        }
      }
    }
  }
  if (!plan.rows.descs.empty())
    plan_launch(plan.rows, h_kv, gqa, rows_steps, kMinTiles, plan.part_rows);
  if (!plan.keys.descs.empty())
    plan_launch(plan.keys, h_kv, gqa, keys_steps, kMinTiles, plan.part_rows);

  plan.off_part_o = 0;
  plan.off_part_lse = partial_o_bytes(plan.part_rows, h_q, head_dim);
  plan.bytes = partial_bytes(plan.part_rows, h_q, head_dim);
  plan.min_bytes = partial_bytes(min_rows, h_q, head_dim);
  plan.min_part_rows = min_rows;
  return plan;
}

}  // namespace medha
