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
  bool paired = false;  // two workgroups to a compute unit, with the short ring (head dim 128)
  int n_slots = 0;    // grid size: key-split, the items; row-split, every sequence's in eights
  int total_rows = 0; // token rows of the launch
  int num_cus = 0;    // compute units planned for
  bool key_split = false;
  bool any_split = false;
};

struct Plan {
  LaunchPlan rows;  // row-split mode: sequences with more than 32 (token, head-in-group) rows
  LaunchPlan keys;  // key-split mode: decodes and other tiny chunks
  int64_t part_rows = 0;  // token rows of split-KV partials (both launches)
  // workspace layout (byte offsets, 256-aligned)
  size_t off_part_o = 0, off_part_lse = 0, bytes = 0;
  // partials of the simple rule's ranges: what a caller has to bring at least, also where the
  // plan chosen writes fewer (a cut that does not pay is dropped), so that what is refused
  // depends on the sizes alone
  int64_t min_part_rows = 0;
  size_t min_bytes = 0;
  // what callers are told to bring
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
// Launches of one, two and four rounds of equal walks (512 to 8192 keys) take 1.70 us a tile and
// 10.3 to 11.5 us outside the walk at head dim 128, 1.05 us and 5.0 to 6.5 us at 64, with 256-row
// workgroups.  At 64 the constants ask 12 tiles for a workgroup's start and end, not 6: plans
// lean towards fewer ranges there.
struct WalkCost {
  double tile_us, fixed_us;
  int wgs_per_cu;  // workgroups a compute unit holds at a time
};

// (the small workgroups of head dim 64 share a compute unit in pairs, where one's start and end
// hide behind the other's walk, at the price of a second copy of the K/V loads)
inline WalkCost walk_cost(int head_dim, int q_blocks) {
  if (head_dim == 128) return q_blocks == 2 ? WalkCost{1.64, 10.0, 1} : WalkCost{1.2, 10.0, 1};
  return q_blocks == 2 ? WalkCost{0.9, 11.0, 1} : WalkCost{0.91, 9.0, 2};
}

// Small workgroups (128 rows) where that is not their only form: alone on a compute unit (head dims 64
// and 128), and in pairs with the short ring (head dim 128).  Equal walks of 8, 16, 32, 64 and 128
// tiles, one round of the device, 8 K/V streams, take
//   alone, d 64      13.4, 19.5, 31.8, 54.1,  98.8 us: 0.71 us a tile and 7.5 us outside the walk
//   alone, d 128     18.8, 27.7, 46.1, 81.1, 148.7: 1.09 and 10
//   in pairs, d 128  27.4, 42.5, 74.4, 132.7, 250.2 for two: 1.86 and 12
//   256 rows, d 128  26.9, 41.9, 72.9, 127.7, 239.4: 1.77 and 12.5 (d 64: 17.0 .. 146.9)
// Against the large form's constants above, these ask for the small ones what they measure at 8 to
// 16 tiles (alone 18.0 and 28.0 us at d 128, 14.2 and 19.4 at 64; a pair 1.04 of a large one at 16,
// measured 1.02) and a twelfth more at 128 (a pair 1.11, measured 1.05): where walks are long, a
// small form wins by the whole round that it saves or not at all.
constexpr WalkCost kAloneCost[2] = {{0.65, 9.0, 1}, {1.25, 8.0, 1}}, kPairedCost{1.85, 8.0, 2};

constexpr int64_t kShortPairedTiles = 10;

// What partials cost: a launch, then their bytes.  The merge kernel takes 8 us for 31 MB and 17
// to 18 us for 99 MB; the constants ask 10 and 25, since partials are written and held as well.
constexpr double kMergeLaunchUs = 3.0, kMergeBytesPerUs = 4.5e6;
// Partials beyond this are not worth their memory (a split that needs more is not considered).
constexpr int64_t kMaxPartialBytes = (int64_t)128 << 20;
// Launches of more sequences keep the simple rule: the estimate has been held against measured
// launches up to here only.  Where the rule leaves a round nearly empty that costs 5 to 15 % (17
// chunks of 200 at 20K, 8/1 heads, 338 us, 318 with the estimate's plan; 24 of them 492 and 444;
// 17 chunks of 600 at 65K 2.99 and 2.53 ms); 64 chunks of 200 and 17 to 64 prompts at head dim
// 128 take the same either way.
constexpr int kMaxPlannedSeqs = 16;
constexpr int kMaxWaves = 8;  // rounds of workgroups per compute unit worth considering

// Workgroups that walk the same number of tiles, on the fullest accelerator die.
struct WalkGroup {
  int64_t tiles, count;
};

// Slots that are free from the same time on.
struct FreeSlots {
  double us;
  int64_t count;
};

// When the last workgroup ends if `machines` slots take the groups in descending length, each
// workgroup going to the slot that is free first.  Slots free at the same time are one entry, so
// equal walks cost one step per round of the device, and the slots a group leaves behind come in
// ascending order, so they are appended, and merged once with the slots it did not touch.
inline double makespan(std::vector<WalkGroup>& groups, int64_t machines, const WalkCost& wc) {
  std::sort(groups.begin(), groups.end(),
            [](const WalkGroup& a, const WalkGroup& b) { return a.tiles > b.tiles; });
  std::vector<FreeSlots> before, after, merged;  // ascending
  for (auto* v : {&before, &after, &merged}) v->reserve(2 * machines);
  before.push_back(FreeSlots{0.0, machines});
  double end = 0.0;
  for (size_t k = 0; k < groups.size();) {
    const int64_t tiles = groups[k].tiles;
    int64_t count = 0;
    for (; k < groups.size() && groups[k].tiles == tiles; ++k) count += groups[k].count;
    const double us = wc.fixed_us + (double)tiles * wc.tile_us;
    after.clear();
    size_t i = 0, j = 0;  // first entries of `before` and `after` not used up
    while (count > 0) {
      const bool old = i < before.size() && (j == after.size() || before[i].us <= after[j].us);
      FreeSlots& first = old ? before[i] : after[j];
      const int64_t n = std::min(count, first.count);
      const double t = first.us + us;
      count -= n;
      first.count -= n;
      if (first.count == 0) ++(old ? i : j);
      if (!after.empty() && after.back().us == t && j < after.size())
        after.back().count += n;
      else
        after.push_back(FreeSlots{t, n});
      end = std::max(end, t);
    }
    merged.clear();
    while (i < before.size() || j < after.size()) {
      const bool old = i < before.size() && (j == after.size() || before[i].us <= after[j].us);
      merged.push_back(old ? before[i++] : after[j++]);
    }
    before.swap(merged);
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

// Row tiles of one sequence that stand for each other in an estimate: `count` of them walk
// `tiles` tiles (before the KV axis is cut).
struct WalkClass {
  int64_t tiles, count;
};

// Classes of a launch's triangles, dealt out by their row tiles (a sequence alone has 8).  With 8
// for every sequence, one plan in 500 is another one, and planning 16 prompts takes twice as long.
constexpr int kWalkClasses = 32;

// What the estimates of a launch have in common, whatever its KV ranges.
struct LaunchWalks {
  std::vector<WalkClass> classes;   // of all sequences, longest walk first within a sequence
  std::vector<int> first_class;     // of each sequence, and the end
  std::vector<char> dealt;          // sequences whose walks differ (see decode_slot_dealt)
  int64_t total_tiles = 0;          // walked by all workgroups
  int64_t busy = 0, unsplit = 0;    // workgroups without a cut: with keys to walk, and all
  int64_t key_tiles = 0;            // tiles if every workgroup walked all keys
  int64_t longest = 1;              // KV tiles of the longest sequence
};

inline LaunchWalks launch_walks(const LaunchPlan& lp, int h_kv, int gqa) {
  LaunchWalks lw;
  int64_t all_row_tiles = 0;
  for (const SeqDesc& sd : lp.descs) all_row_tiles += sd.n_row_tiles;
  lw.first_class.reserve(lp.descs.size() + 1);
  lw.classes.reserve(lp.descs.size() + kWalkClasses);
  for (const SeqDesc& sd : lp.descs) {
    lw.first_class.push_back((int)lw.classes.size());
    // up to 8 classes of row tiles stand for a causal triangle
    const int64_t n_rt = sd.n_row_tiles;
    const int64_t most = std::min<int64_t>(8, ceil_div(kWalkClasses * n_rt, all_row_tiles));
    const bool uneven = uneven_walks(sd, lp.shape, gqa);
    const int64_t classes = uneven ? std::min(n_rt, most) : 1;
    lw.dealt.push_back(uneven);
    for (int64_t c = classes; c-- > 0;) {
      const int64_t lo = c * n_rt / classes, hi = (c + 1) * n_rt / classes;
      const int64_t t = tiles_at(sd, lp.shape, gqa, uneven ? (lo + hi) / 2 : n_rt - 1);
      lw.classes.push_back(WalkClass{t, hi - lo});
      lw.total_tiles += t * (hi - lo) * h_kv;
      if (t > 0) lw.busy += (hi - lo) * h_kv;
    }
    const int64_t kv_tiles = kv_tiles_of(sd, lp.shape.tile_keys);
    lw.unsplit += n_rt * h_kv;
    lw.key_tiles += n_rt * h_kv * kv_tiles;
    lw.longest = std::max(lw.longest, kv_tiles);
  }
  lw.first_class.push_back((int)lw.classes.size());
  return lw;
}

// Workgroups and partial token rows of a launch split by `steps`.
struct SplitSize {
  int64_t slots, part_rows;
  int64_t items;  // slots that are not idle
};

inline SplitSize split_size(const LaunchPlan& lp, int h_kv, int64_t steps, int min_tiles) {
  SplitSize s{0, 0, 0};
  int64_t n_split, tps;
  for (const SeqDesc& sd : lp.descs) {
    split_by_steps(sd, lp.shape.tile_keys, steps, min_tiles, n_split, tps);
    const int64_t items = (int64_t)h_kv * sd.n_row_tiles * n_split;
    s.items += items;
    s.slots += kXcds * ceil_div(items, kXcds);
    if (n_split > 1) s.part_rows += n_split * sd.chunk_len;
  }
  return s;
}

inline double merge_us(int64_t part_rows, int64_t row_bytes) {
  return part_rows > 0 ? kMergeLaunchUs + (double)(part_rows * row_bytes) / kMergeBytesPerUs : 0.0;
}

inline int64_t machines_of(int num_cus, const WalkCost& wc) {
  return std::max<int64_t>(1, num_cus / kXcds) * wc.wgs_per_cu;
}

// The work of a launch with ranges of at most `steps` tiles, spread evenly: no estimate is less.
inline double even_us(const LaunchWalks& lw, int64_t steps, int num_cus, const WalkCost& wc) {
  const int64_t wgs = std::max(lw.busy, lw.total_tiles / steps);
  return ((double)lw.total_tiles * wc.tile_us + (double)wgs * wc.fixed_us) /
         (double)(kXcds * machines_of(num_cus, wc));
}

// Estimated time of a row-split launch whose KV ranges are at most `steps` tiles long.
inline double launch_us(const LaunchPlan& lp, const LaunchWalks& lw, int h_kv, int num_cus,
                        const WalkCost& wc, int64_t steps, int min_tiles, int64_t row_bytes) {
  std::vector<WalkGroup> groups;
  groups.reserve(4 * lw.classes.size());
  int64_t part = 0;
  for (size_t s = 0; s < lp.descs.size(); ++s) {
    const SeqDesc& sd = lp.descs[s];
    int64_t n_split, tps;
    split_by_steps(sd, lp.shape.tile_keys, steps, min_tiles, n_split, tps);
    if (n_split > 1) part += n_split * sd.chunk_len;
    // Workgroups of the fullest die: an even launch's equal runs (decode_slot) give it an
    // eighth, rounded up; decode_slot_dealt gives it one of every 8 whole (head, range) groups,
    // and an eighth, rounded up, of what the last groups hold.
    const int c0 = lw.first_class[s], c1 = lw.first_class[s + 1];
    const int64_t whole_groups = !lw.dealt[s] ? 0 : h_kv * n_split / kXcds;
    const int64_t from = whole_groups * kXcds;  // the other groups: (range, heads of it)
    int64_t before = 0;
    auto add_whole = [&](int64_t tiles, int64_t n) {
      if (tiles > 0 && n > 0) groups.push_back(WalkGroup{tiles, n});
    };
    auto add_rest = [&](int64_t tiles, int64_t count) {
      if (tiles <= 0 || count <= 0) return;
      const int64_t n = ceil_div(before + count, kXcds) - ceil_div(before, kXcds);
      before += count;
      if (n > 0) groups.push_back(WalkGroup{tiles, n});
    };
    for (int c = c0; c < c1; ++c) {
      const WalkClass& wcl = lw.classes[c];
      // `full` ranges are walked to their end, the next one for `left` tiles
      const int64_t full = wcl.tiles / tps, left = wcl.tiles % tps;
      const int64_t upto_full = full * h_kv, upto_left = upto_full + (left > 0 ? h_kv : 0);
      const int64_t w_full = std::min(whole_groups, ceil_div(upto_full, kXcds));
      const int64_t w_left = std::min(whole_groups, ceil_div(upto_left, kXcds)) - w_full;
      add_whole(tps, wcl.count * w_full);
      add_whole(left, wcl.count * w_left);
      const int64_t r_full = std::max<int64_t>(0, upto_full - from);
      const int64_t r_left = std::max<int64_t>(0, upto_left - from) - r_full;
      add_rest(tps, wcl.count * r_full);
      add_rest(left, wcl.count * r_left);
    }
  }
  return makespan(groups, machines_of(num_cus, wc), wc) + merge_us(part, row_bytes);
}

// Longest KV range (in tiles) of a row-split launch, and its estimated time (`best_us`).  The
// simple rule (one round of workgroups over the device, rounded up) can leave a second round
// nearly empty: 47 row tiles in 6 ranges are 282 workgroups on 256 compute units and take twice
// the time of 256.  So the ranges that fill 1, 2, ... whole rounds as well as possible are
// compared with it by estimated time: more rounds waste less of the last one, but pay a
// workgroup's fixed cost each and write more partials.  `base` is the simple rule's answer; it
// is always allowed, others only if their partials fit `max_rows` token rows.
//
// Planning is host time on every call, so what cannot win is not simulated: a plan is no faster
// than its work spread evenly, and its work grows with its workgroups.  (Host time of one plan,
// simulating every candidate -> now: 16 prompts of 1K median at 8/2 heads, d 64, 38 -> 13 us, and
// their iteration, which plans twice, 85 -> 69 us; 8/1 heads, d 128, 15 -> 7 us.)
inline int64_t choose_steps(const LaunchPlan& lp, const LaunchWalks& lw, int h_kv, int num_cus,
                            const WalkCost& wc, int64_t base, int min_tiles, int64_t row_bytes,
                            int64_t max_rows, double& best_us) {
  const int64_t slots = (int64_t)num_cus * wc.wgs_per_cu;
  // (launches of very many rounds end within a walk or two of the even spread)
  best_us = lw.unsplit >= 8 * kMaxWaves * slots
                ? even_us(lw, lw.longest, num_cus, wc)
                : launch_us(lp, lw, h_kv, num_cus, wc, base, min_tiles, row_bytes);
  if (lw.unsplit >= kMaxWaves * slots || lw.longest <= min_tiles) return base;
  const int64_t allowed = std::min(max_rows, kMaxPartialBytes / row_bytes);
  int64_t best = base, prev = base;
  // A few idle compute units are not all loss: the part is power-limited, the others clock
  // higher.  (47 row tiles, 4712 tiles: 16 ranges in 3 rounds, 2 % of them empty, are estimated
  // at 0.97 of 5 ranges in one round with 8 % empty, and measure the same within 2 %.)
  constexpr double kWorth = 0.97;
  auto consider = [&](int64_t steps, int64_t part_rows) {
    if (steps == prev || part_rows > allowed) return;
    prev = steps;
    if (even_us(lw, steps, num_cus, wc) + merge_us(part_rows, row_bytes) >= kWorth * best_us)
      return;
    const double us = launch_us(lp, lw, h_kv, num_cus, wc, steps, min_tiles, row_bytes);
    if (us < kWorth * best_us) {
      best = steps;
      best_us = us;
    }
  };
  const SplitSize uncut = split_size(lp, h_kv, lw.longest, min_tiles);
  consider(lw.longest, uncut.part_rows);
  const SplitSize finest = split_size(lp, h_kv, min_tiles, min_tiles);
  int64_t hi = lw.longest;  // the shortest ranges that fit the rounds so far, and their size
  SplitSize at_hi = uncut;
  for (int waves = 1; waves <= kMaxWaves; ++waves) {
    const int64_t room = waves * slots;
    if (uncut.slots > room) continue;
    if (even_us(lw, lw.longest, num_cus, wc) >= kWorth * best_us) break;
    // The shortest ranges that fit: a search that gallops from a guess (all tiles spread evenly,
    // or what fewer rounds needed, in proportion) and bisects once it has both sides.
    int64_t lo = min_tiles, step = 1;
    int64_t probe = hi == lw.longest ? lw.key_tiles / room : hi * (waves - 1) / waves;
    if (finest.slots <= room) {
      hi = min_tiles;
      at_hi = finest;
    }
    while (lo < hi) {
      probe = std::min(std::max(probe, lo), hi - 1);
      const SplitSize size = split_size(lp, h_kv, probe, min_tiles);
      const bool fits = size.slots <= room;
      if (fits) {
        hi = probe;
        at_hi = size;
      } else {
        lo = probe + 1;
      }
      probe = hi - lo <= step ? (lo + hi) / 2 : fits ? hi - step : lo + step - 1;
      step *= 2;
    }
    consider(hi, at_hi.part_rows);
    if (hi <= min_tiles) break;
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
  int slot = 0, rank = 0, die = 0;
  for (SeqDesc& sd : lp.descs) {
    sd.first_die = (int16_t)die;
    sd.work_start = slot;
    sd.row_rank = rank;
    sd.part_row = 0;
    if (sd.n_split > 1) {
      sd.part_row = (int32_t)part_rows;
      part_rows += (int64_t)sd.n_split * sd.chunk_len;
      lp.any_split = true;
    }
    const int64_t items = (int64_t)h_kv * sd.n_split * sd.n_row_tiles;
    slot += (int)(lp.key_split ? items : kXcds * ceil_div(items, kXcds));
    die = (int)((die + items) % kXcds);
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

// Plans a batch.  `budget` is the size of the workspace at hand: the plan is the one without a limit
// if its partials fit it (so that every workspace of the reported size gives the same plan, whatever
// the choices on the way to it look at), and otherwise takes the KV ranges that are expected to be
// fastest among those whose partials do; the simple rule's need (`min_bytes`) is the least a call has
// to bring.
inline Plan make_plan(const SeqInput* seqs, int batch, int h_q, int h_kv, int head_dim,
                      int num_cus, size_t budget = SIZE_MAX) {
  Plan plan;
  if (budget != SIZE_MAX) {
    plan = make_plan(seqs, batch, h_q, h_kv, head_dim, num_cus);
    if (plan.part_rows == 0 || plan.bytes <= budget) return plan;
    plan = Plan{};
  }
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
  plan.rows.num_cus = plan.keys.num_cus = num_cus;
  plan.keys.key_split = true;
  // Row-split mode: 4 wavefronts x (32 * q_blocks) rows, 64-key tiles.
  plan.rows.q_blocks = max_rows >= 256 ? 2 : 1;
  plan.rows.shape = ModeShape{kWaves * 32 * plan.rows.q_blocks, 64};
  // Key-split mode: one 32-row block, 128-key tiles (32 per wavefront).
  plan.keys.q_blocks = 1;
  plan.keys.shape = ModeShape{32, 32 * kWaves};
  constexpr int kMinTiles = 4;
  const int64_t row_bytes = (int64_t)h_q * (head_dim + 1) * sizeof(float);
  int64_t keys_steps = 1, rows_steps = 1, keys_rows = 0, min_rows = 0;
  int keys_min_tiles = kMinTiles;
  if (!plan.rows.descs.empty()) {
    rows_steps = simple_steps(plan.rows, h_kv, gqa, num_cus);
    min_rows = split_size(plan.rows, h_kv, rows_steps, kMinTiles).part_rows;
  }
  // token rows of partials that fit the budget (the workspace's two arrays are rounded up to
  // 256 bytes each, which can cost the last rows)
  int64_t fit = (int64_t)(std::min<size_t>(budget, (size_t)1 << 60) / row_bytes);
  while (fit > 0 && partial_bytes(fit, h_q, head_dim) > budget) --fit;
  if (!plan.keys.descs.empty()) {
    keys_steps = simple_steps(plan.keys, h_kv, gqa, num_cus * 8);
    const SplitSize simple = split_size(plan.keys, h_kv, keys_steps, kMinTiles);
    const int64_t rows_min = min_rows;
    min_rows += simple.part_rows;
    // About 8 workgroups a compute unit are what a call has to bring scratch for.  Walks of 6 to 24
    // tiles are cut into about 6: a workgroup's start and end weigh more than a finer last round
    // (the timed batch of 64 decodes of 2K median, 32/8 heads, 113.0 -> 110.6 us; 178 of 1130, 32/8,
    // 166.5 -> 145.6; 183 of 8192, 8/1, 168.9 -> 145.4).  How full the last round gets decides each
    // batch: 66 of them take 0.86 to 1.07 of the time, 0.99 in the mean (35 of 4096 at 32/8, d 64,
    // 54.6 -> 56.5).  Ranges of 5 instead of 4 tiles are 1 to 2 % longer (24 decodes of 4K, 32/8
    // heads, 87.2 -> 88.9); long walks fill their rounds with 8.
    const int64_t six = simple_steps(plan.keys, h_kv, gqa, num_cus * 6);
    if (six >= 6 && six <= kShortWalkTiles) keys_steps = six;
    keys_rows = split_size(plan.keys, h_kv, keys_steps, kMinTiles).part_rows;
    // A launch that leaves compute units idle at ranges of 4 tiles, and is merged anyway, takes the
    // shortest ranges that find a unit each: a walk is a chain of trips to HBM, 1.2 us a tile.  (One
    // decode of 2048 at 32/8 heads 14.4 -> 13.6 us a pass, of 8000 19.8 -> 14.8, 8 of 2000 at 8/1
    // heads 20.4 -> 15.5, 100 of 1000 (two launches) 47.4 -> 42.3.  With more ranges than units
    // 8 of 2000 at 32/8 heads take 30.9 -> 34.6, one of 300, which needs no merge, 10.6 -> 13.7.)
    const int64_t launches = ceil_div((int64_t)plan.keys.descs.size(), kMaxInlineSeq);
    if (simple.part_rows > 0 && simple.items < num_cus * launches)
      for (int steps = 1; steps < kMinTiles; ++steps) {
        const SplitSize fine = split_size(plan.keys, h_kv, steps, steps);
        if (fine.items > num_cus * launches) continue;
        if (fine.part_rows + rows_min <= fit) {
          keys_steps = steps;
          keys_min_tiles = steps;
          keys_rows = fine.part_rows;
        }
        break;
      }
  }
  if (!plan.rows.descs.empty()) {
    if ((int)plan.rows.descs.size() <= kMaxPlannedSeqs) {
      double us, small_us;
      rows_steps = choose_steps(plan.rows, launch_walks(plan.rows, h_kv, gqa), h_kv, num_cus,
                                walk_cost(head_dim, plan.rows.q_blocks), rows_steps, kMinTiles,
                                row_bytes, fit - keys_rows, us);
      // The small workgroups as an alternative, `least` to `most` of them, where the estimate falls
      // below `worth` of the plan so far (`worth_short`: with ranges of up to `short_tiles`).
      auto try_small = [&](const WalkCost& cost, bool paired, double worth, int64_t least,
                           int64_t most, int64_t short_tiles = 0, double worth_short = 0.0) {
        LaunchPlan small = plan.rows;
        small.q_blocks = 1;
        small.paired = paired;
        small.shape.rows_per_wg = kWaves * 32;
        set_row_tiles(small, gqa);
        const LaunchWalks walks = launch_walks(small, h_kv, gqa);
        if (even_us(walks, walks.longest, num_cus, cost) >= worth * us) return;
        const int64_t steps = choose_steps(small, walks, h_kv, num_cus, cost, INT32_MAX, kMinTiles,
                                           row_bytes, fit - keys_rows, small_us);
        const int64_t slots = split_size(small, h_kv, steps, kMinTiles).slots;
        if (steps <= short_tiles) worth = worth_short;
        if (small_us < worth * us && slots >= least && slots <= most) {
          plan.rows = std::move(small);
          rows_steps = steps;
          us = small_us;
        }
      };
      const bool big = plan.rows.q_blocks == 2;
      bool behind = true;  // every chunk has a prefix as long as itself
      bool shared = true;  // every K/V stream has two small row tiles to read it
      for (const SeqDesc& sd : plan.rows.descs) {
        behind &= sd.prefix_len >= sd.chunk_len;
        shared &= (int64_t)sd.chunk_len * gqa > kWaves * 32;
      }
      // At head dim 64 they share a compute unit in pairs (else nothing is gained): half the granule,
      // short walks overlapped (14 prompts of 1K median at 8/2 heads 162 -> 150 us a pass, 12 of
      // 700 at 32/8 heads 126.0 -> 121.5; 777 tokens at 900, 32/8 heads, 31.5 -> 29.4; at 20K, 8/2
      // heads, 53.9 -> 51.6, 32/8 heads 160.8 -> 158.7; the same at 1500 tokens at 50K; 1 % longer
      // at 96 and 288 tiles where both fill the device).
      if (head_dim == 64 && big) try_small(walk_cost(64, 1), false, 0.97, num_cus + 1, INT64_MAX);
      // A launch that leaves compute units idle spreads over twice as many of them: a small
      // workgroup has its SIMDs to itself, one wavefront each, and takes two thirds to three quarters
      // of the time a tile (64 tokens at 2000, 8/1 heads, d 128, 18.3 -> 15.2 us; 300 at 1000, 32/8,
      // 29.4 -> 25.9; 200 at 8000, 8/1, 29.6 -> 26.5; d 64: 256 at 1024, 2/1, 13.4 -> 12.7; 200 at
      // 2000, 4/1, 15.4 -> 13.8; 100 at 2000, 32/8, 15.5 -> 14.4; 500 at 6000, 2/1, 17.9 -> 16.6).
      // 16 launches estimated below 0.97 at 128 take 8 to 16 % less, 25 below 0.90 at 64 (all at
      // 0.79 to 0.84) 2 to 20; at 64 from 0.94 on it is 9 % less to 7 more.  Prompts and chunks
      // longer than their prefix keep the large ones: alone they gain as well (1300 tokens at 8/1
      // 27.4 -> 25.4), eight together lose 3 %.
      if (behind && big)
        try_small(kAloneCost[head_dim == 128], false, head_dim == 128 ? 0.97 : 0.90, 1, num_cus);
      // In pairs at head dim 128 (see run_tiles), where the walks are long enough for one's end to
      // hide behind the other's.  Of 187 launches of 1 to 5 chunks, measured in each form, those with
      // ranges of more than 10 tiles gain 1 to 30 %, 4 in the middle, at estimates below 0.98 (1353
      // tokens at 19556, 16/2 heads, 246 -> 219 us; 95 at 35111, 32/8, 85.8 -> 82.2; two of 52 lose
      // 3 and 9), and nothing in the middle above; with shorter ranges they lose 2 %, and up to 16,
      // unless it is below 0.90 (405 tokens at 5443, 8/2 heads, 27.8 -> 32.1; 214 at 6376, 16/4,
      // 32.5 -> 35.0; 950 at 1900, 8/2, 29.9 -> 40.0).
      // Where 129 to 255 rows have no large form, two row tiles that share a K/V stream beat one
      // after the other by 4 to 13 % at estimates of 0.75 to 0.83 (52 tokens at 579341, 32/8 heads,
      // 726 -> 640 us; 31 at 853404, 8/1, 152 -> 138), and lose up to 7 % from 0.84 on (33 at 45708,
      // 8/2, 27.9 -> 29.7); a stream of one row tile alone wants the long ring (16 tokens at 1M 114
      // us, 127 in pairs).
      if (head_dim == 128 && behind && shared) {
        if (big)
          try_small(kPairedCost, true, 0.98, num_cus + 1, INT64_MAX, kShortPairedTiles, 0.90);
        else
          try_small(kPairedCost, true, 0.83, num_cus + 1, INT64_MAX);
      }
    }
  }
  if (!plan.rows.descs.empty())
    plan_launch(plan.rows, h_kv, gqa, rows_steps, kMinTiles, plan.part_rows);
  if (!plan.keys.descs.empty())
    plan_launch(plan.keys, h_kv, gqa, keys_steps, keys_min_tiles, plan.part_rows);

  plan.off_part_o = 0;
  plan.off_part_lse = partial_o_bytes(plan.part_rows, h_q, head_dim);
  plan.bytes = partial_bytes(plan.part_rows, h_q, head_dim);
  plan.min_bytes = partial_bytes(min_rows, h_q, head_dim);
  plan.min_part_rows = min_rows;
  return plan;
}

}  // namespace medha
