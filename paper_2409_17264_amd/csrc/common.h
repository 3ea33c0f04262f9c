// Shared definitions of the HIP attention library: work descriptors handed from
// the host planner to the kernels, vector types, small device helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace medha {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kPageSize = 16;     // tokens per KV page
constexpr int kThreads = 256;     // threads per workgroup (4 wavefronts of 64)
constexpr int kWaves = 4;
constexpr int kXcds = 8;          // accelerator dies; workgroup i is dispatched to die i % 8
constexpr int kMaxInlineSeq = 64; // sequence descriptors per kernel launch (they travel as kernel arguments)
constexpr int kShortWalkTiles = 24;   // key-split launches walking at most this many 128-key tiles per workgroup use the small ring
constexpr int kWideMergeSplits = 16;  // more KV ranges per row than this: the wide merge kernel
constexpr int64_t kLastLevelCacheBytes = (int64_t)256 << 20;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// One sequence of a launch.  Its page table (from pt_off) describes kv_len keys;
// query row j (0 <= j < chunk_len) attends to keys [0, min(prefix_len + j, kv_len - 1)]
// of them, to none if that is negative.  Chunked prefill: kv_len = prefix_len +
// chunk_len.  A decode item: chunk_len == 1, prefix_len == kv_len - 1.  A chunk
// against a KV shard: prefix_len + 1 = keys of the shard its first row sees, which
// may be <= 0 or exceed kv_len.  The sequence owns workgroup slots
// [work_start, work_start + 8 * ceil(h_kv * n_split * n_row_tiles / 8)).
struct SeqDesc {
  int64_t pt_off;           // first entry of the sequence in the page table
  int32_t q_row;            // first query token row in q
  int32_t out_row;          // first token row in out / lse
  int32_t chunk_len;        // query tokens
  int32_t prefix_len;       // see above
  int32_t work_start;       // first workgroup slot
  int32_t n_row_tiles;      // query-row tiles per KV head
  int32_t n_split;          // KV ranges the keys are split into (1 = write out directly)
  int32_t tiles_per_split;  // KV tiles per range
  int32_t part_row;         // first token row of this sequence in the partial workspace
  int32_t row_rank;         // rank of the sequence's first token row among the launch's rows
  int32_t kv_len;           // keys the page-table slice describes
  int16_t dealt;            // slots are handed out by decode_slot_dealt
  int16_t first_die;        // row-split launches: die its first items go to (see turned_slot)
};
static_assert(sizeof(SeqDesc) == 56, "SeqDesc layout");

// Kernel arguments of the attention kernels.  The sequence descriptors ride in the
// argument block itself (no host-to-device copy, no synchronisation); a batch of more
// than kMaxInlineSeq sequences takes several launches.
struct AttnArgs {
  const __bf16* q;
  const __bf16* k_pool;
  const __bf16* v_pool;
  const int32_t* page_table;
  float* out;
  float* lse;
  float* part_o;    // split-KV partial outputs  [part rows][h_q][d]
  float* part_lse;  // split-KV partial LSEs     [part rows][h_q]
  int32_t n_seq;
  int32_t h_q;
  int32_t h_kv;
  float scale_log2;  // softmax_scale * log2(e)
  SeqDesc inline_descs[kMaxInlineSeq];
};
static_assert(sizeof(AttnArgs) <= 4096, "kernel argument block too large");

// Arguments of the merge over the library's own split-KV partials.
struct MergeArgs {
  const float* part_o;
  const float* part_lse;
  float* out;
  float* lse;
  int32_t n_seq;
  int32_t h_q;
  int32_t total_rows;  // token rows of all sequences of the launch
  int32_t reserved;
  SeqDesc inline_descs[kMaxInlineSeq];
};
static_assert(sizeof(MergeArgs) <= 4096, "kernel argument block too large");

// Workgroup slot u of a sequence -> its work item.  Slot u runs on die u % 8
// (the hardware deals consecutive workgroups round-robin to the 8 dies).  The
// sequence's items, ordered (group, row tile) with group = (KV split, KV head),
// are cut into 8 equal contiguous runs, one per die: the row tiles that stream
// the same K/V range share a die and hence its L2.  Slots past a run are idle.
struct SlotItem {
  int valid, kv_head, split, row_tile;
};
__host__ __device__ inline SlotItem decode_slot(int u, int h_kv, int n_split, int n_row_tiles) {
  const int items = h_kv * n_split * n_row_tiles;
  const int per_die = (items + kXcds - 1) / kXcds;
  const int y = u / kXcds;
  const int item = (u % kXcds) * per_die + y;
  SlotItem r;
  r.valid = (y < per_die && item < items) ? 1 : 0;
  const int grp = item / n_row_tiles;
  r.row_tile = item % n_row_tiles;
  r.kv_head = grp % h_kv;
  r.split = grp / h_kv;
  return r;
}

// The same for a sequence whose row tiles walk visibly different numbers of keys: no or little
// prefix, so that the causal triangle is most of the work (later row tiles walk more, later
// splits fewer).  Equal runs would give one die all the full ranges or up to 1.75 times the mean
// work, so every die is given the same mix, longest ranges first:
//   - whole groups are dealt to the dies in turn, 8 at a time, in order of their split;
//   - the last groups, if fewer than 8 remain, deal their row tiles to the dies (there and back,
//     so that no die always has the later ones) if there are two or more for each, and are
//     otherwise cut into 8 equal runs of items.
// 3000 tokens at a 4096 prefix, 8/1 heads: 144 -> 86 us; 14 prompts at 8/2 heads, d 64:
// 238 -> 180 us; 4 prompts at 8/1 heads: 377 -> 286 us.
__host__ __device__ inline SlotItem decode_slot_dealt(int u, int h_kv, int n_split,
                                                      int n_row_tiles) {
  const int n = n_row_tiles, groups = h_kv * n_split;
  const int die = u % kXcds, y = u / kXcds;
  const int whole = groups / kXcds;  // groups a die has to itself
  SlotItem r;
  int grp;
  if (y < whole * n) {
    r.valid = 1;
    grp = (y / n) * kXcds + die;
    r.row_tile = y % n;
  } else {
    const int items = (groups - whole * kXcds) * n;
    const int per_die = (items + kXcds - 1) / kXcds, run = y - whole * n;
    const int item = n >= 2 * kXcds ? run * kXcds + (run & 1 ? kXcds - 1 - die : die)
                                    : die * per_die + run;
    r.valid = (run < per_die && item < items) ? 1 : 0;
    grp = whole * kXcds + item / n;
    r.row_tile = item % n;
  }
  r.kv_head = grp % h_kv;
  r.split = grp / h_kv;
  return r;
}

// Work item of a key-split launch's workgroup `u` (counted from the sequence's first).  One row tile,
// so nothing is shared, and the launch has no idle workgroups: one of these would hold a compute unit
// for itself on its way out, and where they come at regular intervals the others meet on some of a
// die's units.  (100 decodes of 1000 at 8/1 heads 38.7 us with the sequences' slots in eights, 27.1
// without; 20 of 5000 25.3 and 18.0; 45 of 577 at 16/4, d 128, 22.2 and 13.6; 26 of 11127 at 8/2,
// d 64, 35.4 and 32.4.)  Sequences follow one another over the dies, and each gives a die one of 8
// contiguous runs that differ by one item at most: the heads of a page are read near each other
// (item u for workgroup u: 4 shards of 262144, 8 KV heads, 640 -> 647 us; 16 decodes of 8000 at 32/8,
// d 64, 48.7 -> 50.7).
struct KeySplitItem {
  int kv_head, split;
};
__host__ __device__ inline KeySplitItem key_split_item(const SeqDesc& sd, int u, int h_kv) {
  const int items = h_kv * sd.n_split, die = u % kXcds, longer = items % kXcds;
  const int item = die * (items / kXcds) + (die < longer ? die : longer) + u / kXcds;
  return KeySplitItem{item % h_kv, item / h_kv};
}

// A sequence of few items has items for its first few dies only, and the next one as well.  So the
// dies of a row-split launch are counted from another one for every sequence, items % 8 further on:
// slot u stands for the slot that this returns.  Equal runs of several items reach less far than
// that (10 items lie two each on five dies), but counting by the dies reached is no better: 90
// launches of 2 to 24 prompts or chunks take 0.25 % more in the mean, 14 prompts of 300 at 8/1 heads
// the same, 12 chunks of 200 at 40000, 8/2 heads, 1.4 % less, 6 prompts at 16/4 heads 7 % more.
__host__ __device__ inline int turned_slot(int u, int first_die) {
  return (u & ~(kXcds - 1)) | ((u - first_die) & (kXcds - 1));
}

// Work item of slot `u` (counted from the sequence's first) of a row-split launch.  The launch's
// last sequence starts with its longest walks, so that the short ones end the launch (one prompt
// of 5959 tokens at 32/8 heads: 327 -> 306 us).  Sequences before it have others behind them to
// fill the device; eight prompts take 1.5 % longer if all do it.
__host__ __device__ inline SlotItem row_split_item(const SeqDesc& sd, int u, int h_kv,
                                                   bool last_of_launch) {
  u = turned_slot(u, sd.first_die);
  SlotItem r = sd.dealt ? decode_slot_dealt(u, h_kv, sd.n_split, sd.n_row_tiles)
                        : decode_slot(u, h_kv, sd.n_split, sd.n_row_tiles);
  if (sd.dealt && last_of_launch) r.row_tile = sd.n_row_tiles - 1 - r.row_tile;
  return r;
}

// Index of the last of n <= 64 ascending keys that is <= value, key(i) being key i; n >= 1 and
// key(0) <= value.  All 64 lanes have to be active.  A wavefront that asks for one value reads a
// key per lane and counts: one trip to memory where a binary search takes six dependent ones
// (eight prompts, 13291 tokens: the append 26.3 -> 23.2 us; 64 decodes: the merge 7.6 -> 6.6 us).
template <class Key>
__device__ __forceinline__ int find_last(int n, int value, Key key) {
  if (n == 1) return 0;
  const int v0 = __builtin_amdgcn_readfirstlane(value);
  if (__all(value == v0)) {
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int mine = key(min(lane, n - 1));
    return __popcll(__ballot(lane < n && mine <= v0)) - 1;
  }
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (key(mid) <= value) lo = mid; else hi = mid - 1;
  }
  return lo;
}
static_assert(kMaxInlineSeq <= 64, "find_last counts one key per lane");

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Value held by the lane 32 positions away (lane ^ 32), via the gfx950
// half-wave swap: swap(x, x) returns {x of low half, x of high half} in every lane.
__device__ __forceinline__ float other_half(float x, int hi_half) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  unsigned o = hi_half ? r[0] : r[1];
  return __builtin_bit_cast(float, o);
}
__device__ __forceinline__ float max_halves(float x) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

}  // namespace medha
