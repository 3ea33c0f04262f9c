"""Order in which the row-split kernel's workgroups take their work (CPU): the kernel's own slot
functions, compiled for the host."""
import os
import subprocess

import pytest

import paper_2409_17264_amd as medha

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

SOURCE = r"""
#include <cstdio>
#include <set>
#include "common.h"
using namespace medha;
int main() {
  for (int h : {1, 2, 3, 4, 8, 12})
    for (int ns : {1, 2, 3, 5, 8, 17})
      for (int n = 1; n <= 260; n = n < 70 ? n + 1 : n + 19) {
        const int items = h * ns * n, slots = 8 * ((items + 7) / 8);
        std::set<int> seen;
        long work[8] = {}, all = 0;
        int count[8] = {};
        for (int u = 0; u < slots; ++u) {
          const SlotItem a = decode_slot_dealt(u, h, ns, n);
          if (!a.valid) continue;
          if (a.kv_head < 0 || a.kv_head >= h || a.split < 0 || a.split >= ns || a.row_tile < 0 ||
              a.row_tile >= n || !seen.insert((a.split * h + a.kv_head) * n + a.row_tile).second) {
            std::printf("bad slot %d of h %d ns %d n %d\n", u, h, ns, n);
            return 1;
          }
          if (a.split == 0) work[u % 8] += a.row_tile + 1;  // the full ranges of a triangle
          all += a.split == 0 ? a.row_tile + 1 : 0;
          ++count[u % 8];
        }
        if ((int)seen.size() != items) { std::printf("lost: h %d ns %d n %d\n", h, ns, n); return 1; }
        // many row tiles that the dies share: no die has more than its part and two tiles a group
        if (n >= 64 && h * ns < 8)
          for (int d = 0; d < 8; ++d)
            if (work[d] > all / 8 + 2L * h * n) { std::printf("uneven: h %d ns %d n %d\n", h, ns, n); return 1; }
      }
  // key-split launches: workgroup u of a sequence that starts at workgroup `start`
  for (int h : {1, 2, 3, 4, 8, 10, 12})
    for (int ns = 1; ns <= 70; ++ns) {
      SeqDesc sd{};
      sd.n_split = ns;
      std::set<int> seen;
      int count[8] = {}, before[8];
      for (int u = 0; u < h * ns; ++u) {
        const KeySplitItem k = key_split_item(sd, u, h);
        const int item = k.split * h + k.kv_head, die = u % 8;
        if (k.kv_head < 0 || k.kv_head >= h || k.split < 0 || k.split >= ns ||
            !seen.insert(item).second || (count[die]++ > 0 && item != before[die] + 1)) {
          std::printf("bad workgroup %d of h %d ns %d\n", u, h, ns);
          return 1;
        }
        before[die] = item;
      }
      for (int d = 0; d < 8; ++d)
        if (count[d] != h * ns / 8 + (d < h * ns % 8)) { std::printf("run: h %d ns %d\n", h, ns); return 1; }
    }
  std::puts("ok");
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_dealt_slots_cover_every_item_once_and_evenly(tmp_path):
    src, exe = str(tmp_path / "slots.hip"), str(tmp_path / "slots")
    with open(src, "w") as f:
        f.write(SOURCE)
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-inline-asm",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I",
                          os.path.join(ROOT, "paper_2409_17264_amd", "csrc"), src, "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "ok" in run.stdout, run.stdout + run.stderr


@pytest.mark.parametrize("prefix,chunk,h_q,h_kv,mode", [
    ([900 + 31 * i for i in range(40)], [1] * 40, 8, 1, 1),      # one to four ranges of one head
    ([300 * (1 + i % 5) for i in range(33)], [1] * 33, 8, 2, 1),
    ([6143] * 24, [1] * 24, 8, 1, 1),                            # 12, 12, 20, 28 and 10 items each
    ([1535] * 32, [1] * 32, 32, 4, 1),
    ([2600] * 24, [1] * 24, 8, 4, 1),
    ([3583] * 24, [1] * 24, 8, 4, 1),
    ([5000] * 20, [1] * 20, 8, 1, 1),
    ([999] * 100, [1] * 100, 8, 1, 1),                           # two launches
    ([0] * 12, [90 + 16 * i for i in range(12)], 8, 1, 0),       # prompts of 3 to 9 row tiles
])
def test_sequences_of_few_items_are_spread_over_the_dies(prefix, chunk, h_q, h_kv, mode):
    entries, grid_rows, grid_keys, _ = medha.describe_plan(prefix, chunk, h_q, h_kv, 128, 256)
    items, dies = 0, [0] * 8
    order = sorted(range(len(entries)), key=lambda i: entries[i].work_start)
    launch = {seq: i // 64 for i, seq in enumerate(order)}  # 64 sequences each
    rank = [0] * 2
    for s in range(grid_keys if mode else grid_rows):
        it = medha.describe_plan_slot(prefix, chunk, h_q, h_kv, 128, 256, mode, s)
        if it is not None:
            items += 1
            # workgroup -> die: a row-split launch has a workgroup per slot, a key-split one leaves
            # the idle ones out
            dies[(rank[launch[it[0]]] if mode else s) % 8] += 1
            rank[launch[it[0]]] += 1
    assert items == sum(h_kv * e.n_split * e.n_row_tiles for e in entries)
    if mode:
        assert max(dies) - min(dies) <= 1 + max(launch.values()), dies
    else:
        # equal runs of a sequence differ by one item, and those of more than 8 items by their last run
        assert max(dies) <= items / 8 + len(entries) / 2 + 1, dies
