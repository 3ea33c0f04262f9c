"""The row-split planner's own functions, compiled for the host (CPU), and what planning costs."""
import ctypes
import os
import subprocess
import time

import numpy as np
import pytest

import paper_2409_17264_amd as medha
from paper_2409_17264_amd import binding
from paper_2409_17264_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

PRELUDE = r"""
#include <cmath>
#include <cstdio>
#include <functional>
#include <queue>
#include <random>
#include "planner.h"
using namespace medha;
static std::mt19937 rng(7);
static int log_int(double lo, double hi) {
  std::uniform_real_distribution<double> u(0, 1);
  return (int)std::round(lo * std::pow(hi / lo, u(rng)));
}
static std::vector<SeqInput> draw(int n) {
  std::vector<SeqInput> s;
  int row = 0;
  for (int i = 0; i < n; ++i) {
    const int chunk = log_int(1, 8192), prefix = rng() % 2 ? 0 : log_int(1, 300000);
    s.push_back({0, row, row, chunk, prefix, rng() % 8 ? -1 : log_int(1, 100000)});
    row += chunk;
  }
  return s;
}
"""

ESTIMATE = PRELUDE + r"""
// the list schedule, one workgroup at a time
static double plain_makespan(std::vector<WalkGroup> g, int64_t machines, const WalkCost& wc) {
  std::sort(g.begin(), g.end(), [](auto& a, auto& b) { return a.tiles > b.tiles; });
  std::priority_queue<double, std::vector<double>, std::greater<double>> free_at;
  for (int64_t i = 0; i < machines; ++i) free_at.push(0.0);
  double end = 0;
  for (auto& x : g)
    for (int64_t i = 0; i < x.count; ++i) {
      const double t = free_at.top() + (wc.fixed_us + (double)x.tiles * wc.tile_us);
      free_at.pop();
      free_at.push(t);
      end = std::max(end, t);
    }
  return end;
}
// choose_steps without its bounds and its search
static int64_t plain_choice(const LaunchPlan& lp, const LaunchWalks& lw, int h_kv, int cus,
                            const WalkCost& wc, int64_t base, int64_t row_bytes, int64_t max_rows) {
  const int64_t slots = (int64_t)cus * wc.wgs_per_cu;
  if (lw.unsplit >= kMaxWaves * slots || lw.longest <= 4) return base;
  double us = launch_us(lp, lw, h_kv, cus, wc, base, 4, row_bytes);
  const int64_t allowed = std::min(max_rows, kMaxPartialBytes / row_bytes);
  int64_t best = base, prev = base;
  auto consider = [&](int64_t steps) {
    if (steps == prev || split_size(lp, h_kv, steps, 4).part_rows > allowed) return;
    prev = steps;
    const double t = launch_us(lp, lw, h_kv, cus, wc, steps, 4, row_bytes);
    if (t < 0.97 * us) { best = steps; us = t; }
  };
  consider(lw.longest);
  for (int w = 1; w <= kMaxWaves; ++w) {
    if (split_size(lp, h_kv, lw.longest, 4).slots > w * slots) continue;
    int64_t lo = 4, hi = lw.longest;
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      if (split_size(lp, h_kv, mid, 4).slots <= w * slots) hi = mid; else lo = mid + 1;
    }
    consider(lo);
    if (lo <= 4) break;
  }
  return best;
}
int main() {
  for (int it = 0; it < 3000; ++it) {
    std::vector<WalkGroup> g;
    for (int n = 1 + rng() % 40; n > 0; --n) g.push_back({1 + (int64_t)(rng() % 90), 1 + (int64_t)(rng() % 50)});
    const int64_t machines = 1 + rng() % 64;
    const WalkCost wc = walk_cost(it & 1 ? 64 : 128, 1 + it % 3 / 2);
    auto copy = g;
    const double want = plain_makespan(g, machines, wc), got = makespan(copy, machines, wc);
    if (std::fabs(got - want) > 1e-9 * want) { std::printf("makespan %g %g\n", got, want); return 1; }
  }
  const int heads[][2] = {{1, 1}, {8, 1}, {8, 2}, {32, 8}, {12, 3}, {128, 16}};
  int moved = 0;
  for (int it = 0; it < 3000; ++it) {
    const auto& hh = heads[rng() % 6];
    const int gqa = hh[0] / hh[1], d = rng() & 1 ? 64 : 128, qb = 1 + rng() % 2;
    const int cus = rng() % 4 ? 256 : 8 * (1 + rng() % 40);
    LaunchPlan lp;
    for (auto& s : draw(1 + rng() % (it % 3 ? 3 : 16))) {
      SeqDesc sd{};
      sd.chunk_len = s.chunk_len;
      sd.prefix_len = s.prefix_len;
      sd.kv_len = s.kv_len >= 0 ? s.kv_len : s.prefix_len + s.chunk_len;
      lp.descs.push_back(sd);
    }
    lp.shape = ModeShape{kWaves * 32 * qb, 64};
    const int64_t base = simple_steps(lp, hh[1], gqa, cus);
    const LaunchWalks lw = launch_walks(lp, hh[1], gqa);
    const int64_t row_bytes = hh[0] * (d + 1) * 4, rows = rng() % 3 ? (int64_t)1 << 40 : rng() % 100000;
    double us;
    const int64_t got = choose_steps(lp, lw, hh[1], cus, walk_cost(d, qb), base, 4, row_bytes, rows, us);
    const int64_t want = plain_choice(lp, lw, hh[1], cus, walk_cost(d, qb), base, row_bytes, rows);
    if (got != want) { std::printf("choice %ld %ld\n", (long)got, (long)want); return 1; }
    moved += got != base;
  }
  std::printf("ok %d\n", moved);
  return moved > 300 ? 0 : 1;
}
"""

BUDGET = PRELUDE + r"""
// chunks behind a prefix, which choose between three forms of workgroups
static std::vector<SeqInput> draw_behind(int n) {
  std::vector<SeqInput> s;
  int row = 0;
  for (int i = 0; i < n; ++i) {
    const int chunk = log_int(20, 2500), prefix = log_int(chunk, 80000);
    s.push_back({0, row, row, chunk, prefix, -1});
    row += chunk;
  }
  return s;
}
static bool same(const Plan& a, const Plan& b) {
  for (auto pair : {std::make_pair(&a.rows, &b.rows), std::make_pair(&a.keys, &b.keys)}) {
    const LaunchPlan &x = *pair.first, &y = *pair.second;
    if (x.n_slots != y.n_slots || x.q_blocks != y.q_blocks || x.paired != y.paired ||
        x.seq_index != y.seq_index) return false;
    for (size_t i = 0; i < x.descs.size(); ++i)
      if (x.descs[i].n_split != y.descs[i].n_split || x.descs[i].part_row != y.descs[i].part_row ||
          x.descs[i].tiles_per_split != y.descs[i].tiles_per_split) return false;
  }
  return a.bytes == b.bytes;
}
static int less = 0;
static bool check(const std::vector<SeqInput>& seqs, int h_q, int h_kv, int d) {
  auto plan = [&](size_t budget) {
    return make_plan(seqs.data(), (int)seqs.size(), h_q, h_kv, d, 256, budget);
  };
  const Plan full = plan(SIZE_MAX);
  const size_t need = full.workspace_bytes();
  // any workspace of the reported size or more: one plan
  for (size_t b : {need, need + 1, 2 * need, need + 4096})
    if (!same(full, plan(b))) {
      std::printf("another plan with %zu of %zu: heads %d/%d d %d, %d tokens at %d\n", b, need, h_q, h_kv,
                  d, seqs[0].chunk_len, seqs[0].prefix_len);
      return false;
    }
  // less, down to what a call has to bring: a plan that fits
  if (full.min_bytes < need)
    for (size_t b : {full.min_bytes, (full.min_bytes + need) / 2, need - 1}) {
      const Plan p = plan(b);
      if (p.bytes > b || p.min_bytes != full.min_bytes) { std::printf("%zu of %zu\n", p.bytes, b); return false; }
      less += !same(full, p);
    }
  // less still: the simple rule's plan or one without more partials, for the call to refuse
  if (plan(0).bytes > std::max(full.min_bytes, full.bytes)) { std::puts("grew"); return false; }
  return true;
}
int main() {
  const int heads[][2] = {{1, 1}, {8, 1}, {8, 2}, {32, 8}, {12, 3}, {16, 2}, {16, 4}};
  for (int it = 0; it < 30000; ++it) {
    const auto& hh = heads[rng() % 7];
    const int d = rng() & 1 ? 64 : 128;
    if (!check(it % 6 ? draw_behind(1 + rng() % 3) : draw(1 + rng() % (it % 3 ? 3 : 24)), hh[0], hh[1], d))
      return 1;
  }
  // (of 5 million draws: the form of the workgroups changed with the workspace)
  const int rare[][3][2] = {{{583, 21}, {934, 319}, {78031, 22}}, {{55830, 27}, {448, 336}, {552, 73}}};
  for (const auto& r : rare) {
    std::vector<SeqInput> s;
    int row = 0;
    for (const auto& x : r) {
      s.push_back({0, row, row, x[1], x[0], -1});
      row += x[1];
    }
    if (!check(s, 32, 8, 128)) return 1;
  }
  std::printf("ok %d\n", less);
  return less > 200 ? 0 : 1;
}
"""


def _run(tmp_path, source):
    src, exe = str(tmp_path / "planner.hip"), str(tmp_path / "planner")
    with open(src, "w") as f:
        f.write(source)
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-inline-asm",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I",
                          os.path.join(ROOT, "paper_2409_17264_amd", "csrc"), src, "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "ok" in run.stdout, run.stdout + run.stderr


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_estimates_and_choices_are_those_of_the_plain_search(tmp_path):
    _run(tmp_path, ESTIMATE)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_one_plan_for_every_workspace_that_is_large_enough(tmp_path):
    """The plan, and with it every bit of the result, is one and the same with all workspaces of
    the reported size or more; with less it fits what is there."""
    _run(tmp_path, BUDGET)


def _plan_us(prefix, chunk, h_q, h_kv, d):
    """Host time of one plan: the best of many, so that other load on the machine does not count."""
    lib = medha.load_library()
    entries = (binding.PlanEntry * len(prefix))()
    a, b, w = ctypes.c_int32(0), ctypes.c_int32(0), ctypes.c_size_t(0)
    args = (np.asarray(prefix, np.int32).tobytes(), np.asarray(chunk, np.int32).tobytes(),
            len(prefix), h_q, h_kv, d, 256, entries, ctypes.byref(a), ctypes.byref(b),
            ctypes.byref(w))
    best = float("inf")
    for _ in range(40):
        t0 = time.perf_counter()
        for _ in range(10):
            lib.medha_describe_plan(*args)
        best = min(best, (time.perf_counter() - t0) / 10)
    return best * 1e6


def test_planning_costs_a_few_microseconds():
    """In units of the cheapest plan, 64 decodes under the simple rule (5 to 10 us): batches of
    prompts at small heads take 2 to 4 of them, simulating every candidate took 8 to 15; the
    largest prompt there can be took a thousand."""
    unit = _plan_us([2000] * 64, [1] * 64, 32, 8, 128)
    for h_q, h_kv, n, median in [(2, 1, 16, 1024), (8, 2, 16, 1024), (2, 1, 9, 2200), (8, 1, 16, 4096)]:
        chunk = [int(x) for x in wl.lognormal_lengths(n, 7, median, 1.0, 16, 8192)]
        cost = _plan_us([0] * n, chunk, h_q, h_kv, 64)
        assert cost < 6 * unit, (h_q, h_kv, n, median, cost, unit)
    assert _plan_us([0], [2**31 - 1], 32, 8, 64) < 6 * unit
