"""CPU-only tests of the C-ABI library: it loads, exports every symbol the
header declares, and its host-side planner covers the work exactly once."""
import os
import re

import numpy as np
import pytest

import paper_2409_17264_amd as medha
from paper_2409_17264_amd import binding, policy, yardstick

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    declared = {}
    for name in sorted(os.listdir(os.path.join(ROOT, "include"))):
        header = open(os.path.join(ROOT, "include", name)).read()
        body = re.sub(r"/\*.*?\*/", "", header, flags=re.S)      # drop comments
        declared[name] = set(re.findall(r"\b(medha_[a-z0-9_]+)\s*\(", body))
    assert sorted(declared) == ["medha.h", "medha_policy.h", "medha_yardstick.h"]
    product = declared["medha.h"] | declared["medha_policy.h"]
    bound = set(binding.EXPORTS) | set(policy.EXPORTS)
    assert product == bound, product ^ bound
    assert declared["medha_yardstick.h"] == set(yardstick.EXPORTS)
    lib = medha.load_library()
    for name in product:
        assert getattr(lib, name) is not None
    ylib = yardstick.load_library()
    for name in yardstick.EXPORTS:
        assert getattr(ylib, name) is not None
        assert not hasattr(lib, name)          # the yardsticks are not in the product's ABI
    assert lib.medha_abi_version() == 1
    assert lib.medha_strerror(0) == b"ok"
    assert b"workspace" in lib.medha_strerror(-3)


def test_workspace_queries_reject_bad_arguments():
    assert medha.chunked_prefill_workspace_bytes([10], [0], 8, 2, 128) == 0       # empty chunk
    assert medha.chunked_prefill_workspace_bytes([10], [4], 7, 2, 128) == 0       # 7 % 2
    assert medha.chunked_prefill_workspace_bytes([10], [4], 8, 2, 96) == 0        # head_dim
    assert medha.decode_partial_workspace_bytes([-1], 8, 2, 128) == 0
    assert medha.decode_partial_workspace_bytes([5], 64, 1, 128) >= 256           # group > 32: row-split
    assert medha.chunked_prefill_workspace_bytes([100], [16], 8, 2, 128) >= 256


def _simple_rule_rows(prefix, chunk, h_q, h_kv, num_cus):
    """Partial token rows if the keys are cut into about one workgroup per compute unit (key-split
    launches: eight): the least workspace a call has to bring."""
    gqa, total = h_q // h_kv, 0
    rows_per_wg = 256 if max(c * gqa for c in chunk) >= 256 else 128
    for mode, rows, tile, target in ((0, rows_per_wg, 64, num_cus), (1, 32, 128, 8 * num_cus)):
        seqs = [(h_kv * -(-c * gqa // rows), -(-(p + c) // tile), c)
                for p, c in zip(prefix, chunk) if (c * gqa <= 32) == (mode == 1)]
        if sum(wgs for wgs, _, _ in seqs) >= target:
            continue
        steps = max(1, -(-sum(wgs * tiles for wgs, tiles, _ in seqs) // target))
        for _, tiles, c in seqs:
            tiles = max(1, tiles)
            n = max(1, min(-(-tiles // steps), max(1, tiles // 4)))
            n = -(-tiles // -(-tiles // n))
            total += n * c if n > 1 else 0
    return total


def _walks_differ(prefix, chunk, gqa, e):
    """Whether the causal triangle makes the row tiles' walks differ by more than a sixteenth."""
    first, last = (-(-min(prefix + chunk, prefix + -(-rows // gqa)) // 64)
                   for rows in (min(e.rows_per_wg, chunk * gqa), chunk * gqa))
    return e.mode == 0 and e.n_row_tiles > 1 and last - first > last // 16


def _check_plan(prefix, chunk, h_q, h_kv, d, num_cus):
    entries, grid_rows, grid_keys, ws = medha.describe_plan(prefix, chunk, h_q, h_kv, d, num_cus)
    gqa = h_q // h_kv
    spans = {0: [], 1: []}
    part_rows = 0
    for seq, (p, c, e) in enumerate(zip(prefix, chunk, entries)):
        n_rows = c * gqa
        assert e.mode == (1 if n_rows <= 32 else 0)
        assert e.rows_per_wg in ((32,) if e.mode else (128, 256))
        assert e.tile_keys == (128 if e.mode else 64)
        assert e.n_row_tiles == -(-n_rows // e.rows_per_wg)
        kv_tiles = max(1, -(-(p + c) // e.tile_keys))
        # the splits tile the KV axis: enough to cover it, none empty
        assert e.n_split * e.tiles_per_split >= kv_tiles
        assert (e.n_split - 1) * e.tiles_per_split < kv_tiles
        items = h_kv * e.n_split * e.n_row_tiles
        assert e.n_slots == 8 * -(-items // 8)
        spans[e.mode].append((e.work_start, e.n_slots, min(e.tiles_per_split, kv_tiles)))
        # every (kv head, split, row tile) is owned by exactly one slot
        slots = {}
        for s in range(e.n_slots):
            it = medha.describe_plan_slot(prefix, chunk, h_q, h_kv, d, num_cus, e.mode,
                                          e.work_start + s)
            if it is not None:
                assert it[0] == seq
                it = it[1:]
                assert it not in slots
                assert 0 <= it[0] < h_kv and 0 <= it[1] < e.n_split and 0 <= it[2] < e.n_row_tiles
                slots[it] = s
        assert len(slots) == items
        # row tiles sharing (kv head, split) sit on one die (slot % 8): of a sequence with a long
        # prefix when they fit; of one whose row tiles walk different numbers of keys the whole
        # groups of each die
        dies, per_die = {}, -(-items // 8)
        for it, s in slots.items():
            dies.setdefault(it[:2], set()).add(s % 8)
        if _walks_differ(p, c, gqa, e):
            alone = h_kv * e.n_split // 8 * 8
            assert all(len(dies[g % h_kv, g // h_kv]) == 1 for g in range(alone))
        elif per_die % e.n_row_tiles == 0:
            assert all(len(v) == 1 for v in dies.values())
        if e.n_split > 1:
            part_rows += e.n_split * c
    # per launch the sequences' slot ranges tile [0, grid) in some order, and that order puts
    # the workgroups with the longest walks first
    for mode, grid in ((0, grid_rows), (1, grid_keys)):
        end, prev_walk = 0, None
        for start, n_slots, walk in sorted(spans[mode]):
            assert start == end
            end += n_slots
            assert prev_walk is None or walk <= prev_walk
            prev_walk = walk
        assert end == grid
    rows = max(part_rows, _simple_rule_rows(prefix, chunk, h_q, h_kv, num_cus))
    need = rows * h_q * (d + 1) * 4
    assert need <= ws <= need + 1024 + 64 * len(prefix)
    return entries, grid_rows, grid_keys


def test_plans_of_the_named_workloads():
    # cfg2: 8 kv heads x 32 row tiles of 256 rows fill 256 compute units, no KV split
    e, gr, gk = _check_plan([32768], [2048], 32, 8, 128, 256)
    assert (e[0].n_row_tiles, e[0].n_split, gr, gk) == (32, 1, 256, 0)
    # cfg4: few row tiles -> KV split so that about 256 workgroups exist
    for c, tiles, split in [(512, 16, 16), (1024, 32, 8), (2048, 64, 4), (4096, 128, 2),
                            (8192, 256, 1)]:
        e, gr, _ = _check_plan([1 << 20], [c], 8, 1, 128, 256)
        assert (e[0].n_row_tiles, e[0].n_split) == (tiles, split) and gr == 256
    # cfg3: 4 shards x 8 kv heads, split into 8 workgroups per compute unit
    e, _, gk = _check_plan([262143] * 4, [1] * 4, 32, 8, 128, 256)
    assert all(x.mode == 1 and x.n_split == 64 for x in e) and gk == 2048
    # cfg1
    e, gr, _ = _check_plan([1024], [256], 2, 1, 64, 256)
    assert e[0].n_row_tiles == 4 and e[0].n_split > 1


def test_plans_of_ragged_batches():
    rng = np.random.default_rng(0)
    for trial in range(30):
        batch = int(rng.integers(1, 12))
        h_kv = int(rng.choice([1, 2, 4, 8]))
        gqa = int(rng.choice([1, 2, 4, 8]))
        prefix = [int(x) for x in rng.integers(0, 70000, batch)]
        chunk = [int(rng.choice([1, 1, 2, 5, 40, 300, 2000])) for _ in range(batch)]
        _check_plan(prefix, chunk, h_kv * gqa, h_kv, int(rng.choice([64, 128])),
                    int(rng.choice([8, 64, 256, 304])))
    # a decode over zero keys is planned too
    e, _, _ = _check_plan([-1, 0], [1, 1], 8, 2, 128, 256)
    assert e[0].n_split == 1


@pytest.mark.parametrize("prefix,chunk,h_q,h_kv,d", [
    ([10000], [7885], 8, 1, 128),             # planned without a cut, which the simple rule makes
    ([36000], [1700], 8, 1, 128),             # more ranges than the simple rule's
    ([1024], [256], 2, 1, 64),
    ([0] * 5, [300, 1, 2000, 77, 1], 8, 2, 64),
])
def test_described_workspace_is_what_a_call_has_to_bring(prefix, chunk, h_q, h_kv, d):
    described = medha.describe_plan(prefix, chunk, h_q, h_kv, d, 256)[3]
    assert described == medha.chunked_prefill_workspace_bytes(prefix, chunk, h_q, h_kv, d)


@pytest.mark.parametrize("prefix,chunk,h_q,h_kv,d", [
    ([300007], [1500], 8, 1, 128),            # 47 row tiles: 6 ranges would be 282 workgroups
    ([65000] * 4, [600] * 4, 8, 1, 128),      # 4 x 19
    ([20011], [777], 32, 8, 64),              # 8 x 13
    ([50000], [4864], 8, 1, 128),             # 152: more than half the device, unsplit
    ([9000], [33], 8, 1, 128),                # two row tiles, ranges of the shortest kind
    ([9000], [31], 8, 1, 128),                # the same of small workgroups
])
def test_row_split_launches_fill_whole_rounds_of_the_device(prefix, chunk, h_q, h_kv, d):
    """Time of the planned launch in tiles, workgroups of one length each: no more than 1.15 times
    the tiles spread evenly over 256 compute units plus a fixed cost of 12 tiles a round."""
    e, grid, _ = _check_plan(prefix, chunk, h_q, h_kv, d, 256)
    slots = 512 if d == 64 and e[0].rows_per_wg == 128 else 256
    rounds = -(-grid // slots)
    tiles = sum(h_kv * x.n_row_tiles * -(-(p + c) // 64) for x, p, c in zip(e, prefix, chunk))
    assert rounds * max(x.tiles_per_split for x in e) <= 1.15 * tiles / slots + 12 * rounds


@pytest.mark.parametrize("prefix,chunk,h_q,h_kv,d,rows,most", [
    # small workgroups alone on a compute unit, whatever the number of KV heads
    ([1024], [256], 2, 1, 64, 128, 256), ([2000], [64], 8, 1, 64, 128, 256),
    ([2000], [200], 4, 1, 64, 128, 256), ([6000], [512], 2, 1, 64, 128, 256),
    # in pairs where the walks are long; with short ranges the large ones are faster
    ([19556], [1353], 16, 2, 128, 128, 512), ([35111], [95], 32, 8, 128, 128, 512),
    ([5443], [405], 8, 2, 128, 256, 256), ([6376], [214], 16, 4, 128, 256, 256),
    ([1900], [950], 8, 2, 128, 256, 256), ([865], [695], 16, 2, 128, 256, 256),
    # 129 to 255 rows: pairs for long streams, one after the other for the rest
    ([579341], [52], 32, 8, 128, 128, 512), ([853404], [31], 8, 1, 128, 128, 512),
    ([45708], [33], 8, 2, 128, 128, 256), ([31761], [60], 32, 8, 128, 128, 256),
])
def test_small_workgroups_where_they_are_faster(prefix, chunk, h_q, h_kv, d, rows, most):
    e, grid, _, _ = medha.describe_plan(prefix, chunk, h_q, h_kv, d, 256)
    assert e[0].rows_per_wg == rows and (256 < grid <= 512 if most == 512 else grid <= most)


def test_stream_handle_without_the_private_function(monkeypatch):
    import importlib.util
    import types
    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    spec = importlib.util.spec_from_file_location("binding_again", binding.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._stream() == 1234


def test_bench_refuses_more_than_one_gpu_and_finds_its_traffic_figures():
    import subprocess
    import sys
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode != 0 and "one GPU" in res.stderr
    # every counter summary bench.py reads an HBM figure from is there and holds one
    src = open(os.path.join(ROOT, "bench.py")).read()
    names = set(re.findall(r'"([a-z0-9_]+\.txt)"', src))
    names |= {f"prefill_kernel_cfg4_c{c}.txt" for c in (32, 128, 512, 1024, 2048, 4096, 8192)}
    assert {"prefill_kernel_cfg2.txt", "decode_kernel_cfg3.txt", "mixed_cfg5.txt"} <= names
    for name in sorted(names):
        lines = [l for l in open(os.path.join(ROOT, "profiles", name))
                 if l.startswith("hbm_bytes_per_launch")]
        assert lines and float(lines[0].split("=")[1].split()[0]) > 1e6, name


def test_described_slots_of_a_prompt_are_the_kernels():
    """One prompt of 5959 tokens at 32/8 heads, 94 row tiles for each KV head: a head per die, the
    longest walks first.  A long prefix keeps equal runs of ascending row tiles."""
    got = [medha.describe_plan_slot([0], [5959], 32, 8, 128, 256, 0, s) for s in range(24)]
    assert got == [(0, s % 8, 0, 93 - s // 8) for s in range(24)]
    got = [medha.describe_plan_slot([32768], [2048], 32, 8, 128, 256, 0, s) for s in range(24)]
    assert got == [(0, s % 8, 0, s // 8) for s in range(24)]
    # 64 sequences go out in one launch; each launch has a last sequence of its own
    first = [medha.describe_plan_slot([0] * 66, [300] * 66, 8, 8, 128, 256, 0, 16 * i)
             for i in (0, 62, 63, 64, 65)]
    assert first == [(0, 0, 0, 0), (62, 0, 0, 0), (63, 0, 0, 1), (64, 0, 0, 0), (65, 0, 0, 1)]
    for bad in (dict(mode=2, slot=0), dict(mode=0, slot=-1), dict(mode=0, slot=752), dict(mode=1, slot=0)):
        with pytest.raises(medha.MedhaError):
            medha.describe_plan_slot([0], [5959], 32, 8, 128, 256, bad["mode"], bad["slot"])
