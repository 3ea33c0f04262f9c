"""The workloads this library is timed on, through its public entry points.

Four kinds of call sequence, each written the way a serving program makes it:

  prefill     one chunk of one long request against its paged KV-cache prefix, output
              and workspace buffers kept from call to call;
  iteration   one scheduler iteration: the new tokens' keys and values are appended to the
              cache, then one attention call over the whole batch (a prefill chunk and / or
              decodes, or a set of fresh prompts), nothing kept but the inputs;
  kvp_decode  one query token against S contiguous KV shards, then the LSE merge;
  kvp_chunk   one prefill chunk against S contiguous KV shards, then the LSE merge.

Inputs follow ``workloads.py``: i.i.d. N(0,1) queries, keys and values in bf16, 16-token
pages dealt out by a seeded permutation of the pool, softmax scale 1/sqrt(d), log-normal
context lengths.  A case holds every size, so that inputs of different seeds have the same
shapes; the seed draws values and page tables.
"""
import math

import numpy as np
import torch

import paper_2409_17264_amd as medha
from paper_2409_17264_amd import workloads as wl

PAGE = wl.PAGE_SIZE
MAX_FLOPS = 3.54e13   # the largest listed case: an 8192-token chunk at a 1M-token prefix
MAX_KV_BYTES = 4.30e9  # the KV cache of one 1M-token request at 8 KV heads

# (query heads, KV heads, head dim): the full 8B-sized layer, one GPU's share of the
# 70B-sized one, and the small-head shapes of the tests
HEADS = [(32, 8, 128), (32, 8, 128), (8, 1, 128), (8, 1, 128), (8, 2, 128), (32, 8, 64),
         (8, 2, 64), (2, 1, 64)]


def listed():
    return [
        # one chat request generating its next token: launch latency and host work
        dict(name="decode_one", kind="iteration", h_q=32, h_kv=8, d=128, prefix=0, chunk=0,
             prompts=0, decodes=1, median=2048, lengths=0),
        # the smallest prefill: 2 query heads on one KV head, d 64, 1024 + 256 tokens
        dict(name="prefill_tiny", kind="prefill", h_q=2, h_kv=1, d=64, prefix=1024, chunk=256),
        # a decode-only iteration of a busy server: 64 requests, log-normal contexts
        dict(name="decode_batch", kind="iteration", h_q=32, h_kv=8, d=128, prefix=0, chunk=0,
             prompts=0, decodes=64, median=2048, lengths=5007),
        # fresh prompts of assorted lengths entering together (no prefix, causal only)
        dict(name="prompt_batch", kind="iteration", h_q=32, h_kv=8, d=128, prefix=0, chunk=0,
             prompts=8, decodes=0, median=1024, lengths=11),
        # head dim 64, odd prefix and chunk: what a scheduler that sizes chunks by time sends
        dict(name="prefill_d64_odd", kind="prefill", h_q=32, h_kv=8, d=64, prefix=20011,
             chunk=777),
        # the 8B-sized layer at a 32K prefix
        dict(name="prefill_32k", kind="prefill", h_q=32, h_kv=8, d=128, prefix=32768, chunk=2048),
        # one GPU's share of the 70B-sized layer, a time-sized chunk at an odd prefix
        dict(name="prefill_odd", kind="prefill", h_q=8, h_kv=1, d=128, prefix=300007, chunk=1500),
        # adaptive chunking's end of the range: 32 tokens at a 1M-token prefix
        dict(name="prefill_1m_c32", kind="prefill", h_q=8, h_kv=1, d=128, prefix=1 << 20,
             chunk=32),
        # and its beginning: the largest single call
        dict(name="prefill_1m_c8192", kind="prefill", h_q=8, h_kv=1, d=128, prefix=1 << 20,
             chunk=8192),
        # KV-cache-parallel decode of one 1M-token request, 4 shards, merged
        dict(name="kvp_decode_1m", kind="kvp_decode", h_q=32, h_kv=8, d=128, prefix=(1 << 20) - 1,
             chunk=1, shards=4),
        # KV-cache-parallel prefill chunk at a prefix that is no multiple of anything
        dict(name="kvp_chunk", kind="kvp_chunk", h_q=8, h_kv=1, d=128, prefix=262150, chunk=600,
             shards=4),
        # a long request's chunk packed with 64 decodes in one call
        dict(name="mixed", kind="iteration", h_q=32, h_kv=8, d=128, prefix=524288, chunk=1024,
             prompts=0, decodes=64, median=2048, lengths=5007),
    ]


def _log_int(rng, lo, hi):
    """Integer spread over its logarithm in [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    h_q, h_kv, d = rng.choice(HEADS)
    kind = rng.choice(["prefill", "prefill", "prefill", "iteration", "iteration", "iteration",
                       "kvp_decode", "kvp_chunk"])
    case = dict(kind=kind, h_q=h_q, h_kv=h_kv, d=d)
    if kind == "iteration":
        mix = rng.choice(["decodes", "decodes", "prompts", "mixed", "mixed"])
        case.update(prefix=0, chunk=0, prompts=0, decodes=0, lengths=rng.randrange(1 << 20))
        if mix == "prompts":
            case.update(prompts=_log_int(rng, 1, 16), median=_log_int(rng, 128, 4096))
        else:
            case.update(decodes=_log_int(rng, 1, 128), median=_log_int(rng, 256, 8192))
        if mix == "mixed":
            case.update(prefix=_log_int(rng, 256, 524288), chunk=_log_int(rng, 16, 2048))
    elif kind == "prefill":
        case.update(prefix=_log_int(rng, 512, 1 << 20), chunk=_log_int(rng, 16, 8192))
    elif kind == "kvp_decode":
        case.update(prefix=_log_int(rng, 8192, 1 << 20) - 1, chunk=1, shards=rng.randrange(2, 9))
    else:
        case.update(prefix=_log_int(rng, 4096, 1 << 20), chunk=_log_int(rng, 16, 4096),
                    shards=rng.randrange(2, 9))
    # no dearer than the largest listed case
    while case["prefix"] > 1024 and (_pairs(case) * 4.0 * d * h_q > MAX_FLOPS
                                     or _keys(case) * 4.0 * d * h_kv > MAX_KV_BYTES):
        case["prefix"] = case["prefix"] * 3 // 4
    return case


def _lengths(case):
    """(prefix_len, chunk_len) of every sequence of the batch, the long request first."""
    prefix, chunk = [], []
    if case["chunk"]:
        prefix.append(case["prefix"])
        chunk.append(case["chunk"])
    if case.get("prompts"):
        lens = wl.lognormal_lengths(case["prompts"], case["lengths"], case["median"], 1.0, 16, 8192)
        prefix += [0] * len(lens)
        chunk += [int(n) for n in lens]
    if case.get("decodes"):
        if case["decodes"] == 1:
            lens = [case["median"]]
        else:
            lens = wl.lognormal_lengths(case["decodes"], case["lengths"], case["median"])
        prefix += [int(n) - 1 for n in lens]
        chunk += [1] * len(lens)
    return np.array(prefix, np.int32), np.array(chunk, np.int32)


def _pairs(case):
    p, c = (x.astype(np.float64) for x in _lengths(case))
    return float((c * p + c * (c + 1) / 2).sum())


def _keys(case):
    p, c = _lengths(case)
    return float(p.astype(np.float64).sum() + c.sum())


def _shards(n, shards):
    """Page-aligned cut points of n keys in `shards` contiguous ranges of nearly equal length."""
    per = -(-(-(-n // shards)) // PAGE) * PAGE
    return [min(n, i * per) for i in range(shards + 1)]


def prepare(case, seed):
    prefix, chunk = _lengths(case)
    b = wl.make_prefill_batch(case["kind"], case["h_q"], case["h_kv"], case["d"], prefix, chunk,
                              seed, "cuda")
    s = dict(kind=case["kind"], b=b)
    rows = (b.tokens, b.h_q, b.d)
    if case["kind"] == "iteration":
        s["k_new"] = wl.randn_bf16((b.tokens, b.h_kv, b.d), seed * 1000 + 4, "cuda")
        s["v_new"] = wl.randn_bf16((b.tokens, b.h_kv, b.d), seed * 1000 + 5, "cuda")
        s["pt"] = torch.from_numpy(b.page_table).cuda()
        return s
    s["out"] = torch.empty(rows, dtype=torch.float32, device="cuda")
    s["lse"] = torch.empty(rows[:2], dtype=torch.float32, device="cuda")
    if case["kind"] == "prefill":
        need = medha.chunked_prefill_workspace_bytes(prefix, chunk, b.h_q, b.h_kv, b.d)
        s["pt"] = torch.from_numpy(b.page_table).cuda()
    else:
        # every shard is a slice of the request's page table with its own key count; the rows
        # of the chunk see what lies before them in the shard
        n, shards = int(prefix[0] + chunk[0]), case["shards"]
        cuts = _shards(n, shards)
        slices = [b.page_table[lo // PAGE:-(-hi // PAGE)] for lo, hi in zip(cuts[:-1], cuts[1:])]
        s["offs"] = np.concatenate([[0], np.cumsum([len(x) for x in slices])]).astype(np.int64)
        s["pt"] = torch.from_numpy(np.concatenate(slices)).cuda()
        s["kv_len"] = np.diff(cuts).astype(np.int32)
        s["q_row"] = np.zeros(shards, np.int32)
        s["part"] = torch.empty((shards * b.tokens,) + rows[1:], dtype=torch.float32, device="cuda")
        s["part_lse"] = torch.empty((shards * b.tokens, b.h_q), dtype=torch.float32, device="cuda")
        if case["kind"] == "kvp_decode":
            need = medha.decode_partial_workspace_bytes(s["kv_len"], b.h_q, b.h_kv, b.d)
        else:
            s["chunk"] = np.full(shards, b.tokens, np.int32)
            s["visible0"] = np.array([int(prefix[0]) + 1 - lo for lo in cuts[:-1]], np.int32)
            need = medha.chunk_partial_workspace_bytes(s["chunk"], s["kv_len"], b.h_q, b.h_kv, b.d)
    s["ws"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    b = s["b"]
    if s["kind"] == "iteration":
        medha.kv_append(s["k_new"], s["v_new"], b.k_pool, b.v_pool, s["pt"], b.page_table_offs,
                        b.prefix_len, b.chunk_len)
        out, lse = medha.chunked_prefill_attn(b.q, b.k_pool, b.v_pool, s["pt"], b.page_table_offs,
                                              b.prefix_len, b.chunk_len, b.scale)
        return {"out": out, "lse": lse, "k_pool": b.k_pool, "v_pool": b.v_pool}
    if s["kind"] == "prefill":
        medha.chunked_prefill_attn(b.q, b.k_pool, b.v_pool, s["pt"], b.page_table_offs,
                                   b.prefix_len, b.chunk_len, b.scale, s["out"], s["lse"], s["ws"])
        return {"out": s["out"], "lse": s["lse"]}
    if s["kind"] == "kvp_decode":
        medha.decode_partial_attn(b.q, b.k_pool, b.v_pool, s["pt"], s["offs"], s["q_row"],
                                  s["kv_len"], b.scale, s["part"], s["part_lse"], s["ws"])
    else:
        medha.chunk_partial_attn(b.q, b.k_pool, b.v_pool, s["pt"], s["offs"], s["q_row"],
                                 s["chunk"], s["kv_len"], s["visible0"], b.scale, s["part"],
                                 s["part_lse"], s["ws"])
    shards = len(s["q_row"])
    medha.lse_merge(s["part"].view(shards, b.tokens, b.h_q, b.d),
                    s["part_lse"].view(shards, b.tokens, b.h_q), s["out"], s["lse"])
    return {"out": s["out"], "lse": s["lse"], "part": s["part"], "part_lse": s["part_lse"]}


def work(case):
    _, chunk = _lengths(case)
    tokens = float(chunk.sum())
    row = case["h_q"] * case["d"]
    # q read, out and lse written, every key and value of the batch read once
    n_bytes = tokens * (2 * row + 4 * row + 4 * case["h_q"])
    n_bytes += _keys(case) * 4 * case["d"] * case["h_kv"]
    if case["kind"] == "iteration":   # the new tokens' K and V: read, and written to the cache
        n_bytes += tokens * 2 * 4 * case["d"] * case["h_kv"]
    if case["kind"].startswith("kvp"):  # each shard's partials are results of their own
        n_bytes += case["shards"] * tokens * (4 * row + 4 * case["h_q"])
    return {"bytes": n_bytes, "flops": _pairs(case) * 4.0 * case["d"] * case["h_q"]}


def tolerance(case):
    # Four times what the outputs differ from the same attention in 64 bits: the probabilities'
    # rounding to bf16 puts 1.2e-3 to 1.7e-3 (2-norm) on `out` over the listed cases and 14
    # drawn ones, and up to 3.4e-2 of the root mean square on one element (rows of few keys).
    return {"rel": 6.8e-3, "max": 0.14}
