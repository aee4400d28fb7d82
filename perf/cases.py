"""The work whose speed this repository is judged by: requests over retrieved packets, through the
library's public entry points.

A case is one kind of call sequence a serving program makes, with its sizes:

  mode "step"      kvp_assemble over all layers, then kvp_query_prefill layer by layer
  mode "decode"    kvp_query_prefill with one query row per request, token after token over all
                   layers, on a cache that is already assembled
  mode "in_place"  kvp_prefill_packets layer by layer: no cache, the packets are read in the store

  dtype, layers, q_heads, kv_heads, head_dim     the model's shape
  requests                                       requests in the batch
  packets_min .. packets_max                     packets a request retrieves
  pool                                           packets in the store that the requests draw from, the
                                                 popular ones more often (0: every packet is read once)
  len_min .. len_max                             rows of a packet, spread over the logarithm
  q_min .. q_max                                 query rows of a request
  tokens                                         mode "decode": tokens generated in one pass
  paged                                          cache layout: blocks of 16 rows in random order
  pruned                                         every (packet, layer) lost 10 to 50 % of its rows offline

Lengths, row counts and which packets a request names follow from the case alone, so the work of a
case is one number; the values, the order of retrieval and the block table follow from the seed.
K and V are normal with deviation 0.5, queries with 1, as in this repository's workloads.
"""
import math
import random

import numpy as np
import torch

import paper_2604_13226_amd as kvp

BLOCK = 16          # rows of a cache block
DEVICE = "cuda:0"
ROPE_BASE = 5.0e5


def _case(name, **kw):
    c = dict(name=name, mode="step", dtype="bf16", layers=1, q_heads=32, kv_heads=8, head_dim=128, requests=1,
             packets_min=1, packets_max=1, pool=0, len_min=512, len_max=512, q_min=32, q_max=32, tokens=0,
             paged=False, pruned=False)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest configuration: one layer, two short packets, in full precision.  Launches and
        # the host path count here.
        _case("tiny_fp32", dtype="f32", q_heads=4, kv_heads=2, head_dim=64, packets_min=2, packets_max=2,
              len_min=72, len_max=72, q_min=16, q_max=16),
        # A store kept in full precision at a model's real width: a few passages and a question.
        _case("fp32_k5", dtype="f32", layers=2, packets_min=5, packets_max=5, len_min=272, len_max=1040),
        # A small model's head dimension, a few users at once, on a paged cache.
        _case("d64_paged_b4", layers=4, head_dim=64, requests=4, packets_min=3, packets_max=8, len_min=80, len_max=1040,
              q_min=16, q_max=64, paged=True),
        # Five passages and a question over a model's whole depth (2.9K rows of context).
        _case("llama_k5", layers=32, packets_min=5, packets_max=5, len_min=272, len_max=1040),
        # Twenty short passages; seven query heads share a KV head.
        _case("qwen_k20", layers=28, q_heads=28, kv_heads=4, packets_min=20, packets_max=20, len_min=144, len_max=528,
              q_min=64, q_max=64),
        # The benchmark's headline point: 16 packets of 512 rows, 8K context.
        _case("llama_8k", layers=32, packets_min=16, packets_max=16),
        # Tokens generated over that context, one request: the latency of a small launch.
        _case("llama_8k_decode", mode="decode", layers=32, packets_min=16, packets_max=16, q_min=1, q_max=1, tokens=4),
        # The same question asked of the store in place, with nothing assembled.
        _case("llama_8k_in_place", mode="in_place", layers=32, packets_min=16, packets_max=16),
        # The same packets after offline pruning: every layer keeps rows of its own.
        _case("llama_8k_pruned", layers=32, packets_min=16, packets_max=16, pruned=True),
        # Long contexts in a batch, 128 query rows each: the matrix cores' case.
        _case("long_b8", requests=8, packets_min=32, packets_max=32, len_min=528, len_max=528, q_min=128, q_max=128),
        # Tokens generated over those contexts: the memory's case.
        _case("long_b8_decode", mode="decode", requests=8, packets_min=32, packets_max=32, len_min=528, len_max=528,
              q_min=1, q_max=1, tokens=4),
        # A serving batch: 64 ragged requests on a paged cache, popular packets in many of them.
        _case("serving_mix", requests=64, packets_min=3, packets_max=16, pool=1024, len_min=32, len_max=2064, q_min=16,
              q_max=256, paged=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "batch", "other_shape", "decode", "in_place", "pruned"])
    q_heads, kv_heads = rng.choice([(32, 8), (28, 4)])
    c = _case("", q_heads=q_heads, kv_heads=kv_heads)
    c["len_min"] = _log_int(rng, 16, 528)
    c["len_max"] = _log_int(rng, c["len_min"], 1040)
    c["packets_min"] = _log_int(rng, 1, 32)
    c["packets_max"] = c["packets_min"]
    c["layers"] = _log_int(rng, 1, 32)
    c["q_min"] = _log_int(rng, 1, 256)
    c["q_max"] = c["q_min"]
    if kind == "batch":
        c.update(requests=_log_int(rng, 2, 64), layers=rng.randint(1, 4), paged=rng.random() < 0.7)
        c["packets_max"] = min(32, 2 * c["packets_min"])
        c["q_max"] = min(256, 4 * c["q_min"])
        c["pool"] = rng.choice([0, 512])
    elif kind == "other_shape":  # full precision, and head dimensions other than 128
        c["dtype"] = rng.choice(["f32", "bf16"])
        c["head_dim"] = rng.choice([64, 128] if c["dtype"] == "f32" else [64, 256])
        c.update(requests=_log_int(rng, 1, 4), layers=rng.randint(1, 4), paged=rng.random() < 0.5)
        c["packets_min"] = c["packets_max"] = _log_int(rng, 1, 8)
        c["q_min"] = _log_int(rng, 1, 32)
        c["q_max"] = 2 * c["q_min"]
    elif kind == "decode":
        c.update(mode="decode", requests=_log_int(rng, 1, 16), q_min=1, q_max=1, tokens=rng.randint(1, 8),
                 paged=rng.random() < 0.5)
    elif kind == "in_place":
        c.update(mode="in_place", requests=_log_int(rng, 1, 8), pruned=rng.random() < 0.25)
    elif kind == "pruned":
        c.update(pruned=True)
    while not _affordable(c):
        for what in ("layers", "requests", "packets"):
            if what == "packets":
                c["packets_min"] = max(1, c["packets_min"] // 2)
                c["packets_max"] = max(1, c["packets_max"] // 2)
            elif c[what] > 1:
                c[what] //= 2
                break
    del c["name"]
    return c


def _affordable(c):
    """No more than the largest listed cases: bytes as 8K context over 32 layers, operations as the
    serving batch (in full precision and other head dimensions as the listed cases of that kind), and
    as many launches as four tokens over 32 layers."""
    w = work(c)
    plain = c["dtype"] == "bf16" and c["head_dim"] == 128
    return (w["bytes"] <= 3.2e9 and w["flops"] <= (5.0e11 if plain else 6.0e9) and max(c["tokens"], 1) * c["layers"] <= 128)


# ---- what follows from the case alone ---------------------------------------------------------
def _geometry(c):
    """(lens, wants, n_q, kept): rows of every stored packet, the packets each request names, its
    query rows, and (pruned) the rows every layer kept of every packet."""
    key = ",".join("%s=%s" % (k, c[k]) for k in sorted(c) if k != "name")
    rng = random.Random(key)
    wants, n_pack = [], c["pool"]
    for _ in range(c["requests"]):
        k = rng.randint(c["packets_min"], c["packets_max"])
        if c["pool"]:  # popularity falls with the rank
            chosen = set()
            while len(chosen) < k:
                chosen.add(int(c["pool"] ** rng.random()) - 1)
            wants.append(sorted(chosen))
        else:
            wants.append(list(range(n_pack, n_pack + k)))
            n_pack += k
    lens = [_log_int(rng, c["len_min"], c["len_max"]) for _ in range(n_pack)]
    n_q = [rng.randint(c["q_min"], c["q_max"]) for _ in range(c["requests"])]
    kept = None
    if c["pruned"]:
        kept = [[n - int(round(n * rng.uniform(0.1, 0.5))) for _ in range(c["layers"])] for n in lens]
    return lens, wants, n_q, kept


def work(case):
    """Bytes and operations of the entry points' own inputs and outputs: kvp_assemble reads every
    named packet once and writes the cache once; a prefill call reads the visible rows once, reads
    q, k_new, v_new and writes the new rows and the output."""
    c = case
    lens, wants, n_q, kept = _geometry(c)
    eb = 2 if c["dtype"] == "bf16" else 4
    row = 2 * c["kv_heads"] * c["head_dim"] * eb           # K and V of one position in one layer
    q_row = c["q_heads"] * c["head_dim"] * eb
    n_bytes = flops = 0
    used = sorted({p for want in wants for p in want})
    for layer in range(c["layers"]):
        rows_of = [k[layer] for k in kept] if kept else lens
        unique = sum(rows_of[p] for p in used)
        ctx = [sum(rows_of[p] for p in want) for want in wants]
        if c["mode"] == "step":
            n_bytes += (unique + sum(ctx)) * row
        for t in range(c["tokens"] if c["mode"] == "decode" else 1):
            for r in range(c["requests"]):
                seen = unique / len(wants) if c["mode"] == "in_place" else ctx[r] + t
                n_bytes += seen * row + n_q[r] * (2 * row + 2 * q_row)
                pairs = n_q[r] * (ctx[r] + t) + n_q[r] * (n_q[r] + 1) / 2
                flops += 4 * pairs * c["q_heads"] * c["head_dim"]
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # About four times what a float64 computation from the same inputs differs by, over the listed
    # cases and some drawn ones.  bf16 (rel 2.5e-3): the query and the probabilities are rounded to
    # bf16 before the matrix products and the output after them.  f32 (rel 7e-7): sums of up to a few
    # thousand terms.
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 3e-6}


# ---- the pass -----------------------------------------------------------------------------------
class State:
    pass


def prepare(case, seed):
    c = case
    lens, wants, n_q, kept = _geometry(c)
    order = random.Random(seed)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def normal(shape, scale):
        return torch.randn(shape, generator=gen, dtype=dtype, device=DEVICE).mul_(scale)

    s = State()
    s.mode, s.layers, s.tokens = c["mode"], c["layers"], c["tokens"]
    used = sorted({p for want in wants for p in want})
    wants = [order.sample(want, len(want)) for want in wants]
    ctx = [sum(lens[p] for p in want) for want in wants]
    rows = [ctx[r] + n_q[r] + c["tokens"] for r in range(c["requests"])]
    arena = sum(kvp.packet_bytes(c["layers"], c["kv_heads"], c["head_dim"], c["dtype"], lens[p]) for p in used)
    s.store = kvp.kvp_store_create(c["layers"], c["q_heads"], c["kv_heads"], c["head_dim"], c["dtype"], ROPE_BASE,
                                   max(rows) + 64, arena)
    for p in used:
        shape = (c["layers"], c["kv_heads"], lens[p], c["head_dim"])
        k, v = normal(shape, 0.5), normal(shape, 0.5)
        if kept is None:
            kvp.kvp_store_put(s.store, p, k, v)
        else:  # (random values: the first rows are as good a subset as any)
            kvp.kvp_store_put_compressed(s.store, p, lens[p], [k[l, :, :kept[p][l]] for l in range(c["layers"])],
                                         [v[l, :, :kept[p][l]] for l in range(c["layers"])])
    s.requests = [(np.array(want, np.int64), 0) for want in wants]
    s.q_off = np.zeros(c["requests"] + 1, np.int32)
    s.q_off[1:] = np.cumsum(n_q)
    tot_q = int(s.q_off[-1])
    calls = max(c["tokens"], 1) * c["layers"]
    s.q = normal((calls, tot_q, c["q_heads"], c["head_dim"]), 1.0)
    s.k_new = normal((calls, tot_q, c["kv_heads"], c["head_dim"]), 0.5)
    s.v_new = normal((calls, tot_q, c["kv_heads"], c["head_dim"]), 0.5)
    s.out = torch.zeros_like(s.q)
    s.workspace = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(s.store, c["requests"], tot_q, max(rows)))
    if c["mode"] == "in_place":
        s.k_tail = torch.zeros_like(s.k_new)
        return s
    if c["paged"]:
        blocks = [-(-n // BLOCK) for n in rows]
        ids = order.sample(range(sum(blocks)), sum(blocks))
        table = np.zeros((c["requests"], max(blocks)), np.int32)
        for r, n in enumerate(blocks):
            table[r, :n] = [ids.pop() for _ in range(n)]
        s.cache = kvp.Cache.paged(s.store, c["requests"], sum(blocks), table, BLOCK)
    else:
        s.cache = kvp.Cache.contiguous(s.store, c["requests"], max(rows))
    if c["pruned"]:
        s.cache.with_ctx_rows(c["layers"])
    if c["mode"] == "decode":
        kvp.kvp_assemble(s.store, s.requests, s.cache)
        s.prompt_len = s.cache.ctx_len.copy()
    return s


def run(s):
    if s.mode == "in_place":
        for l in range(s.layers):
            kvp.kvp_prefill_packets(s.store, s.requests, l, s.q[l], s.k_new[l], s.v_new[l], s.q_off, s.k_tail[l],
                                    s.workspace, s.out[l])
        return {"out": s.out, "k_tail": s.k_tail}
    if s.mode == "step":
        kvp.kvp_assemble(s.store, s.requests, s.cache)
        for l in range(s.layers):
            kvp.kvp_query_prefill(s.store, s.cache, l, s.q[l], s.k_new[l], s.v_new[l], s.q_off, s.workspace, s.out[l])
    else:
        s.cache.ctx_len[:] = s.prompt_len
        for t in range(s.tokens):
            for l in range(s.layers):
                i = t * s.layers + l
                kvp.kvp_query_prefill(s.store, s.cache, l, s.q[i], s.k_new[i], s.v_new[i], s.q_off, s.workspace, s.out[i])
            s.cache.ctx_len += 1
    return {"out": s.out, "k": s.cache.k, "v": s.cache.v}
