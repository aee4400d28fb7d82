"""GPU parity at the sizes where a kernel's tiling can go wrong: one row either side of a tile, a row
block and a round of waves, the smallest call, ranges split as finely as they can be."""
import numpy as np
import pytest
import torch

import kvp_workloads as W
from tests.gpu_harness import build_store, make_cache, oracle_workload, run_workload
from tests.test_gpu_parity import compare

pytestmark = pytest.mark.gpu

GENERIC, MFMA, F32, NARROW = 0, 1, 2, 3   # kvp_debug_last_plan(store, 3)
_run_workload, LAST = run_workload, {}


def run_workload(w):
    """The harness's, and keeps which kernel its last call took."""
    import paper_2604_13226_amd as kvp
    got = _run_workload(w)
    LAST["kernel"] = int(kvp.kvp_debug_last_plan(got["store"], 3)[0])
    return got


def _request(dtype, d, g, ctx, n_q, n_kv=2, paged=False, seed=5, n_req=1):
    w = W.random_small(seed, dtype=dtype, d=d, n_q_heads=n_kv * g, n_kv_heads=n_kv, n_layers=1, n_packets=2, k=0, n_q=n_q, n_req=n_req)
    w.packet_lens[:] = [max(ctx // 3, 1), ctx - max(ctx // 3, 1)] if ctx > 1 else [1, 1]
    for rq in w.requests:
        rq.packet_ids = [0, 1] if ctx > 1 else [0] * ctx
    w.paged = paged
    return w


@pytest.mark.parametrize("d,g,ctx,n_q,paged,target", [
    (64, 1, 0, 1, False, None), (64, 2, 1, 1, True, None), (64, 2, 16, 16, False, None), (64, 7, 31, 5, True, None),
    (128, 4, 95, 33, False, None), (128, 1, 127, 1, False, None), (128, 1, 128, 32, True, None), (128, 7, 129, 9, False, None),
    (128, 4, 1000, 8, True, "4000"), (64, 4, 700, 9, False, "4000"), (256, 1, 250, 7, False, None), (256, 2, 300, 17, True, "4000"),
])
def test_fp32_matrix_kernel(gpu_device, monkeypatch, d, g, ctx, n_q, paged, target):
    if target:
        monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", target)  # ranges of 64 rows: waves without a tile, many partial rows
    w = _request("f32", d, g, ctx, n_q, paged=paged)
    compare(w, run_workload(w), oracle_workload(w))
    assert LAST["kernel"] == F32


@pytest.mark.parametrize("d,g,ctx,n_q,paged,target", [
    (64, 1, 0, 1, False, None), (64, 4, 1, 33, True, None), (64, 7, 63, 5, False, None), (64, 4, 64, 32, True, None),
    (64, 4, 255, 65, False, None), (64, 7, 1300, 19, True, "4000"), (64, 2, 2000, 64, False, None), (256, 1, 0, 1, True, None),
    (256, 4, 63, 32, False, None), (256, 2, 65, 70, True, None), (256, 7, 900, 20, False, "4000"), (256, 4, 1500, 9, True, None),
])
def test_bf16_head_dims_64_and_256(gpu_device, monkeypatch, d, g, ctx, n_q, paged, target):
    if target:
        monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", target)
    w = _request("bf16", d, g, ctx, n_q, paged=paged, n_req=2)
    compare(w, run_workload(w), oracle_workload(w))
    assert LAST["kernel"] == MFMA


@pytest.mark.parametrize("dtype,d,g,ctx,n_q,paged,target", [
    ("f32", 64, 2, 40, 20, False, None), ("f32", 128, 4, 100, 33, True, "4000"), ("f32", 256, 1, 30, 70, False, None),
    ("bf16", 64, 4, 70, 40, True, None), ("bf16", 64, 7, 0, 65, False, "4000"), ("bf16", 256, 2, 100, 30, False, None),
    ("bf16", 256, 2, 100, 30, False, "4000"), ("bf16", 256, 7, 300, 20, True, "4000"),
    # bf16, 128 columns, at most 32 packed rows: one tile of query rows, two of them, a later tile of a wave, split
    ("bf16", 128, 4, 40, 8, True, None), ("bf16", 128, 1, 17, 32, False, None), ("bf16", 128, 1, 300, 20, True, "1"),
    ("bf16", 128, 2, 700, 16, False, "4000"),
    # and more than 32: row blocks of 128 (query rows in one tile, in two), of 256 with a half block, split
    ("bf16", 128, 4, 70, 40, True, None), ("bf16", 128, 1, 50, 100, False, None), ("bf16", 128, 4, 100, 90, True, None),
    ("bf16", 128, 7, 900, 20, False, "4000"),
])
def test_an_infinity_in_v_reaches_only_the_rows_that_see_it(gpu_device, monkeypatch, dtype, d, g, ctx, n_q, paged, target):
    import paper_2604_13226_amd as kvp
    if target:
        monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", target)
    w = _request(dtype, d, g, ctx, n_q, paged=paged)
    store = build_store(w, kvp)
    q_off = np.array([0, n_q], np.int32)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, ctx + n_q))

    def call(change):
        cache = make_cache(w, kvp, store)
        kvp.kvp_assemble(store, [(rq.packet_ids, 0) for rq in w.requests], cache)
        q, kn, vn = w.query(0, 0, "cuda:0")
        change(vn)
        out = torch.empty_like(q)
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, ws, out)
        return out.float().cpu()

    at, col = (2 * n_q) // 3, d // 2 + 3
    clean = call(lambda vn: None)
    kernel = F32 if dtype == "f32" else NARROW if d == 128 and n_q * g <= 32 else MFMA
    plan = kvp.kvp_debug_last_plan(store, 1)
    assert int(kvp.kvp_debug_last_plan(store, 3)[0]) == kernel
    assert target != "4000" or int(plan[6 + 5]) > 1 or ctx + n_q <= 65     # the rows were cut
    for value in (float("inf"), float("nan")):
        def change(vn):
            vn[at, 0, col] = value
        got = call(change)
        assert torch.equal(got[:at], clean[:at])                     # rows before it: untouched
        hit = torch.zeros(clean.shape, dtype=torch.bool)
        hit[at:, :g, col] = True                                      # the query heads of KV head 0
        assert torch.equal(got[~hit], clean[~hit])
        assert bool((torch.isinf(got[hit]) if value == float("inf") else torch.isnan(got[hit])).all())


@pytest.mark.parametrize("shape", ["128", "two groups", "256"])
@pytest.mark.parametrize("ctx,n_q,target", [(0, 30, None), (200, 70, None), (700, 33, "4000")])
def test_an_infinity_in_v_new_in_place(gpu_device, monkeypatch, ctx, n_q, target, shape):
    """The same without a cache, over the shapes of the 128-row kernel's workgroups."""
    import paper_2604_13226_amd as kvp
    if target:
        monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", target)
    monkeypatch.setenv("KVP_ATTN_BM", "256" if shape == "256" else "128")
    if shape == "two groups":
        monkeypatch.setenv("KVP_ATTN_SPLIT_IN_WG", "1")
    g, d = 4, 128
    w = _request("bf16", d, g, ctx, n_q)
    store = build_store(w, kvp)
    q_off = np.array([0, n_q], np.int32)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, ctx + n_q))

    def calls(change):  # in place, and over a cache
        q, kn, vn = w.query(0, 0, "cuda:0")
        change(vn)
        reqs = [(rq.packet_ids, 0) for rq in w.requests]
        out, out2, tail = torch.empty_like(q), torch.empty_like(q), torch.empty_like(kn)
        kvp.kvp_prefill_packets(store, reqs, 0, q, kn, vn, q_off, tail, ws, out)
        cache = make_cache(w, kvp, store)
        kvp.kvp_assemble(store, reqs, cache)
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, ws, out2)
        return out.float().cpu(), out2.float().cpu()

    at, col = (2 * n_q) // 3, d // 2 + 3
    clean = calls(lambda vn: None)
    for value in (float("-inf"), float("nan")):
        def change(vn):
            vn[at, 0, col] = value
        hit = torch.zeros(clean[0].shape, dtype=torch.bool)
        hit[at:, :g, col] = True
        for got, want in zip(calls(change), clean):
            assert torch.equal(got[~hit], want[~hit])
            assert bool(((got[hit] == value) if value == value else torch.isnan(got[hit])).all())


@pytest.mark.parametrize("d,g,ctx,n_q,paged", [
    (64, 1, 0, 2, False), (64, 4, 70, 40, True), (64, 2, 63, 65, False), (256, 1, 0, 2, True), (256, 2, 100, 30, False),
])
@pytest.mark.parametrize("value", [3.3895313892515355e38, -3.3895313892515355e38])
def test_the_largest_v_of_a_later_token_stays_out_of_earlier_rows(gpu_device, d, g, ctx, n_q, paged, value):
    """The largest bf16 times any positive weight a masked entry could be given would show: the rows
    before the token, and the columns beside it, keep every bit."""
    import paper_2604_13226_amd as kvp
    w = _request("bf16", d, g, ctx, n_q, paged=paged)
    store = build_store(w, kvp)
    q_off = np.array([0, n_q], np.int32)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, ctx + n_q))
    outs = []
    for large in (False, True):
        cache = make_cache(w, kvp, store)
        kvp.kvp_assemble(store, [(rq.packet_ids, 0) for rq in w.requests], cache)
        q, kn, vn = w.query(0, 0, "cuda:0")
        if large:
            vn[n_q - 1, 0, d // 2 + 3] = value
        out = torch.empty_like(q)
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, ws, out)
        outs.append(out.float().cpu())
    changed = outs[0] != outs[1]
    assert bool(changed[n_q - 1, :g, d // 2 + 3].all())
    changed[n_q - 1, :g, d // 2 + 3] = False
    assert not bool(changed.any())


@pytest.mark.parametrize("d", [64, 256])
def test_a_prerotated_query_enters_the_scores_as_it_is(gpu_device, d):
    """Queries x * ones for 128 values of x against a key y * ones and keys of zeros: the value behind a zero
    key comes out as exp(-S) with S = x y sqrt(d), 14 to 28, so that one more rounding of x to bf16 (2^-8 of it at
    most) would be up to ten per cent.  Bound: the output's own rounding, 2^-8 of a value just above a
    power of two, and 2^-10 for the fp32 score (28 times at most 256 roundings of 2^-24)."""
    import paper_2604_13226_amd as kvp
    n_q, g, y = 32, 4, 1.734375 * 8 / d ** 0.5
    store = kvp.kvp_store_create(1, g, 1, d, "bf16", 5.0e5, 4096, kvp.packet_bytes(1, 1, d, "bf16", 2))
    k = torch.zeros((1, 1, 2, d), dtype=torch.bfloat16, device="cuda:0")
    v = torch.zeros_like(k)
    k[0, 0, 0], v[0, 0, 1] = y, 1.0
    kvp.kvp_store_put(store, 0, k, v)
    cache = kvp.Cache.contiguous(store, 1, 2 + n_q)
    kvp.kvp_assemble(store, [([0], 0)], cache)                          # Delta = 0: nothing is rotated
    x = 1.0 + torch.arange(128, dtype=torch.float64) / 128
    q = x.view(n_q, g, 1).expand(n_q, g, d).to(device="cuda:0", dtype=torch.bfloat16).contiguous()
    zero = torch.zeros((n_q, 1, d), dtype=torch.bfloat16, device="cuda:0")
    out = torch.empty_like(q)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, 2 + n_q))
    kvp.kvp_query_prefill(store, cache, 0, q, zero, zero, np.array([0, n_q], np.int32), ws, out, kvp.KVP_PREROTATED)
    s = x * float(k[0, 0, 0, 0]) * d ** 0.5
    seen = 1.0 + torch.arange(n_q, dtype=torch.float64).repeat_interleave(g) + 1.0   # keys of zeros: one stored, t + 1 of the query
    want = torch.exp(-s) / (1.0 + seen * torch.exp(-s))
    got = out.double().cpu().view(128, d)
    assert float((got / want[:, None] - 1).abs().max()) <= 2.0 ** -8 + 2.0 ** -10


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 256), ("bf16", 64), ("bf16", 256)])
def test_v_near_the_top_of_its_range_does_not_overflow(gpu_device, dtype, d):
    """All of V is 2^121 and one key of the second tile scores 7.9 (log2) above the rest: 103 weights of at most
    one keep every sum below 2^128, and the output is 2^121; relative to the first tile's maximum that
    key's weight alone would bring 2^128.9."""
    import paper_2604_13226_amd as kvp
    n_q, g, rows = 3, 2, 100
    store = kvp.kvp_store_create(1, g, 1, d, dtype, 5.0e5, 4096, kvp.packet_bytes(1, 1, d, dtype, rows))
    k = torch.zeros((1, 1, rows, d), dtype=store.torch_dtype, device="cuda:0")
    v = torch.full_like(k, 2.0 ** 121)
    k[0, 0, 90] = 7.9 * np.log(2.0) / d ** 0.5
    kvp.kvp_store_put(store, 0, k, v)
    cache = kvp.Cache.contiguous(store, 1, rows + n_q)
    kvp.kvp_assemble(store, [([0], 0)], cache)
    q = torch.ones((n_q, g, d), dtype=store.torch_dtype, device="cuda:0")
    kn, vn = torch.zeros_like(q[:, :1]).contiguous(), torch.full_like(q[:, :1], 2.0 ** 121).contiguous()
    out = torch.empty_like(q)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, rows + n_q))
    kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, np.array([0, n_q], np.int32), ws, out, kvp.KVP_PREROTATED)
    # (103 additions, and for bf16 the cut of a probability to 17 bits and the output's rounding)
    assert float((out.double().cpu() / 2.0 ** 121 - 1).abs().max()) <= (2.0 ** -8 if dtype == "bf16" else 2.0 ** -16)


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 64), ("bf16", 256)])
def test_a_workspace_that_holds_only_the_generic_kernels_rows(gpu_device, monkeypatch, dtype, d):
    """The matrix kernels' partial rows come in larger blocks: a call whose workspace holds the generic
    kernel's and not theirs is served all the same, and the next call with room enough as before it."""
    import paper_2604_13226_amd as kvp
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", "4000")               # ranges of 64 rows with either kernel
    w = _request(dtype, d, 2, 900, 3)
    store = build_store(w, kvp)
    q_off = np.array([0, 3], np.int32)
    full = kvp.kvp_prefill_workspace_bytes(store, 1, 3, 903)
    outs = []
    kernels = []
    for size in (full, 30 * 8 * (d + 2) * 4 + (1 << 14), full):    # 15 ranges, 2 heads: 30 slots of 8 rows, and the query
        cache = make_cache(w, kvp, store)
        kvp.kvp_assemble(store, [(rq.packet_ids, 0) for rq in w.requests], cache)
        q, kn, vn = w.query(0, 0, "cuda:0")
        out = torch.full_like(q, float("nan"))
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, kvp.alloc_workspace(size), out)
        outs.append(out.float().cpu())
        kernels.append(int(kvp.kvp_debug_last_plan(store, 3)[0]))
    best = F32 if dtype == "f32" else MFMA
    assert kernels == [best, GENERIC, best]
    assert torch.equal(outs[0], outs[2])
    # one computation in two orders: the tolerance of the parity tests
    assert float((outs[0] - outs[1]).abs().max()) <= (1e-5 if dtype == "f32" else 2e-2)
    with pytest.raises(kvp.KvpError):
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, kvp.alloc_workspace(256), out)


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 64), ("bf16", 256)])
@pytest.mark.parametrize("captured", ["small", "full"])
def test_a_captured_plan_leaves_calls_with_another_workspace_alone(gpu_device, monkeypatch, dtype, d, captured):
    """Whether a call steps back to the generic kernel follows from its own workspace, also while a graph
    holds the plan of the other kernel for the same geometry."""
    import paper_2604_13226_amd as kvp
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", "4000")               # ranges of 64 rows with either kernel
    w = _request(dtype, d, 2, 900, 3)
    store = build_store(w, kvp)
    cache = make_cache(w, kvp, store)
    kvp.kvp_assemble(store, [(rq.packet_ids, 0) for rq in w.requests], cache)
    q_off = np.array([0, 3], np.int32)
    q, kn, vn = w.query(0, 0, "cuda:0")
    ws = {"full": kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, 3, 903)),
          "small": kvp.alloc_workspace(30 * 8 * (d + 2) * 4 + (1 << 14))}   # 15 ranges, 2 heads: the generic kernel's 30 slots, and the query
    out = torch.empty_like(q)

    def call(size):
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, ws[size], out)

    def result(run):
        out.fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        return out.clone()

    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        want = {size: result(lambda: call(size)) for size in ("full", "small")}
        assert not torch.equal(want["full"], want["small"])            # two kernels, two orders of the sums
        call(captured)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(captured)
        for _ in range(3):
            assert torch.equal(result(graph.replay), want[captured])
            for size in ("full", "small", "full"):
                assert torch.equal(result(lambda: call(size)), want[size])
    del graph
    kvp.kvp_release_captured_plans(store)


@pytest.mark.parametrize("g,ctx,n_q,paged,target,n_req", [
    (1, 0, 1, False, None, 1), (4, 1, 1, True, None, 2), (4, 31, 1, False, None, 1), (7, 32, 4, True, None, 3), (4, 255, 8, False, None, 1),
    (8, 257, 4, True, "4000", 1), (1, 1000, 32, False, "4000", 2), (2, 16, 16, True, None, 1), (4, 5000, 1, False, None, 1),
    (4, 2047, 2, True, "1", 2), (7, 3000, 3, False, "40", 1), (32, 700, 1, False, None, 1),
])
def test_bf16_requests_of_few_packed_rows(gpu_device, monkeypatch, g, ctx, n_q, paged, target, n_req):
    """At most 32 packed rows: eight waves with tiles of their own; "1": one range, so every wave takes
    several tiles and the query rows come in a later one."""
    if target:
        monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", target)
    w = _request("bf16", 128, g, ctx, n_q, paged=paged, n_req=n_req)
    compare(w, run_workload(w), oracle_workload(w))
    assert LAST["kernel"] == NARROW


@pytest.mark.parametrize("dtype,d,n_q,kernel", [
    ("bf16", 128, 40, MFMA), ("bf16", 128, 3, NARROW), ("bf16", 64, 5, MFMA), ("bf16", 256, 5, MFMA),
    ("f32", 64, 5, F32), ("f32", 128, 5, F32), ("f32", 256, 5, F32), ("f32", 96, 3, GENERIC), ("bf16", 96, 3, GENERIC),
])
@pytest.mark.parametrize("splits", [9, 16, 17, 24, 25, 32, 33, 40, 41, 64])
def test_a_merge_of_many_splits(gpu_device, monkeypatch, dtype, d, n_q, kernel, splits):
    """The merge takes a row's pieces several at a time, as many up front as the launch may need: split
    counts either side of each of its steps, every format of the partial rows."""
    import paper_2604_13226_amd as kvp
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", str(splits))
    at_least = 256 if dtype == "bf16" and d == 128 else 64
    w = _request(dtype, d, 1, splits * at_least - n_q - 7, n_q, n_kv=1)
    got = run_workload(w)
    p = kvp.kvp_debug_last_plan(got["store"], 1)
    assert LAST["kernel"] == kernel and int(p[2]) == 1 and int(p[6 + 5]) == splits
    compare(w, got, oracle_workload(w))


@pytest.mark.parametrize("splits", [2, 4, 5, 8])
@pytest.mark.parametrize("d,g,n_q,bm", [(128, 1, 33, None), (128, 7, 37, None), (128, 4, 65, "256"), (128, 5, 7, None),
                                        (64, 1, 33, None), (64, 7, 37, None), (256, 5, 7, None), (256, 4, 65, None)])
def test_a_merge_of_few_splits_of_bf16_rows(gpu_device, monkeypatch, d, g, n_q, bm, splits):
    """The matrix kernel's partial rows are merged four at a time, each wave every fourth split: few splits, rows that end
    inside a quad, several row blocks; tolerance of every bf16 case (Q, P and the output rounded to bf16)."""
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", str(splits * 2 * -(-g * n_q // int(bm or 128))))
    if bm:
        monkeypatch.setenv("KVP_ATTN_BM", bm)
    w = _request("bf16", d, g, splits * 256 - n_q - 7, n_q)
    got = run_workload(w)
    import paper_2604_13226_amd as kvp
    assert LAST["kernel"] == MFMA and int(kvp.kvp_debug_last_plan(got["store"], 1)[6 + 5]) == splits
    compare(w, got, oracle_workload(w))


def _merged(monkeypatch, d, splits, score, v, v_new, n_q=9, g=4, n_kv=1):
    """One request of `splits` ranges of 256 rows, the query rows in the last: all rows of range i score score[i] (log2, a bf16
    key's rounding aside) and hold v[i] (a number, or one for each column), the query rows score zero and hold
    v_new.  Returns the output [n_q][n_kv g][d] and the one of float64, from the keys as they are."""
    import paper_2604_13226_amd as kvp
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", str(splits * n_kv))
    n = 256 * splits - n_q
    store = kvp.kvp_store_create(1, n_kv * g, n_kv, d, "bf16", 1.0e4, n + 64, 1 << 20)
    cache = kvp.Cache.contiguous(store, 1, n + n_q)
    cache.ctx_len[0] = n
    k, val = torch.zeros(splits, 256, d), torch.zeros(splits, 256, d)
    k[:, :, 0] = torch.tensor(score)[:, None] * float(np.log(2)) * d ** 0.5 / 16
    for i in range(splits):
        val[i] = torch.as_tensor(v[i], dtype=torch.float32)
    k, val = (x.view(-1, d)[:n].to(torch.bfloat16).cuda() for x in (k, val))
    cache.k[0, 0, :, :n], cache.v[0, 0, :, :n] = k, val
    q = torch.zeros(n_q, n_kv * g, d, dtype=torch.bfloat16, device="cuda:0")
    q[:, :, 0] = 16
    kn = torch.zeros(n_q, n_kv, d, dtype=torch.bfloat16, device="cuda:0")
    vn, out = torch.full_like(kn, v_new), torch.empty_like(q)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, n + n_q))
    kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, np.array([0, n_q], np.int32), ws, out, kvp.KVP_PREROTATED)
    plan = kvp.kvp_debug_last_plan(store, 1)
    assert int(kvp.kvp_debug_last_plan(store, 3)[0]) == MFMA and int(plan[2]) == n_kv and int(plan[6 + 5]) == splits
    s = torch.cat([k[:, 0].double().cpu() * 16 / d ** 0.5, torch.zeros(n_q, dtype=torch.float64)])
    w = torch.exp(s - s.max())[None] * (torch.arange(n + n_q)[None] <= n + torch.arange(n_q)[:, None])
    want = (w / w.sum(1, keepdim=True)) @ torch.cat([val, vn[:, 0]]).double().cpu()
    return out.double().cpu(), want[:, None].expand(-1, n_kv * g, -1)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("splits,at", [(4, 0), (4, 2), (7, 2), (7, 3), (20, 0), (20, 3), (41, 7), (41, 8)])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_a_split_of_no_weight_does_not_reach_the_output(gpu_device, monkeypatch, d, splits, at, value):
    """The query rows weigh 2^300 times what is stored, whose ranges hold an infinity or NaN in one column: whichever
    of the merge's waves takes it, the output is what the query rows hold."""
    v = [0.0] * splits
    v[at] = torch.zeros(d)
    v[at][d // 2 + 3] = value
    got, _ = _merged(monkeypatch, d, splits, [-300.0] * (splits - 1) + [-200.0], v, 1.0)
    assert bool((got == 1).all())


@pytest.mark.parametrize("splits", [8, 16, 23])
@pytest.mark.parametrize("d", [64, 256])
def test_large_sums_of_splits_of_little_weight_do_not_overflow(gpu_device, monkeypatch, d, splits):
    """Two ranges whose unnormalised sums come near the end of fp32's range (256 weights of 2^-8 times 3e38), 2^-20 of the
    query rows' weight: the merge adds them weighed.  Bound: the output's rounding to bf16, and 2^-10 for the scores in fp32."""
    score, v = [-300.0] * splits, [0.0] * splits
    for at in (1, 5):
        score[at], v[at] = -20.0, 3e38
    got, want = _merged(monkeypatch, d, splits, score, v, 0.0)
    assert float((got / want - 1).abs().max()) <= 2.0 ** -8 + 2.0 ** -10


@pytest.mark.parametrize("splits", [4, 21])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_splits_whose_weight_is_below_the_normal_range_count(gpu_device, monkeypatch, d, splits):
    """A range 2^-135 of the query rows' weight holds 3e38; at 128 columns, where a partial row is scaled by its largest
    number, ranges of one score hold 2^60 and 2^-80.  Bound: the output's rounding to bf16, 2^-10 for the scores in
    fp32 and the scaled rows in fp16, 2^-13 for a weight of 14 bits."""
    score, v, v_new = [-300.0] * splits, [0.0] * splits, 1.0
    score[1], v[1] = -135.0, 3e38
    if d == 128:
        score, v, v_new = [0.0] * splits, [2.0 ** -80] * splits, 2.0 ** -80
        v[1] = 2.0 ** 60
    got, want = _merged(monkeypatch, d, splits, score, v, v_new)
    assert float((got / want - 1).abs().max()) <= 2.0 ** -8 + 2.0 ** -10 + 2.0 ** -13


@pytest.mark.parametrize("d,splits", [(128, 2), (128, 5), (128, 17), (256, 2), (256, 5), (256, 17), (256, 33), (256, 41)])
@pytest.mark.parametrize("g,n_q", [(4, 17), (1, 37)])
def test_a_merge_of_eight_heads(gpu_device, monkeypatch, d, splits, g, n_q):
    """As many groups as XCDs: items and merge of a head on one, partial rows left in its L2 (other tests have one or two heads,
    whose rows are written through it and whose merge runs row by row)."""
    import paper_2604_13226_amd as kvp
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", str(8 * splits))
    at_least = 256 if d == 128 else 64
    w = _request("bf16", d, g, splits * at_least - n_q - 7, n_q, n_kv=8)
    got = run_workload(w)
    p = kvp.kvp_debug_last_plan(got["store"], 1)
    assert LAST["kernel"] == MFMA and int(p[2]) == 8 and int(p[6 + 5]) == splits
    compare(w, got, oracle_workload(w))


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("ctx,n_q", [(384, 10), (385, 48), (1000, 33), (1009, 20), (1023, 60), (1500, 100), (2047, 9)])
def test_query_rows_as_a_range_of_their_own(gpu_device, ctx, n_q, paged):
    w = _request("bf16", 128, 4, ctx, n_q, n_kv=8, paged=paged)
    compare(w, run_workload(w), oracle_workload(w))
    assert LAST["kernel"] == MFMA


@pytest.mark.parametrize("g,n_kv,ctx,n_q,ranges", [(8, 1, 16100, 16, 64), (8, 1, 16368, 16, 53), (6, 2, 12152, 10, 49)])
def test_query_rows_as_the_last_of_64_ranges(gpu_device, g, n_kv, ctx, n_q, ranges):
    """As many ranges as the merge takes, the query rows' own among them; contexts where that one came on top."""
    import paper_2604_13226_amd as kvp
    w = _request("bf16", 128, g, ctx, n_q, n_kv=n_kv)
    got = run_workload(w)
    p = kvp.kvp_debug_last_plan(got["store"], 1)
    assert LAST["kernel"] == MFMA and int(p[6 + 5]) == ranges
    compare(w, got, oracle_workload(w))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("what", ["key", "small", "smallest"])
def test_fp32_numbers_that_bf16_parts_do_not_hold(gpu_device, d, what):
    """A key with an infinity that scores minus infinity weighs nothing; V of 2^-100, whose last parts would fall below bf16's
    range, keeps fp32's precision (bound: 60 sums of 2^-24 in either order); V of 2^-120 at least
    what a cut at 2^-126 leaves."""
    import paper_2604_13226_amd as kvp
    ctx, n_q, g = 50, 9, 2
    w = _request("f32", d, g, ctx, n_q, n_kv=1)
    store = build_store(w, kvp)
    cache = make_cache(w, kvp, store)
    kvp.kvp_assemble(store, [(rq.packet_ids, 0) for rq in w.requests], cache)
    q, kn, vn = w.query(0, 0, "cuda:0")
    q = q.abs().contiguous()
    scale = {"key": 1.0, "small": 2.0 ** -100, "smallest": 2.0 ** -120}[what]
    if what == "key":
        cache.k[0, 0, 0, 7, 5] = float("-inf")
    cache.v[0, 0, :, :ctx] *= scale
    vn *= scale
    out = torch.empty_like(q)
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, n_q, ctx + n_q))
    kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, np.array([0, n_q], np.int32), ws, out, kvp.KVP_PREROTATED)
    k, v = cache.k[0, 0, 0, :ctx + n_q].double(), cache.v[0, 0, 0, :ctx + n_q].double()
    s = torch.einsum("thd,kd->thk", q.double(), k.nan_to_num(neginf=-1e30)) / d ** 0.5
    s.masked_fill_(torch.arange(ctx + n_q, device="cuda")[None, None] > ctx + torch.arange(n_q, device="cuda")[:, None, None], float("-inf"))
    want = torch.softmax(s, -1) @ v
    assert bool(torch.isfinite(out).all())
    err = float((out.double() - want).norm() / want.norm())
    assert err <= (2.0 ** -7 if what == "smallest" else 60 * 2.0 ** -24), err


def _one_token(d, q, k, v):
    """fp32 attention of one token of 32 heads over rows of k and v as they are; its own row is zero.  (result, float64)"""
    import paper_2604_13226_amd as kvp
    n = len(k)
    store = kvp.kvp_store_create(1, 32, 1, d, "f32", 1.0e4, n + 64, 1 << 20)
    cache = kvp.Cache.contiguous(store, 1, n + 1)
    cache.ctx_len[0] = n
    cache.k[0, 0, 0, :n], cache.v[0, 0, 0, :n] = k, v
    q, zero, out = q.float().cuda(), torch.zeros(1, 1, d, device="cuda:0"), torch.empty(1, 32, d, device="cuda:0")
    ws = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, 1, n + 1))
    kvp.kvp_query_prefill(store, cache, 0, q[None].contiguous(), zero, zero, np.array([0, 1], np.int32), ws, out, kvp.KVP_PREROTATED)
    assert int(kvp.kvp_debug_last_plan(store, 3)[0]) == F32
    scores = torch.cat([q.double() @ cache.k[0, 0, 0, :n].double().T / d ** 0.5, torch.zeros(32, 1, device="cuda:0")], 1)
    return out[0].double(), torch.softmax(scores, 1)[:, :n] @ cache.v[0, 0, 0, :n].double()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what", ["scores", "values"])
def test_fp32_products_keep_their_small_parts(gpu_device, d, what):
    """Numbers whose bits below the eighth are all ones, all of one sign: what a product of parts leaves out would
    add up.  Bound: four roundings of 2^-24, of the scaled query, the score or weight, the product and the sum."""
    a, scale = 1 + 2.0 ** -7 - 2.0 ** -19, 1.4426950408889634 / d ** 0.5       # (the kernel's query: times scale)
    if what == "scores":                                                       # column 0 of V marks the rows, column 1 one that scores zero
        q, k, v = torch.full((32, d), 2 * a / scale / 8), torch.full((100, d), a), torch.zeros(100, d)
        k[0] = 0
        v[1:, 0] = 1
        v[0, 1] = 1
        got, want = _one_token(d, q, k, v)
        score = (want[:, 0] / want[:, 1]).log() - float(np.log(99))
        err = ((got[:, 0] / got[:, 1]).log() - float(np.log(99)) - score).abs() / score
    else:                                                                      # every weight a / 2, under the largest score of its tile
        q, k, v = torch.zeros(32, d), torch.zeros(100, d), torch.full((100, d), a)
        q[:, 0] = 8 / scale
        k[::32, 0], v[::32] = (1 - float(np.log2(a))) / 8, 0
        got, want = _one_token(d, q, k, v)
        err = (got / want - 1).abs()
    assert float(err.max()) <= 4 * 2.0 ** -24, float(err.max())


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("what", ["column of V", "key", "query"])
def test_fp32_numbers_out_of_the_parts_range(gpu_device, d, what):
    """Numbers so small that their parts would fall below bf16's range, in one column of V beside ordinary ones, or in keys or
    queries whose partners are as large.  Bound: 16 roundings of 2^-24 (the weights of 300 rows; a cut leaves 2e-6 and more)."""
    gen = torch.Generator().manual_seed(5)
    q, k, v = (torch.randn(n, d, generator=gen, dtype=torch.float64) for n in (32, 300, 300))
    if what == "column of V":
        v[:, 5] *= 2.0 ** -115
    else:
        q *= 2.0 ** (118 if what == "key" else -118)
        k *= 2.0 ** (-118 if what == "key" else 118)
    got, want = _one_token(d, q.float(), k.float(), v.float())
    cols = [5] if what == "column of V" else list(range(d))
    err = float((got - want)[:, cols].norm() / want[:, cols].norm())
    assert err <= 2.0 ** -20, err


@pytest.mark.parametrize("d", [64, 128, 256])
def test_fp32_sums_over_many_rows(gpu_device, monkeypatch, d):
    """One range of 20000 rows, V of one sign: what an addition to a large sum cuts would add up.  Bound: 16 roundings of 2^-24
    (a wave's sums of 2500 to 5000 weighted rows in any order, each rounded to nearest, err by about their square root)."""
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", "1")
    gen = torch.Generator().manual_seed(6)
    q, k = torch.randn(32, d, generator=gen), torch.randn(20000, d, generator=gen)
    v = 1 + (torch.rand(20000, d, generator=gen) - 0.5) * 2.0 ** -7
    got, want = _one_token(d, q, k, v)
    err = float((got / want - 1).abs().square().mean().sqrt())
    assert err <= 2.0 ** -20, err


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 64)])
def test_a_capture_takes_the_kept_plan_of_either_kernel(gpu_device, monkeypatch, dtype, d):
    """A geometry warmed up with a workspace that holds only the generic kernel's rows can be captured with a larger one:
    the graph launches from the plan there is."""
    import paper_2604_13226_amd as kvp
    monkeypatch.setenv("KVP_ATTN_TARGET_ITEMS", "4000")               # ranges of 64 rows with either kernel
    w = _request(dtype, d, 2, 900, 3)
    store = build_store(w, kvp)
    cache = make_cache(w, kvp, store)
    kvp.kvp_assemble(store, [(rq.packet_ids, 0) for rq in w.requests], cache)
    q_off = np.array([0, 3], np.int32)
    q, kn, vn = w.query(0, 0, "cuda:0")
    full = kvp.alloc_workspace(kvp.kvp_prefill_workspace_bytes(store, 1, 3, 903))
    small = kvp.alloc_workspace(30 * 8 * (d + 2) * 4 + (1 << 14))          # 15 ranges, 2 heads: the generic kernel's 30 slots, and the query
    out = torch.empty_like(q)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, small, out)
        torch.cuda.synchronize()
        want = out.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            kvp.kvp_query_prefill(store, cache, 0, q, kn, vn, q_off, full, out)
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
    del graph
    kvp.kvp_release_captured_plans(store)
