"""GPU parity at the sizes where a kernel's tiling can go wrong: one row either side of a tile, a row
block and a round of waves, the smallest call, ranges split as finely as they can be."""
import pytest

import kvp_workloads as W
from tests.gpu_harness import oracle_workload, run_workload
from tests.test_gpu_parity import compare

pytestmark = pytest.mark.gpu


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
