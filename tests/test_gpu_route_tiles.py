"""Prefill routing at the edges of its dispatch, against the oracle: expert counts around one,
two and four 16-expert tiles (fused top-k) and above 64 (a launch of its own), token counts
around the workgroup's 8, 16 and 32 rows, long and short rows, both dtypes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from gpu_support import DELTA, LOGIT_TOL, expected_routing, rel_l2
from workloads import make_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_21614_amd as m
    return m


CASES = [
    ("bf16", 65, 64, 1, 1), ("bf16", 71, 96 * 2, 16, 8), ("bf16", 73, 128, 17, 5), ("bf16", 100, 576, 32, 8),
    ("bf16", 90, 4096, 33, 6), ("bf16", 100, 4096, 64, 6), ("bf16", 67, 2112, 65, 8), ("bf16", 500, 64, 256, 8),
    ("bf16", 4097, 64, 40, 6), ("bf16", 8193, 64, 20, 4), ("bf16", 8210, 64, 60, 8), ("bf16", 8200, 64, 70, 3),
    ("bf16", 8209, 64, 9, 2), ("f32", 65, 64, 16, 2), ("f32", 81, 2048, 48, 6), ("f32", 300, 192, 129, 8),
    ("f32", 4100, 64, 64, 6), ("f32", 8200, 64, 33, 6),
    # either side of a workgroup per CU (2048, 4096 tokens) and of the loads' limits; the larger tiles
    ("bf16", 2048, 64, 64, 6), ("bf16", 2049, 64, 64, 6), ("bf16", 2100, 64, 20, 4), ("bf16", 2055, 64, 128, 8),
    ("bf16", 1030, 64, 256, 8), ("bf16", 70, 4096, 17, 3), ("bf16", 70, 4160, 17, 3), ("f32", 2049, 64, 64, 8),
    ("f32", 2100, 64, 20, 4), ("f32", 2060, 64, 3, 2), ("f32", 90, 1024, 28, 4), ("f32", 90, 1088, 28, 4),
    ("f32", 100, 64, 40, 6), ("f32", 8200, 64, 20, 4), ("f32", 8200, 64, 9, 2), ("f32", 8200, 64, 70, 3),
    ("f32", 2049, 64, 128, 8), ("f32", 1030, 64, 256, 8), ("f32", 500, 64, 256, 8),
]


@pytest.mark.parametrize("dtype,T,H,E,k", CASES)
def test_route_tiles(moe, dtype, T, H, E, k):
    from paper_2608_21614_amd.device import to_device, to_host
    print(f"[case] route {dtype} T={T} H={H} E={E} k={k}", flush=True)
    lay = make_layer(T, H, E, 64, k, dtype=dtype, bias="zipf" if T % 2 else "none", n_resident=1, residency="random",
                     seed=T + E)
    dims = moe.make_dims(T, H, E, 64, k, slots=0, dtype=1 if dtype == "bf16" else 0)
    lg = torch.empty((T, E), dtype=torch.float32, device="cuda")
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    w = torch.empty((T, k), dtype=torch.float32, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    bias = None if lay.bias is None else to_device(lay.bias)
    moe.moe_route_topk(dims, to_device(lay.x), to_device(lay.w_router), bias, lg, idx, w, ws)
    torch.cuda.synchronize()
    ref = oracle.router_logits(lay.x, lay.w_router, lay.bias)
    got = to_host(lg).astype(np.float64)
    assert np.abs(got - ref).max() < DELTA / 2 and rel_l2(got, ref) <= LOGIT_TOL
    sel = to_host(idx)
    np.testing.assert_array_equal(sel, expected_routing(ref, sel, k)[0])
    # on the scores the GPU computed, the selection and the gates are the oracle's
    own_idx, own_w = oracle.topk(got, k)
    np.testing.assert_array_equal(sel, own_idx)
    np.testing.assert_allclose(to_host(w), own_w, rtol=2e-6, atol=1e-7)


@pytest.mark.parametrize("dtype,T,E,k,bias", [
    ("bf16", 100, 16, 3, "none"), ("bf16", 100, 40, 8, "some"), ("f32", 2060, 64, 6, "some"), ("f32", 90, 9, 4, "all"),
    ("bf16", 8200, 24, 8, "some"), ("bf16", 70, 100, 5, "some"), ("bf16", 20, 24, 4, "some"),
])
def test_route_ties_of_computed_scores(moe, dtype, T, E, k, bias):
    """Experts with the same router row, so that scores tie exactly, and experts (some, or all) whose
    bias is -inf: the lowest ids among equals, and equal gates where all scores are -inf."""
    from paper_2608_21614_amd.device import to_device, to_host
    print(f"[case] route ties {dtype} T={T} E={E} k={k} bias {bias}", flush=True)
    lay = make_layer(T, 64, E, 64, k, dtype=dtype, bias="none", n_resident=1, residency="random", seed=E)
    wr = lay.w_router[np.arange(E) // 3 * 3].copy()      # triples of equal rows
    b = None
    if bias != "none":
        b = np.zeros(E, np.float32)
        b[(np.arange(E) % 4 != 1) if bias == "some" else slice(None)] = -np.inf
    dims = moe.make_dims(T, 64, E, 64, k, slots=0, dtype=1 if dtype == "bf16" else 0)
    lg = torch.empty((T, E), dtype=torch.float32, device="cuda")
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    w = torch.empty((T, k), dtype=torch.float32, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    moe.moe_route_topk(dims, to_device(lay.x), to_device(wr), None if b is None else to_device(b), lg, idx, w, ws)
    torch.cuda.synchronize()
    got = to_host(lg).astype(np.float64)
    if bias == "none":
        assert (got[:, 0] == got[:, 1]).all() and (got[:, 0] == got[:, 2]).all()
    own_idx, own_w = oracle.topk(got, k)
    np.testing.assert_array_equal(to_host(idx), own_idx)
    np.testing.assert_allclose(to_host(w), own_w, rtol=2e-6, atol=1e-7)
