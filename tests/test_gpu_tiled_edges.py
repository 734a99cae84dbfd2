"""The prefill FFN (tiled kernels) at the edges of its tiles, against the oracle: row counts
around its token-block classes (bf16: 64, 128, 192; fp32: every 32) and its token tile (256
and 128 rows), more token tiles than one sweep takes, a single K slab pair, widths that
leave half a weight tile, and more groups and items than workgroups start with."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from gpu_support import TOL, host_f64, rel_l2
from test_gpu_parity import run_and_check_layer
from workloads import make_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_21614_amd as m
    return m


# T, H, E, F, k, S, Fs, resident
CASES = [(T, 128, 1, 64, 1, 0, 0, 1) for T in (65, 128, 129, 192, 193, 256, 257)] + [
    (1300, 64, 1, 64, 1, 0, 0, 1),       # six token tiles, one slab pair, half a weight tile in phase 2
    (1100, 192, 2, 128, 2, 1, 192, 2),   # two groups and a shared one of five token tiles, H % 128 = 64
    (150, 320, 256, 64, 8, 0, 0, 256),   # up to 256 groups of a few rows
    (200, 512, 64, 1024, 8, 2, 576, 48),  # more items than workgroups (claims, other XCDs' queues)
    (70, 2048, 4, 192, 2, 0, 0, 0),      # no resident expert: no items
    (66, 256, 16, 320, 4, 3, 64, 5),     # shared groups larger than every routed one
]


F32_ROWS = [(T, 128, 1, 64, 1, 0, 0, 1) for T in (96, 97, 160, 161, 225, 289)]


@pytest.mark.parametrize("dtype,T,H,E,F,k,S,Fs,res",
                         [("bf16", *c) for c in CASES] + [("f32", *c) for c in CASES + F32_ROWS])
def test_tile_edges(moe, dtype, T, H, E, F, k, S, Fs, res):
    print(f"[case] tiled {dtype} T={T} H={H} E={E} F={F} k={k} S={S} Fs={Fs} resident={res}", flush=True)
    lay = make_layer(T, H, E, F, k, dtype=dtype, shared=S, shared_ffn=Fs, n_resident=res, residency="random",
                     bias="zipf", seed=T + H)
    run_and_check_layer(moe, lay)


# T, H, E, F, k, S, Fs, resident; item shapes of phase 1 and of phase 2 (0: 128 x 128, 1: 128 x 32, 2: 64 x 32)
F32_SHAPES = [
    (280, 512, 64, 512, 8, 0, 0, 64, 0, 0),      # about 35 rows a group: two and four token blocks
    (600, 512, 64, 512, 8, 0, 0, 64, 0, 0),      # 75 rows: four and six blocks
    (920, 448, 64, 512, 8, 1, 448, 64, 0, 0),    # 115 rows: six, eight, and a second token tile
    (500, 1024, 64, 1024, 8, 0, 0, 64, 0, 0),    # longer sums
    (160, 2048, 16, 1024, 8, 0, 0, 16, 1, 1),
    (300, 2048, 4, 1024, 2, 0, 0, 4, 1, 1),      # 150 rows: five tiles of 32
    (150, 1088, 4, 960, 2, 0, 0, 2, 2, 2),       # widths that leave half a weight tile of 128, none of 64
    (100, 64, 2, 4096, 1, 0, 0, 2, 1, 2),        # one stage of slabs in phase 1, many in phase 2
]


@pytest.mark.parametrize("T,H,E,F,k,S,Fs,res,ph1,ph2", F32_SHAPES)
def test_f32_item_shapes(moe, T, H, E, F, k, S, Fs, res, ph1, ph2):
    from paper_2608_21614_amd.device import to_host
    print(f"[case] tiled f32 T={T} H={H} E={E} F={F} k={k} S={S} Fs={Fs} resident={res}", flush=True)
    lay = make_layer(T, H, E, F, k, dtype="f32", shared=S, shared_ffn=Fs, n_resident=res, residency="random",
                     bias="none", seed=T + H)
    dev, _, _ = run_and_check_layer(moe, lay, sample=np.arange(0, T, 5))
    # the tables' header, at the start of the workspace where the scores are the caller's
    assert to_host(dev.ws[:32].view(torch.int32)).tolist()[3:5] == [ph1, ph2]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,E,k,S,slots", [(70, 12, 3, 2, 5), (150, 64, 8, 0, 3)])
def test_shared_slots_stay_in_their_room(moe, dtype, T, E, k, S, slots):
    """Resident experts that share slots (more of them than slots): the experts that the tables
    have room for run as any others, the rows of the rest are left alone, and nothing is
    written past the workspace."""
    from paper_2608_21614_amd.device import DeviceLayer, to_device, to_host
    print(f"[case] shared slots {dtype} T={T} E={E} k={k} S={S} slots={slots}", flush=True)
    H, F, Fs = 192, 128, 64
    lay = make_layer(T, H, E, F, k, dtype=dtype, shared=S, shared_ffn=Fs if S else 0, n_resident=slots, residency="random",
                     bias="none", seed=T + E)
    holds = lay.slot_experts()                       # slot -> the expert whose weights are in it
    dev = DeviceLayer(lay)
    dev.set_residency(np.arange(E) % slots)
    o = dev.alloc_outputs()
    n = moe.moe_workspace_bytes(dev.dims)
    ws = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    moe.moe_layer_forward(dev.args(o), ws[:n])       # the fused call returns, too
    y = torch.full((T * k + S * T, H), 777.0, dtype=torch.float32, device="cuda")
    moe.moe_grouped_ffn(dev.dims, dev.x, o["perm"], o["counts"], o["seg_start"], dev.expert_slot, dev.w13, dev.w2,
                        dev.ws13, dev.ws2, y, ws[:n])
    torch.cuda.synchronize()
    assert bool((ws[n:] == 0xA5).all())
    counts, seg, perm, got = to_host(o["counts"]), to_host(o["seg_start"]), to_host(o["perm"]), host_f64(y)
    active = np.flatnonzero(counts)
    assert len(active) > slots
    for i, e in enumerate(active):
        rows = slice(seg[e], seg[e] + counts[e])
        if i < slots:
            w = int(holds[e % slots])
            ref = oracle.expert_ffn(lay.x, (perm[rows] // k).astype(np.int32), lay.w13(w), lay.w2(w))
            assert rel_l2(got[rows], ref) <= TOL[dtype], e
        else:
            assert (got[rows] == 777.0).all(), e
    for s in range(S):
        ref = oracle.expert_ffn(lay.x, np.arange(T, dtype=np.int32), lay.ws13(s), lay.ws2(s))
        assert rel_l2(got[T * k + s * T:T * k + (s + 1) * T], ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype,T", [("bf16", 40), ("bf16", 70), ("f32", 40), ("f32", 70), ("f32", 300)])
def test_rows_without_a_pair_are_zero(moe, dtype, T):
    """moe_grouped_ffn on its own, with packed rows that name no pair (-1, or past the batch) among
    the resident ones: such a row has no token and its output is zero; the others are what they are
    without it."""
    from paper_2608_21614_amd.device import DeviceLayer, to_device, to_host
    print(f"[case] rows without a pair {dtype} T={T}", flush=True)
    lay = make_layer(T, 128, 4, 192, 2, dtype=dtype, shared=1, shared_ffn=64, n_resident=3, residency="random", seed=T)
    dev = DeviceLayer(lay)
    o = dev.alloc_outputs()
    dev.forward(o)
    P, n_res = 2 * T, int(to_host(o["n_res"])[0])
    perm = to_host(o["perm"]).copy()
    gone = np.arange(0, n_res, 5)
    perm[gone] = np.resize([-1, P, -7, 2**30], len(gone))
    y = [torch.full((P + T, 128), 777.0, dtype=torch.float32, device="cuda") for _ in range(2)]
    for out, p in zip(y, (o["perm"], to_device(perm))):
        moe.moe_grouped_ffn(dev.dims, dev.x, p, o["counts"], o["seg_start"], dev.expert_slot, dev.w13, dev.w2, dev.ws13,
                            dev.ws2, out, dev.ws)
    torch.cuda.synchronize()
    want, got = to_host(y[0]).copy(), to_host(y[1])
    want[gone] = 0.0
    np.testing.assert_array_equal(got, want)
