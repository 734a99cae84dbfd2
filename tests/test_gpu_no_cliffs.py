"""Calls next to each other in size or type that should take about the same time, timed on the
GPU in turn: neither may fall off a cliff.  The bounds leave room for the noise of a shared
machine; what they guard against was a factor of two or more."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_21614_amd as m
    return m


def times_us(*calls, passes=8, rounds=7):
    """Median time of a pass of each call, the calls taken in turn."""
    got = [[] for _ in calls]
    for r in range(rounds + 1):
        for call, ts in zip(calls, got):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(passes):
                call()
            b.record()
            b.synchronize()
            if r:
                ts.append(1e3 * a.elapsed_time(b) / passes)
    return [sorted(ts)[len(ts) // 2] for ts in got]


def test_pack_moves_fp32_as_fast_as_bf16(moe):
    """The same 184 MB as a bf16 and as an fp32 matrix: it was 2.2 times as slow in fp32 with stores
    of half a line; HBM bounds both, and the fp32 copy takes 0.95 to 1 of the bf16 one."""
    src = [torch.randn((5632, 16384 if dt == torch.bfloat16 else 8192), device="cuda").to(dt)
           for dt in (torch.bfloat16, torch.float32)]
    dst = [torch.empty_like(s) for s in src]
    bf16, f32 = times_us(*(lambda s=s, d=d: moe.moe_pack_weights(s, d) for s, d in zip(src, dst)))
    print(f"[cliff] pack: bf16 {bf16:.1f} us, fp32 {f32:.1f} us", flush=True)
    assert f32 <= 1.4 * bf16


@pytest.mark.parametrize("H,E,F", [(2048, 1, 1024), (4096, 2, 256), (512, 2, 2048)])
def test_fp32_past_the_decode_batch(moe, H, E, F):
    """A layer of few experts in fp32 with 64 tokens (the decode kernels) and with 96: half as many
    rows again, which took 2.0 to 3.1 times as long where every item was 128 x 128 (now 0.9 to 1.4)."""
    from paper_2608_21614_amd.device import DeviceLayer
    from workloads import make_layer
    calls = []
    for T in (64, 96):
        dev = DeviceLayer(make_layer(T, H, E, F, 1, dtype="f32", n_resident=E, residency="random", seed=3))
        args = dev.args(dev.alloc_outputs())
        calls.append(lambda dev=dev, args=args: moe.moe_layer_forward(args, dev.ws))
    few, more = times_us(*calls)
    print(f"[cliff] fp32 H={H} E={E} F={F}: 64 tokens {few:.1f} us, 96 tokens {more:.1f} us", flush=True)
    assert more <= 1.7 * few


def test_fp32_offloaded_rows_pack_at_the_copy_rate(moe):
    """What the offloaded rows add to an fp32 prefill layer (about 195 MB written from a batch that
    the caches hold) against a plain copy of as many bytes: 0.77 of it, and 1.36 with a quarter of
    the workgroups."""
    from paper_2608_21614_amd.device import DeviceLayer
    from workloads import make_layer
    dev = DeviceLayer(make_layer(4096, 2048, 64, 64, 6, dtype="f32", n_resident=2, residency="random", seed=3))
    o = dev.alloc_outputs()
    calls = [lambda a=dev.args(o, pack_offloaded=p): moe.moe_layer_forward(a, dev.ws) for p in (True, False)]
    calls[0]()
    torch.cuda.synchronize()
    n_off = 4096 * 6 - int(o["n_res"][0])
    src = torch.randn((n_off, 2048), device="cuda")
    with_pack, without, copy = times_us(*calls, lambda: o["off_rows"][:n_off].copy_(src))
    print(f"[cliff] fp32 pack of {n_off} rows: {with_pack - without:.1f} us, copy {copy:.1f} us", flush=True)
    assert with_pack - without <= copy


def test_repack_of_wide_rows_either_side_of_one_launch(moe):
    """moe_repack with offloaded rows of 64 KB: 512 pairs (one launch) against 520 (two): 0.9 times as
    long, and 1.7 where 128 workgroups packed the rows."""
    graphs = []
    for T in (64, 65):
        E, k, H, r = 128, 8, 16384, 16
        P = T * k
        dims = moe.make_dims(T, H, E, 64, k, slots=r, dtype=moe.MOE_F32)
        g = torch.Generator().manual_seed(T)
        idx = torch.stack([torch.randperm(E, generator=g)[:k] for _ in range(T)]).int().cuda()
        slot = torch.full((E,), -1, dtype=torch.int32)
        slot[:r] = torch.arange(r, dtype=torch.int32)
        i32 = [torch.empty(n, dtype=torch.int32, device="cuda") for n in (E, E, P, P, 1)]
        x, rows = torch.randn((T, H), device="cuda"), torch.empty((P, H), device="cuda")
        w, off_w, slot = torch.rand((T, k), device="cuda"), torch.empty(P, device="cuda"), slot.cuda()
        keep = (idx, slot, i32, x, rows, w, off_w)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                moe.moe_repack(dims, idx, w, slot, x, *i32, rows, off_w)
        graphs.append((graph, keep))
    one, two = times_us(*(lambda g=g: g.replay() for g, _ in graphs))
    print(f"[cliff] repack of 64 KB rows: 512 pairs {one / 10:.1f} us, 520 pairs {two / 10:.1f} us", flush=True)
    assert one <= 1.3 * two
