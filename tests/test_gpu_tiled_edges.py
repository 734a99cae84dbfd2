"""The prefill FFN (tiled kernels) at the edges of its tiles, against the oracle: row counts
around its token-block classes (bf16: 64, 128, 192; fp32: every 32) and its token tile (256
and 128 rows), more token tiles than one sweep takes, a single K slab pair, widths that
leave half a weight tile, and more groups and items than workgroups start with."""
from __future__ import annotations

import pytest
import torch

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
