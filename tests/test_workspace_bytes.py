"""moe_workspace_bytes of prefill shapes: the item tables' room in it does not depend on
the FFN's tiles (the fixed scratch array accepts or refuses a layer by this size)."""
from __future__ import annotations

import random

import paper_2608_21614_amd as moe


def _ceil(a, b):
    return -(-a // b)


def _expected(T, H, E, F, k, S, Fs, slots, bf16):
    def a256(n):
        return _ceil(max(n, 1), 256) * 256
    P, G = T * k, min(E, slots, T * k)
    head = [T * E * 4, P * 4, P * 4, E * 4, E * 4, 4, P * 4, P * 4, 0]
    if not bf16:
        return sum(a256(n) for n in head + [(P + S * T) * max(F, Fs if S else 0) * 4, 0, 0, (P + S * T) * H * 4])
    rt = 0 if G == 0 else _ceil(P, 256) + G
    tps = _ceil(T, 256)
    items = rt * _ceil(F, 128) + S * tps * (_ceil(Fs, 128) if S else 0) + (rt + S * tps) * _ceil(H, 256)
    t16 = _ceil(T, 16) * 16
    rows = P + 15 * G
    return sum(a256(n) for n in head + [
        (rows + S * t16) * max(F, Fs if S else 0) * 2, (rows + (t16 if S else 0)) * H * 2, 32 + 32 * items,
        (P + S * T) * H * 2])


def test_prefill_workspace_bytes():
    rng = random.Random(5)
    for _ in range(400):
        E = rng.randint(1, 256)
        S = rng.choice([0, 0, 1, 2, 8])
        c = (rng.choice([65, 66, 100, 257, 1000, 5000]), 64 * rng.randint(1, 40), E, 64 * rng.randint(1, 40),
             rng.randint(1, min(E, 8)), S, 64 * rng.randint(1, 40) if S else 0, rng.randint(0, E))
        T, H, E, F, k, S, Fs, slots = c
        for dtype in (moe.MOE_BF16, moe.MOE_F32):
            dims = moe.make_dims(T, H, E, F, k, S, Fs, slots, dtype)
            assert moe.moe_workspace_bytes(dims) == _expected(*c, dtype == moe.MOE_BF16), (c, dtype)
