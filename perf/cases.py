"""Performance cases of the MoE layer: what a serving program asks of this library.

A case is a plain dict.  ``kind`` names the calls that one pass makes:

* ``layer``  ``moe_layer_forward``: router, top-k gate, repacking, expert FFN, combine.
  With ``offload`` the caller also takes the list of offloaded rows for the host.
* ``hybrid`` the same layer as the four separate calls that a CPU-GPU hybrid runtime makes
  (``moe_route_topk``, ``moe_repack``, ``moe_grouped_ffn``, ``moe_combine``), with the host's
  results for the offloaded rows merged by the combine.
* ``route``  ``moe_route_topk`` alone: the routing step of a runtime that places experts itself.
* ``load``   ``moe_pack_weights`` on one expert's two matrices: an expert enters a slot.

Sizes: ``tokens`` T, ``hidden`` H, ``experts`` E, ``ffn`` F, ``top_k`` k, ``shared`` S experts of
width ``shared_ffn``, ``resident`` experts in slots, ``dtype``, and ``zipf`` (the router bias makes
expert popularity Zipf(1.1) and the most popular experts are the resident ones; otherwise the
resident ones are drawn at random).  Inputs follow the synthetic layers of ``workloads``:
x ~ N(0, 1), weights ~ N(0, 0.02^2).
"""
from __future__ import annotations

import math

import torch

import paper_2608_21614_amd as moe

_W_STD = 0.02
_ZIPF = 1.1


def _case(kind, tokens, hidden, experts, ffn, top_k, resident, dtype="bf16", shared=0, shared_ffn=0, zipf=False,
          offload=False, name=None):
    c = {"kind": kind, "tokens": tokens, "hidden": hidden, "experts": experts, "ffn": ffn, "top_k": top_k,
         "resident": resident, "dtype": dtype, "shared": shared, "shared_ffn": shared_ffn, "zipf": zipf,
         "offload": offload}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one user's decode step, a model of many small experts: launches and latency
        _case("layer", 1, 2048, 128, 768, 8, 128, zipf=True, name="decode_1"),
        # the smallest layer of the repository, in fp32 (parity and unit-test sized work)
        _case("layer", 16, 256, 8, 512, 2, 8, dtype="f32", name="tiny_f32"),
        # decode under tight memory: 2 of 8 wide experts resident, the other pairs go to the host
        _case("layer", 16, 4096, 8, 14336, 2, 2, offload=True, name="decode_16_offload"),
        # the benchmark's decode batch: 4 of 8 wide experts
        _case("layer", 32, 4096, 8, 14336, 2, 4, offload=True, name="decode_32"),
        # a fine-grained decode batch with a wide shared expert
        _case("layer", 64, 2048, 60, 1408, 4, 30, shared=1, shared_ffn=5632, zipf=True, offload=True,
              name="decode_64_shared"),
        # the hybrid runtime's GPU part of a decode batch, many small experts
        _case("hybrid", 64, 2048, 128, 768, 8, 64, zipf=True, offload=True, name="hybrid_64"),
        # a large decode batch or a short prefill remainder, ragged, many small experts
        _case("layer", 150, 2048, 128, 768, 8, 64, zipf=True, offload=True, name="batch_150"),
        # a ragged prefill chunk over wide experts, all resident
        _case("layer", 333, 4096, 8, 14336, 2, 8, name="prefill_333_wide"),
        # the benchmark's prefill chunk
        _case("layer", 2048, 2048, 64, 1408, 6, 48, shared=2, shared_ffn=1408, zipf=True, name="prefill_2048"),
        # a long prompt in one call, everything resident
        _case("layer", 8192, 2048, 64, 1408, 6, 64, shared=2, shared_ffn=1408, zipf=True, name="prefill_8192"),
        # the benchmark's prefill chunk in fp32
        _case("layer", 2048, 2048, 64, 1408, 6, 48, dtype="f32", shared=2, shared_ffn=1408, zipf=True,
              name="prefill_2048_f32"),
        # a stage boundary brings a wide expert into a slot
        _case("load", 1, 4096, 8, 14336, 2, 1, name="load_expert"),
    ]


def _loguniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: any kind, batch sizes 1 to 8192, few wide or many narrow experts."""
    kind = rng.choice(["layer"] * 7 + ["hybrid"] * 2 + ["route"] + ["load"])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    tokens = _loguniform(rng, 1, 8192)
    if rng.random() < 0.4:
        hidden, experts, top_k = 64 * rng.randint(32, 64), rng.choice([8, 8, 16]), rng.choice([1, 2, 2, 4])
        ffn = 64 * _loguniform(rng, 32, 224)
    else:
        hidden, experts, top_k = 64 * rng.randint(16, 64), rng.randint(40, 256), rng.randint(4, 8)
        ffn = 64 * rng.randint(8, 32)
    resident = max(1, experts // rng.choice([1, 2, 2, 4, 8]))
    shared = rng.choice([0, 0, 1, 2])
    shared_ffn = 64 * rng.randint(8, 48) if shared else 0
    # bounds of the listed cases: weights on the card, and the largest batch's arithmetic
    elt = 2 if dtype == "bf16" else 4
    while resident > 1 and 3 * hidden * ffn * elt * resident > 2.8e9:
        resident //= 2
    per_token = 6.0 * hidden * (ffn * top_k + shared_ffn * shared)
    tokens = max(1, min(tokens, int((9.0e11 if dtype == "bf16" else 1.7e11) / per_token)))
    return _case(kind, tokens, hidden, experts, ffn, top_k, resident, dtype, shared, shared_ffn,
                 zipf=rng.random() < 0.6, offload=kind == "hybrid" or (kind == "layer" and tokens <= 64))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _randn(seed, tag, shape, std, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 100003 + tag)
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)


def _popularity(case):
    r = torch.arange(1, case["experts"] + 1, dtype=torch.float64)
    p = r ** -_ZIPF if case["zipf"] else torch.ones_like(r)
    return p / p.sum()


def _routing_inputs(case, seed):
    """x, router weight, bias (or None), expert -> slot map."""
    T, H, E, R = case["tokens"], case["hidden"], case["experts"], case["resident"]
    dt = _torch_dtype(case)
    x = _randn(seed, 1, (T, H), 1.0, dt)
    wr = _randn(seed, 2, (E, H), _W_STD, dt)
    g = torch.Generator().manual_seed(int(seed) * 100003 + 3)
    order = torch.randperm(E, generator=g)  # order[r]: the expert of popularity rank r
    bias = None
    if case["zipf"]:
        scale = _W_STD * math.sqrt(H) * math.sqrt(6.0) / math.pi
        b = torch.empty(E, dtype=torch.float32)
        b[order] = (scale * torch.log(_popularity(case))).float()
        bias = b.cuda()
    slot = torch.full((E,), -1, dtype=torch.int32)
    slot[order[:R]] = torch.randperm(R, generator=g).to(torch.int32)
    return x, wr, bias, slot.cuda()


def _expert(case, seed, slot, shared=False):
    """Row-major [2F, H] (gate rows, then up rows) and [H, F] of the expert in a slot, or of a shared one."""
    H, F = case["hidden"], case["shared_ffn" if shared else "ffn"]
    tag = (5000 if shared else 1000) + 2 * slot
    dt = _torch_dtype(case)
    return _randn(seed, tag, (2 * F, H), _W_STD, dt), _randn(seed, tag + 1, (H, F), _W_STD, dt)


def _host_results(case, seed):
    """The host's outputs for the offloaded rows (as many as there could be)."""
    std = 0.02 * _W_STD * case["hidden"] * math.sqrt(case["ffn"])  # about an expert output's size
    return _randn(seed, 4, (case["tokens"] * case["top_k"], case["hidden"]), std, torch.float32)


def _packed(case, seed, n, shared=False):
    if n == 0:
        return None, None
    H, F, dt = case["hidden"], case["shared_ffn" if shared else "ffn"], _torch_dtype(case)
    w13 = torch.empty((n, 2 * F, H), dtype=dt, device="cuda")
    w2 = torch.empty((n, H, F), dtype=dt, device="cuda")
    for i in range(n):
        a, b = _expert(case, seed, i, shared)
        moe.moe_pack_weights(a, w13[i])
        moe.moe_pack_weights(b, w2[i])
    return w13, w2


def prepare(case, seed):
    T, H, E, k, S = case["tokens"], case["hidden"], case["experts"], case["top_k"], case["shared"]
    dt = _torch_dtype(case)
    code = moe.MOE_BF16 if case["dtype"] == "bf16" else moe.MOE_F32
    st = {"case": case, "code": code}
    if case["kind"] == "load":
        st["src"] = _expert(case, seed, 0)
        st["dst"] = tuple(torch.empty_like(w) for w in st["src"])
        return st

    def i32(*shape):
        return torch.zeros(shape, dtype=torch.int32, device="cuda")

    def f32(*shape):
        return torch.zeros(shape, dtype=torch.float32, device="cuda")

    st["x"], st["wr"], st["bias"], st["slot"] = _routing_inputs(case, seed)
    dims = st["dims"] = moe.make_dims(T, H, E, case["ffn"], k, S, case["shared_ffn"], case["resident"], code)
    st["ws"] = torch.empty(moe.moe_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    st["logits"], st["idx"], st["w"] = f32(T, E), i32(T, k), f32(T, k)
    if case["kind"] == "route":
        return st
    st["w13"], st["w2"] = _packed(case, seed, case["resident"])
    st["ws13"], st["ws2"] = _packed(case, seed, S, shared=True)
    st["out"] = torch.empty((T, H), dtype=dt, device="cuda")
    if case["offload"]:
        st["counts"], st["seg"], st["n_res"] = i32(E), i32(E), i32(1)
        st["perm"], st["inv"] = i32(T * k), i32(T * k)
        st["off_rows"], st["off_w"] = torch.zeros((T * k, H), dtype=dt, device="cuda"), f32(T * k)
    if case["kind"] == "hybrid":
        st["y"] = f32(T * k + S * T, H)
        st["y_off"] = _host_results(case, seed)
    else:
        more = {}
        if case["offload"]:
            more = {"counts": st["counts"], "seg_start": st["seg"], "perm": st["perm"], "inv_perm": st["inv"],
                    "n_res": st["n_res"], "off_rows": st["off_rows"], "off_w": st["off_w"]}
        st["args"] = moe.layer_args(dims, st["x"], st["wr"], st["bias"], st["slot"], st["w13"], st["w2"], st["ws13"],
                                    st["ws2"], st["out"], code, logits=st["logits"], topk_idx=st["idx"],
                                    topk_w=st["w"], **more)
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "load":
        for src, dst in zip(st["src"], st["dst"]):
            moe.moe_pack_weights(src, dst)
        return list(st["dst"])
    if case["kind"] == "route":
        moe.moe_route_topk(st["dims"], st["x"], st["wr"], st["bias"], st["logits"], st["idx"], st["w"], st["ws"])
        return [st["logits"], st["idx"], st["w"]]
    if case["kind"] == "hybrid":
        d = st["dims"]
        moe.moe_route_topk(d, st["x"], st["wr"], st["bias"], st["logits"], st["idx"], st["w"], st["ws"])
        moe.moe_repack(d, st["idx"], st["w"], st["slot"], st["x"], st["counts"], st["seg"], st["perm"], st["inv"],
                       st["n_res"], st["off_rows"], st["off_w"])
        moe.moe_grouped_ffn(d, st["x"], st["perm"], st["counts"], st["seg"], st["slot"], st["w13"], st["w2"],
                            st["ws13"], st["ws2"], st["y"], st["ws"])
        moe.moe_combine(d, st["idx"], st["w"], st["inv"], st["slot"], st["y"], st["y_off"], st["n_res"], st["out"],
                        st["code"])
    else:
        moe.moe_layer_forward(st["args"], st["ws"])
    outs = [st["out"], st["logits"], st["idx"], st["w"]]
    if case["offload"]:
        outs += [st["counts"], st["n_res"], st["perm"], st["off_rows"], st["off_w"]]
    return outs


# ---------------------------------------------------------------------------
# accounting and references
# ---------------------------------------------------------------------------

def _inclusion(case):
    """Share of the tokens that select the expert of each popularity rank (they add up to k)."""
    p, k = _popularity(case), case["top_k"]
    if k >= case["experts"]:
        return torch.ones_like(p)
    lo, hi = 0.0, 1e12
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        if float((1 - torch.exp(-mid * p)).sum()) < k:
            lo = mid
        else:
            hi = mid
    return 1 - torch.exp(-hi * p)


def work(case):
    T, H, E, F, k = case["tokens"], case["hidden"], case["experts"], case["ffn"], case["top_k"]
    S, Fs = case["shared"], case["shared_ffn"]
    b = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "load":
        return {"bytes": 2 * 3 * F * H * b, "flops": 0}
    byts = (T * H + E * H) * b + 4 * (T * E + 2 * T * k)  # x and the router in; scores, ids and gates out
    flops = 2.0 * T * H * E
    if case["kind"] == "route":
        return {"bytes": byts, "flops": flops}
    q = _inclusion(case)[:case["resident"]]
    active, pairs = float((1 - (1 - q) ** T).sum()), float(T * q.sum())
    off = T * k - pairs
    byts += 3 * H * (F * active + Fs * S) * b + T * H * b  # active experts' weights, the output
    flops += 6.0 * H * (F * pairs + Fs * S * T)
    if case["offload"]:
        byts += off * (H * b + 4) + 4 * (E + 1 + T * k)
    if case["kind"] == "hybrid":
        byts += off * H * 4  # the host's results
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["kind"] == "load":
        return "exact"
    # whole values: a near tie of two scores may order or choose them the other way
    differ = 2e-3 if case["tokens"] > 64 else 0.02
    if case["kind"] == "route" or case["dtype"] == "f32":
        return {"rel": 1e-5, "differ": differ}
    return {"rel": 1e-2, "differ": differ}


def _ffn64(x, w13, w2):
    F = w13.shape[0] // 2
    h = x @ w13.double().t()
    return (torch.nn.functional.silu(h[:, :F]) * h[:, F:]) @ w2.double().t()


def exact(case, seed):
    if case["kind"] == "load":
        outs = []
        for w in _expert(case, seed, 0):  # blocks of 16 rows x 32 columns; piece l: row l % 16, columns 8 (l // 16)..
            R, K = w.shape
            outs.append(w.view(R // 16, 16, K // 32, 4, 8).permute(0, 2, 3, 1, 4).reshape(R, K))
        return outs
    T, H, E, k, S = case["tokens"], case["hidden"], case["experts"], case["top_k"], case["shared"]
    x, wr, bias, slot = _routing_inputs(case, seed)
    x64 = x.double()
    logits = x64 @ wr.double().t()
    if bias is not None:
        logits = logits + bias.double()
    top, idx = torch.sort(logits, dim=1, descending=True, stable=True)
    top, idx = top[:, :k], idx[:, :k]
    w = torch.softmax(top, dim=1)
    outs = [logits, idx.to(torch.int32), w]
    if case["kind"] == "route":
        return outs
    # packed order: resident pairs first, then offloaded; by expert, then by token
    flat = idx.reshape(-1)
    res_pair = (slot >= 0)[flat]
    key = torch.where(res_pair, 0, E) + flat
    perm = torch.sort(key, stable=True).indices
    n_res = int(res_pair.sum())
    out = torch.zeros((T, H), dtype=torch.float64, device="cuda")
    gate = w.reshape(-1)
    for e in range(E):
        s = int(slot[e])
        q = (flat == e).nonzero()[:, 0] if s >= 0 else None
        if q is None or q.numel() == 0:
            continue
        tok = q // k
        out.index_add_(0, tok, _ffn64(x64[tok], *_expert(case, seed, s)) * gate[q][:, None])
    if case["kind"] == "hybrid":
        q = perm[n_res:]
        out.index_add_(0, q // k, _host_results(case, seed)[:q.numel()].double() * gate[q][:, None])
    for s in range(S):
        out += _ffn64(x64, *_expert(case, seed, s, shared=True))
    outs = [out] + outs
    if case["offload"]:
        counts = torch.bincount(flat, minlength=E).to(torch.int32)
        off_rows = torch.zeros((T * k, H), dtype=x.dtype, device="cuda")
        off_w = torch.zeros(T * k, dtype=torch.float64, device="cuda")
        q = perm[n_res:]
        off_rows[:q.numel()] = x[q // k]
        off_w[:q.numel()] = gate[q]
        outs += [counts, torch.tensor([n_res], dtype=torch.int32, device="cuda"), perm.to(torch.int32), off_rows,
                 off_w]
    return outs
