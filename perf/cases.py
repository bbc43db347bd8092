"""The cases the performance of this library is measured on: passes of the denoising step's attention path through the
public entry points (paper_2512_17077_amd.hcsa), from one tiny fp32 layer, where a call is launch latency and host
work, to the batches that fill the card.

A case is a dict of plain values:

  kind       "step"     selection, then attention over the kept rows: what a Reuse step with fresh lists runs per layer
             "select"   selection alone (K is streamed once)
             "attend"   attention over kept rows, lists in hand (K and V rows gathered)
             "packed"   packing of the kept rows at Refresh time, then attention over the packed cache
             "refresh"  dense bidirectional attention of whole sequences
             "mixed"    one call over a batch of Reuse and Refresh sequences, lists in hand
             "mixed_step"  selection for the Reuse sequences, then that one call
  dtype      "bf16" or "f32"
  hq hkv d   query heads, KV heads, head_dim
  batch      sequences; the first `dense` of a fixed shuffle of them are Refresh sequences in the mixed kinds
  kv_lo/hi   their KV lengths are drawn uniformly from this range (equal bounds: all equal), always the same for a case
  dense_kv   KV length, and number of queries, of the Refresh sequences in the mixed kinds
  keep_lo/hi retention ratio per sequence
  block      queries of a Reuse sequence (its active block)
  pool_w, forced, head_sum   options of selection
  layout     number that fixes the drawn lengths and ratios

Shapes are those of this repository's benchmark workloads and tests: 32 heads x 128 with and without grouped queries,
the tiny fp32 layer of 4 heads x 64, blocks of 32, retention 5 to 50 %, pooling window 3 by default (Table 2 of the
paper).  Values are seeded Gaussians; 5 % of the K rows are scaled up, as heads with salient positions have them.
"""
import math
import random

import torch

from paper_2512_17077_amd import hcsa

BASE = {"kind": "step", "dtype": "bf16", "hq": 32, "hkv": 32, "d": 128, "batch": 1, "dense": 0, "kv_lo": 1024, "kv_hi": 1024,
        "dense_kv": 0, "keep_lo": 0.25, "keep_hi": 0.25, "block": 32, "pool_w": 1, "forced": 0, "head_sum": 0, "layout": 0}


def _case(name, **what):
    return dict(BASE, name=name, **what)


def listed():
    return [
        # the tiny single layer (fp32, 0.3 MB): nothing but launches and host work
        _case("tiny_step_f32", dtype="f32", hq=4, hkv=4, d=64, kv_lo=256, kv_hi=256, pool_w=1),
        # one request, one layer of an 8B model (prompt 768 + generation 256): interactive use
        _case("layer_step"),
        # a handful of requests of odd lengths at the paper's defaults (window 3, half kept), the active block forced in
        _case("small_batch_step", batch=4, kv_lo=511, kv_hi=2047, keep_lo=0.5, keep_hi=0.5, pool_w=3, forced=32, layout=4),
        # a full serving batch with ragged lengths and retention: its selection and its Reuse attention
        _case("batch_select", kind="select", batch=16, kv_lo=512, kv_hi=4096, keep_lo=0.1, keep_hi=0.5, layout=3),
        _case("batch_attend", kind="attend", batch=16, kv_lo=512, kv_hi=4096, keep_lo=0.1, keep_hi=0.5, layout=3),
        # the same batch with the packed cache: packed once after a Refresh, then attended over
        _case("batch_packed", kind="packed", batch=16, kv_lo=512, kv_hi=4096, keep_lo=0.1, keep_hi=0.5, layout=3),
        # Refresh of one request, of a full batch, and of a ragged batch of a small grouped-query model
        _case("layer_refresh", kind="refresh"),
        _case("batch_refresh", kind="refresh", batch=8, kv_lo=2048, kv_hi=2048),
        _case("ragged_refresh_d64", kind="refresh", hq=16, hkv=4, d=64, batch=7, kv_lo=300, kv_hi=3000, layout=7),
        # long-context burst with grouped queries: 24 Reuse sequences beside 8 in Refresh
        _case("burst_select", kind="select", hkv=8, batch=24, kv_lo=8192, kv_hi=8192, keep_lo=0.05, keep_hi=0.05),
        _case("burst_attend", kind="mixed", hkv=8, batch=32, dense=8, kv_lo=8192, kv_hi=8192, dense_kv=2048, keep_lo=0.05,
              keep_hi=0.05),
        # fp32, as a reference run of a small layer uses it: Reuse sequences and one Refresh in a batch
        _case("mixed_step_f32", kind="mixed_step", dtype="f32", hq=8, hkv=4, d=64, batch=4, dense=1, kv_lo=500, kv_hi=1500,
              dense_kv=700, keep_lo=0.2, keep_hi=0.5, layout=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = dict(BASE)
        c["kind"] = rng.choice(("step", "step", "select", "attend", "packed", "refresh", "refresh", "mixed", "mixed_step"))
        c["layout"] = rng.randint(10, 10**6)
        if rng.random() < 0.15:
            c["dtype"] = "f32"
            c["hq"], c["hkv"], c["d"] = rng.choice(((4, 4, 64), (8, 4, 64), (8, 2, 128)))
            c["batch"] = _log(rng, 1, 6)
            hi = _log(rng, 200, 2000)
            most_flops, most_bytes = 1.0e9, 5e7
        else:
            c["hq"], c["hkv"], c["d"] = rng.choice(((32, 32, 128), (32, 32, 128), (32, 8, 128), (16, 4, 128), (16, 16, 64), (8, 4, 64)))
            c["batch"] = _log(rng, 1, 40)
            hi = _log(rng, 256, 8192)
            most_flops, most_bytes = 5e11, 4.5e8
        c["kv_hi"] = hi
        c["kv_lo"] = hi if rng.random() < 0.3 else max(64, int(hi * rng.uniform(0.1, 0.9)))
        a, b = sorted(rng.uniform(0.05, 0.5) for _ in range(2))
        c["keep_lo"], c["keep_hi"] = (a, b) if rng.random() < 0.6 else (a, a)
        c["block"] = rng.choice((16, 32, 32, 32, 32, 64))
        c["pool_w"] = rng.choice((1, 1, 3, 3, 5))
        c["forced"] = c["block"] if rng.random() < 0.25 else 0
        c["head_sum"] = 1 if rng.random() < 0.12 else 0
        if c["kind"].startswith("mixed"):
            if c["batch"] < 2:
                continue
            c["dense"] = rng.randint(1, max(1, c["batch"] // 3))
            c["dense_kv"] = _log(rng, 200, 2048)
        w = work(c)
        if w["bytes"] <= most_bytes and w["flops"] <= most_flops and w["flops"] / most_flops + w["bytes"] / most_bytes < 1.2:
            return c


def _layout(c):
    """(KV lengths, query counts, kept rows per head, modes) of a case's sequences."""
    rng = random.Random(c["layout"])
    n = c["batch"]
    modes = [0] * n
    if c["kind"] == "refresh":
        modes = [1] * n
    elif c["dense"]:
        for b in rng.sample(range(n), c["dense"]):
            modes[b] = 1
    kv, nq, keep = [], [], []
    for m in modes:
        length = rng.randint(c["kv_lo"], c["kv_hi"])
        ratio = rng.uniform(c["keep_lo"], c["keep_hi"])
        if m and c["kind"] != "refresh":
            length = c["dense_kv"]
        kv.append(length)
        nq.append(length if m else c["block"])
        keep.append(0 if m else min(length, max(1, c["forced"], int(ratio * length + 0.5))))
    return kv, nq, keep, modes


def _prefix(x):
    out = [0]
    for v in x:
        out.append(out[-1] + v)
    return out


def prepare(case, seed):
    c = dict(BASE, **case)
    kv, nq, keep, modes = _layout(c)
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    q = torch.randn((sum(nq), hq, d), generator=gen, device=dev, dtype=torch.float32).to(dt)
    k = torch.randn((sum(kv), hkv, d), generator=gen, device=dev, dtype=torch.float32).to(dt)
    v = torch.randn((sum(kv), hkv, d), generator=gen, device=dev, dtype=torch.float32).to(dt)
    if c["kind"] != "refresh":
        salient = torch.rand((sum(kv), hkv, 1), generator=gen, device=dev) < 0.05
        k.mul_(torch.where(salient, 4.0, 1.0).to(dt))
    cu_q, cu_kv, cu_k = (torch.tensor(_prefix(x), dtype=torch.int32, device=dev) for x in (nq, kv, keep))
    s = {"case": c, "cu_k": cu_k, "total_k": sum(keep), "max_k": max(keep), "tensors": (q, k, v, cu_q, cu_kv)}
    scale = 1.0 / math.sqrt(d)
    s["batch"] = hcsa.make_batch(q, k, v, cu_q, cu_kv, max(nq), max(kv), scale)
    s["o"] = torch.zeros_like(q)
    s["mode"] = torch.tensor(modes, dtype=torch.uint8, device=dev) if any(modes) and c["kind"] != "refresh" else None
    if c["kind"] == "refresh":
        return s

    def space(n):
        return torch.empty(n, dtype=torch.uint8, device=dev) if n else None

    s["idx"] = torch.zeros((hq, s["total_k"]), dtype=torch.int32, device=dev)
    s["ws_select"] = space(hcsa.dllm_hcsa_select_workspace(s["batch"], s["max_k"]))
    s["ws_attend"] = space(hcsa.dllm_hcsa_attend_workspace(s["batch"], s["max_k"]))
    if c["kind"] == "packed":
        s["kp"] = torch.empty((hq, s["total_k"], d), dtype=dt, device=dev)
        s["vp"] = torch.empty_like(s["kp"])
        s["packed"] = hcsa.make_packed_batch(q, s["kp"], s["vp"], cu_q, cu_k, max(nq), s["max_k"], scale)
        s["ws_attend"] = space(hcsa.dllm_hcsa_attend_workspace(s["packed"], s["max_k"]))
    if c["kind"] in ("attend", "packed", "mixed"):
        _select(s)   # the lists a Reuse step has in hand
    return s


def _select(s):
    c = s["case"]
    if c["forced"] or c["head_sum"]:
        return hcsa.dllm_hcsa_select_ex(s["batch"], s["cu_k"], s["total_k"], s["max_k"], s["idx"], c["pool_w"], c["forced"],
                                        bool(c["head_sum"]), s["ws_select"])
    return hcsa.dllm_hcsa_select(s["batch"], s["cu_k"], s["total_k"], s["max_k"], s["idx"], c["pool_w"], s["ws_select"])


def _attend(s):
    return hcsa.dllm_hcsa_attend(s["batch"], s["idx"], s["cu_k"], s["total_k"], s["max_k"], s["mode"], s["o"], s["ws_attend"])


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "refresh":
        return hcsa.dllm_dense_refresh_attend(s["batch"], s["o"])
    if kind == "select":
        return _select(s)
    if kind in ("attend", "mixed"):
        return _attend(s)
    if kind in ("step", "mixed_step"):
        _select(s)
        return {"idx": s["idx"], "o": _attend(s)}
    kp, vp = hcsa.dllm_hcsa_pack(s["batch"], s["idx"], s["cu_k"], s["total_k"], s["max_k"], s["kp"], s["vp"])
    o = hcsa.dllm_hcsa_attend(s["packed"], None, s["cu_k"], s["total_k"], s["max_k"], None, s["o"], s["ws_attend"])
    return {"k": kp, "v": vp, "o": o}


def work(case):
    c = dict(BASE, **case)
    kv, nq, keep, modes = _layout(c)
    row = c["d"] * (4 if c["dtype"] == "f32" else 2)
    sparse = [b for b in range(c["batch"]) if not modes[b]]
    kvs, nqs, kept = (sum(x[b] for b in sparse) for x in (kv, nq, keep))
    nbytes = flops = 0.0
    if c["kind"] in ("select", "step", "mixed_step"):   # K and the block's queries in, lists out
        nbytes += kvs * c["hkv"] * row + nqs * c["hq"] * row + kept * c["hq"] * 4
        flops += 2.0 * kvs * c["hq"] * c["d"]
    if c["kind"] in ("attend", "step", "mixed", "mixed_step"):   # lists, kept K and V rows and Q in, O out
        nbytes += kept * c["hq"] * (2 * row + 4) + 2 * nqs * c["hq"] * row
    if c["kind"] == "packed":   # lists and kept rows in, packed rows out; packed rows and Q in, O out
        nbytes += kept * c["hq"] * (4 * row + 4) + kept * c["hq"] * 2 * row + 2 * nqs * c["hq"] * row
    flops += 0.0 if c["kind"] in ("select", "refresh") else sum(4.0 * nq[b] * keep[b] for b in sparse) * c["hq"] * c["d"]
    for b in range(c["batch"]):
        if modes[b]:
            flops += 4.0 * nq[b] * kv[b] * c["hq"] * c["d"]
            nbytes += 2 * nq[b] * c["hq"] * row + 2 * kv[b] * c["hkv"] * row
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # Selected positions and packed rows are the same in every correct implementation (the score arithmetic is part
    # of the definition); a case that returns nothing else is exact.  Outputs of attention: against the same in fp64
    # the listed bf16 cases are off by up to 2.3e-3 (norm) and 1.5e-2 (largest; probabilities and outputs are rounded
    # to bf16), the fp32 ones by up to 6.4e-7 and 8e-6; about four times that is allowed.
    if case["kind"] == "select":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 2.6e-6, "max": 3.2e-5}
    return {"rel": 9e-3, "max": 6e-2}
