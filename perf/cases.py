"""Performance cases of the ReTopK library: what a serving program has it do.

Every case goes through the public entry points of
``paper_2607_27692_amd.retopk``: one decode step of one attention layer (the
call made once per layer and token), one Exact Top-K or full-attention call on
the same layer (the path's two baselines, and the choice below the context
where the selector pays off), or the initialisation of a layer's
query-support cache at the end of a prompt, read back as a program that keeps
prompt caches does.

Keys, values and queries follow the synthetic workloads of
``paper_2607_27692_amd.inputs`` (clustered keys, queries on a random walk with
jumps), drawn on the GPU from the seed.  A decoding state holds a walk of
several cache lengths of queries and moves one query and one KV row further
per call, so that repeated calls meet the path mix of a running decode (reuse,
similarity fallback, scheduled refresh) and not one query again and again;
after the allocated rows the length stays, and after the last query the walk
starts over, when the cache no longer holds its first queries.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_27692_amd import retopk as R

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, batch, hq, hkv, d, dtype, context, k, cap, r, window, tau, refresh,
          centers, jump, grow):
    c = dict(kind=kind, batch=batch, hq=hq, hkv=hkv, d=d, dtype=dtype, context=context, k=k,
             cap=cap, r=r, window=window, tau=tau, refresh=refresh, centers=centers, jump=jump,
             grow=grow)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one fp32 head on 2K rows, where launches are all there is.
        _case("decode_2k_f32", "decode", 1, 1, 1, 64, "f32", 2048, 32, 64, 4, 64, 0.8, 16, 16,
              0.1, 64),
        # One layer (32 query heads on 8 KV heads) early in a conversation.
        _case("decode_16k", "decode", 1, 32, 8, 128, "bf16", 16384, 256, 256, 4, 128, 0.8, 32,
              64, 0.05, 128),
        # The headline layer: 128K rows, K = 512.
        _case("decode_128k", "decode", 1, 32, 8, 128, "bf16", 131072, 512, 512, 8, 256, 0.8, 64,
              256, 0.05, 256),
        # 28 query heads on 4 KV heads (groups of 7) with the paper's default selector settings.
        _case("decode_128k_28x4", "decode", 1, 28, 4, 128, "bf16", 131072, 512, 32, 4, 32, 0.85,
              128, 256, 0.05, 256),
        # Four sequences whose queries jump often: most KV groups take the full scan.
        _case("decode_64k_x4", "decode", 4, 32, 8, 128, "bf16", 65536, 1024, 512, 8, 256, 0.9,
              16, 256, 0.3, 256),
        # The longest context of the context sweep.
        _case("decode_1m", "decode", 1, 32, 8, 128, "bf16", 1048576, 512, 512, 8, 256, 0.8, 64,
              2048, 0.05, 64),
        # Exact Top-K where it is still the faster choice for a layer.
        _case("exact_32k", "exact", 1, 32, 8, 128, "bf16", 32768, 512, 256, 8, 128, 0.8, 32, 128,
              0.05, 256),
        # Exact Top-K on the headline layer (also what a refresh step costs).
        _case("exact_128k", "exact", 1, 32, 8, 128, "bf16", 131072, 512, 512, 8, 256, 0.8, 64,
              256, 0.05, 256),
        # Exact Top-K without a handle (serving loops that cannot allocate), heads of 64
        # elements, a length that is a multiple of nothing.
        _case("exact_noalloc_d64", "noalloc", 2, 16, 8, 64, "bf16", 23001, 256, 32, 4, 32, 0.85,
              128, 64, 0.05, 7),
        # Full attention over a short history: few rows for a whole chip.
        _case("full_16k_28x4", "full", 1, 28, 4, 128, "bf16", 16384, 512, 32, 4, 32, 0.85, 128,
              256, 0.05, 128),
        # Full attention on the headline layer.
        _case("full_128k", "full", 1, 32, 8, 128, "bf16", 131072, 512, 512, 8, 256, 0.8, 64, 256,
              0.05, 256),
        # The end of a 128K prompt: 512 cache entries per head, each with its exact support.
        _case("prefill_128k", "prefill", 1, 32, 8, 128, "bf16", 131072, 512, 512, 8, 256, 0.8, 64,
              256, 0.05, 1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["exact"] * 2 + ["full"] * 2 + ["prefill"] * 2 + ["noalloc"])
    # bf16 is what models store; fp32 is the small-model and debugging type
    dtype = "bf16" if rng.random() < 0.85 else "f32"
    hq, hkv = rng.choice([(32, 8), (32, 8), (28, 4), (40, 8), (16, 8), (8, 8), (24, 8), (8, 1),
                          (12, 2), (1, 1)])
    d = rng.choice([128, 128, 128, 64])
    batch = rng.choice([1, 1, 1, 2, 3, 4]) if kind != "prefill" else rng.choice([1, 1, 2])
    # rows of all sequences and KV heads: no more than the largest listed case of the kind reads
    most = {"decode": 4 << 20, "exact": 1 << 20, "full": 1 << 20, "noalloc": 1 << 20,
            "prefill": 1 << 20}[kind]
    hi = min(1 << 20, most // (batch * hkv))
    cap = rng.choice([32, 64, 100, 128, 256, 512])
    if kind == "noalloc":        # the library's fixed scratch of 64 MiB
        hi = min(hi, ((60 << 20) // (batch * hq) - 9000) // 13 // 4096 * 4096)
    if kind == "prefill":        # no more scores than the largest listed prefill
        hi = min(hi, (1 << 31) // (batch * hq * cap), 1 << 17)
        if dtype == "f32":       # one position at a time
            hi, cap = min(hi, 16384), min(cap, 64)
    if dtype == "f32":
        hi = min(hi, max(2048, (1 << 19) // (batch * hkv)))
    context = _log_int(rng, 1024, max(1100, hi))
    if rng.random() < 0.3:
        context = max(1024, context >> 10 << 10)
    k = min(rng.choice([32, 64, 128, 256, 300, 512, 512, 1024]), context // 4)
    r = rng.choice([1, 4, 4, 8, 8])
    window = rng.choice([0, 32, 128, 200, 256])
    tau = rng.choice([0.8, 0.8, 0.85, 0.9])
    return _case(None, kind, batch, hq, hkv, d, dtype, context, k, min(cap, context // 2), r,
                 window, tau, rng.choice([0, 16, 32, 64, 128]), max(16, min(2048, context // k)),
                 rng.choice([0.02, 0.05, 0.05, 0.1, 0.3]), rng.choice([7, 64, 256]))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _config(case):
    return dict(batch=case["batch"], n_q_heads=case["hq"], n_kv_heads=case["hkv"],
                head_dim=case["d"], max_len=case["context"] + case["grow"], k=case["k"],
                cache_cap=case["cap"], r=case["r"], window=case["window"], tau=case["tau"],
                refresh=case["refresh"], dtype=case["dtype"])


def _n_queries(case):
    """Decode queries of a state: several cache lengths for a decode, else a few."""
    if case["kind"] == "decode":
        return max(256, 4 * case["cap"])
    return 1 if case["kind"] == "prefill" else 16


def _inputs(case, seed):
    """K and V [B, Hkv, rows, d], prompt-tail queries [B, Hq, cap, d] and decode
    queries [T, B, Hq, d], as paper_2607_27692_amd.inputs draws them."""
    dev = torch.device("cuda")
    gen = torch.Generator(dev)
    gen.manual_seed(seed)
    B, Hq, Hkv, d = case["batch"], case["hq"], case["hkv"], case["d"]
    rows, nc, dt = case["context"] + case["grow"], case["centers"], _DTYPES[case["dtype"]]
    centers = torch.randn((B, Hkv, nc, d), generator=gen, device=dev) / math.sqrt(d)
    k = torch.empty((B, Hkv, rows, d), dtype=dt, device=dev)
    v = torch.empty((B, Hkv, rows, d), dtype=dt, device=dev)
    for b in range(B):
        for g in range(Hkv):
            z = torch.randint(nc, (rows,), generator=gen, device=dev)
            x = torch.randn((rows, d), generator=gen, device=dev)
            k[b, g] = x.add_(centers[b, g][z], alpha=2.0)
            v[b, g] = torch.randn((rows, d), generator=gen, device=dev)
    n = case["cap"] + _n_queries(case)
    unit = centers / centers.norm(dim=-1, keepdim=True) * math.sqrt(d)
    unit = unit.repeat_interleave(Hq // Hkv, dim=1).reshape(B * Hq, nc, d)
    target = torch.randint(nc, (n, B * Hq), generator=gen, device=dev)
    jumps = torch.rand((n, B * Hq, 1), generator=gen, device=dev) < case["jump"]
    noise = torch.randn((n, B * Hq, d), generator=gen, device=dev) * 0.436
    lane = torch.arange(B * Hq, device=dev)
    walk = torch.empty((n, B * Hq, d), device=dev)
    q = unit[lane, target[0]]
    walk[0] = q
    root = math.sqrt(d)
    for u in range(1, n):
        x = torch.add(noise[u], q, alpha=0.9)
        q = torch.where(jumps[u], unit[lane, target[u]], x * (root / x.norm(dim=-1, keepdim=True)))
        walk[u] = q
    walk = walk.to(dt)
    tail = walk[:case["cap"]].permute(1, 0, 2).reshape(B, Hq, case["cap"], d).contiguous()
    return k, v, tail, walk[case["cap"]:].reshape(-1, B, Hq, d).contiguous()


def prepare(case, seed):
    k, v, tail, dec = _inputs(case, seed)
    cfg = _config(case)
    s = dict(case=case, k=k, v=v, tail=tail, dec=dec, t=0)
    shape = (case["batch"], case["hq"])
    if case["kind"] == "noalloc":
        s["cfg"] = R.make_config(**cfg)
    else:
        s["h"] = R.Handle(**cfg)
    if case["kind"] == "prefill":
        # where the program keeps a prompt's cache on the host
        bh, cap = case["batch"] * case["hq"], case["cap"]
        host = dict(qbar=torch.empty((bh, cap, case["d"]), dtype=torch.float32, pin_memory=True),
                    supp=torch.empty((bh, cap, case["k"]), dtype=torch.int32, pin_memory=True),
                    cnt=torch.empty((bh, cap), dtype=torch.int32, pin_memory=True))
        s["host"] = {name: x.numpy() for name, x in host.items()}
        s["pinned"] = host
        return s
    s["out"] = torch.empty(shape + (case["d"],), dtype=torch.float32, device="cuda")
    if case["kind"] != "full":
        s["sel"] = torch.empty(shape + (case["k"],), dtype=torch.int32, device="cuda")
    if case["kind"] == "decode":
        s["h"].prefill_init(tail, case["cap"], k, v, case["context"])
    return s


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "prefill":
        h, host = state["h"], state["host"]
        h.prefill_init(state["tail"], case["cap"], state["k"], state["v"], case["context"])
        R.retopk_get_state(h.h, host["qbar"], host["supp"], host["cnt"])
        return host
    t = state["t"]
    state["t"] = t + 1
    q = state["dec"][t % state["dec"].shape[0]]
    length = case["context"] + min(t + 1, case["grow"])
    if kind == "full":
        state["h"].full(q, state["k"], state["v"], length, state["out"])
        return {"out": state["out"]}
    if kind == "decode":
        state["h"].decode_step(q, state["k"], state["v"], length, state["out"], state["sel"])
    elif kind == "exact":
        state["h"].exact(q, state["k"], state["v"], length, state["out"], state["sel"])
    else:
        R.exact_topk_attention_noalloc(state["cfg"], q, state["k"], state["v"], length,
                                       state["out"], state["sel"])
    return {"out": state["out"], "sel": state["sel"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without, and what it may differ by
# ---------------------------------------------------------------------------

def work(case):
    B, Hq, Hkv, d, K, C = (case[x] for x in ("batch", "hq", "hkv", "d", "k", "cap"))
    e = 2 if case["dtype"] == "bf16" else 4
    n, heads = case["context"] + 1, B * Hq
    io = heads * (d * e + d * 4)                      # queries in, outputs out
    support = heads * K * 4
    if case["kind"] == "prefill":
        return {"bytes": B * Hkv * n * d * e + heads * C * (d * e + d * 4 + K * 4),
                "flops": 2.0 * heads * C * n * d}
    if case["kind"] == "full":
        return {"bytes": 2 * B * Hkv * n * d * e + io, "flops": 4.0 * heads * n * d}
    values = heads * K * d * e
    if case["kind"] in ("exact", "noalloc"):
        return {"bytes": B * Hkv * n * d * e + values + io + support,
                "flops": 2.0 * heads * (n + K) * d}
    # A decode step: the cached queries, the retrieved supports, their keys and the
    # window's (at least one support's worth), the selected values, the cache entry
    # written; and the keys of the KV groups in which some head's query jumped.
    scanned = B * Hkv * (1.0 - (1.0 - case["jump"]) ** (Hq // Hkv))
    cand = K + case["window"]
    step = heads * (C * d * 4 + min(case["r"], C) * K * 4 + cand * d * e + d * 4 + K * 4)
    return {"bytes": step + scanned * n * d * e + values + io + support,
            "flops": 2.0 * heads * (C + cand + K) * d + 2.0 * scanned * (Hq // Hkv) * n * d}


def tolerance(case):
    if case["kind"] == "prefill":
        # normalised queries: one rounding to fp32; supports: near ties at the K-th score
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}
    if case["kind"] == "full":
        return {"rel": 1e-5}
    # fp32 sums in any order are within 1e-6.  A near tie at a head's K-th score can
    # go either way, which swaps one support entry of that head: against 64-bit
    # scores one such swap among 128 heads measured 2.3e-3 (one head of 128 off by
    # 2.6e-2), in about one pass of four at K = 1024.
    return {"rel": 1e-2, "max": 0.3, "differ": 0.01}


# ---------------------------------------------------------------------------
# 64-bit results
# ---------------------------------------------------------------------------

def _attend(q, k, v, idx):
    """Softmax attention of one query over rows idx of k and v, in float64."""
    s = (k[idx].double() @ q) / math.sqrt(q.shape[0])
    p = torch.softmax(s, dim=0)
    return p @ v[idx].double()


def _top_k(q, k, n, K):
    """Indices of the K largest float64 scores of rows [0, n)."""
    s = k[:n].double() @ q
    return torch.topk(s, min(K, n)).indices


def exact(case, seed):
    """The first pass of run() on a new state."""
    k, v, tail, dec = _inputs(case, seed)
    B, Hq, Hkv, d = case["batch"], case["hq"], case["hkv"], case["d"]
    G, C, K, n = Hq // Hkv, case["cap"], case["k"], case["context"] + 1
    unit = lambda x: x / x.norm(dim=-1, keepdim=True)  # noqa: E731
    if case["kind"] == "prefill":
        return {"qbar": unit(tail.double()).reshape(B * Hq, C, d).cpu().numpy(), "supp": None,
                "cnt": None}
    out = torch.empty((B, Hq, d), dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(Hq):
            kk, vv, q = k[b, h // G], v[b, h // G], dec[0, b, h].double()
            if case["kind"] == "full":
                idx = torch.arange(n, device="cuda")
            elif case["kind"] != "decode":
                idx = _top_k(q, kk, n, K)
            else:
                rho = unit(tail[b, h].double()) @ unit(q)
                best = torch.topk(rho, min(case["r"], C))
                if float(best.values[0]) < case["tau"]:
                    idx = _top_k(q, kk, n, K)
                else:
                    sets = [_top_k(tail[b, h, u].double(), kk, case["context"] - C + u + 1, K)
                            for u in best.indices.tolist()]
                    sets.append(torch.arange(max(0, n - case["window"]), n, device="cuda"))
                    cand = torch.unique(torch.cat(sets))
                    s = kk[cand].double() @ q
                    idx = cand[torch.topk(s, min(K, cand.numel())).indices]
            out[b, h] = _attend(q, kk, vv, idx)
    return {"out": out} if case["kind"] == "full" else {"out": out, "sel": None}
