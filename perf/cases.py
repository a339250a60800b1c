"""The calls this library is timed on: decode steps (append, then attention)
and prompt steps (prompt write, then causal attention) over a paged KV cache,
through the package's public entry points.

A case gives the shape of one layer's call: head counts, head_dim, the pools'
element type, the range the requests' lengths are drawn from (from the case's
own ``sizes`` number, so that a case's work does not depend on its inputs) and
how the call is made.  ``prepare`` draws the values from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_15330_amd as bl

PAGE = 16
FP8_MAX = 448.0


def _decode(name, B, heads, D, lo, hi, kv="bf16", rows="pool", law="uniform", graph=False, sizes=0):
    """One decode step of B requests with lo..hi tokens each (the new one
    included).  rows: "pool" = new rows in the pools' element type, "bf16" =
    bf16 rows quantised into fp8 pools.  graph: the step replayed from a HIP
    graph, as a serving loop with fixed buffers does."""
    return {"name": name, "kind": "decode", "B": B, "H_q": heads[0], "H_kv": heads[1], "D": D, "kv": kv,
            "rows": rows, "law": law, "lo": lo, "hi": hi, "graph": graph, "sizes": sizes}


def _prompt(name, B, heads, D, cached, new, kv="bf16", sizes=0):
    """One prompt step: B requests of new[0]..new[1] prompt tokens each, after
    cached[0]..cached[1] tokens already in the cache."""
    return {"name": name, "kind": "prompt", "B": B, "H_q": heads[0], "H_kv": heads[1], "D": D, "kv": kv,
            "cached_lo": cached[0], "cached_hi": cached[1], "new_lo": new[0], "new_hi": new[1], "sizes": sizes}


def listed():
    return [
        # the smallest call: a few short requests of a small model (8/2 heads
        # of 64), called eagerly, where host work and launches count
        _decode("decode_tiny", 3, (8, 2), 64, 1, 200),
        # one interactive user of an 8B-class model (32/8 heads of 128), the
        # step replayed from a graph as latency-bound serving does
        _decode("decode_one_graph", 1, (32, 8), 128, 1500, 2500, graph=True),
        # 64 requests of 1-4k tokens, the ordinary chat batch
        _decode("decode_chat", 64, (32, 8), 128, 1024, 4096),
        # 256 requests of 6-13.5k tokens, the paper's summarization batch and
        # the largest decode step here
        _decode("decode_summarization", 256, (32, 8), 128, 6000, 13500),
        # the same kind of requests on one GPU of a tensor-parallel server (4/2
        # heads a GPU), the geometry of the serving model's live mode
        _decode("decode_tp_shard", 48, (4, 2), 128, 6000, 13500),
        # fp8 pools, 64/8 heads, Zipf lengths: many short and a few long ones
        _decode("decode_fp8_zipf", 512, (64, 8), 128, 128, 32768, kv="fp8", law="zipf"),
        # fp8 pools fed with bf16 rows (quantised on append), a chat batch
        _decode("decode_fp8_quant", 32, (32, 8), 128, 500, 8000, kv="fp8", rows="bf16"),
        # the smallest prompt step: four short prompts, some after a short prefix
        _prompt("prompt_tiny", 4, (8, 2), 64, (0, 16), (1, 300)),
        # follow-up turns of chats whose history is cached
        _prompt("prompt_turns", 8, (32, 8), 128, (2000, 8000), (16, 256)),
        # one 2048-token chunk on one GPU of the tensor-parallel server
        _prompt("prompt_tp_chunk", 1, (4, 2), 128, (4000, 10000), (2048, 2048)),
        # four 2048-token chunks after their cached part, fp8 pools
        _prompt("prompt_chunked_fp8", 4, (32, 8), 128, (4000, 10000), (2048, 2048), kv="fp8"),
        # four whole prompts of 6-12k tokens: the paper's documents, the
        # largest prompt step here
        _prompt("prompt_summarization", 4, (32, 8), 128, (0, 0), (6000, 12000)),
    ]


# a drawn case stays below the largest listed ones' time: fp8 steps take
# longer a byte, and head_dim 64 prompts longer a flop
_MAX_KV_BYTES = {"bf16": 8e9, "fp8": 4e9}
_MAX_FLOPS = {64: 0.6e12, 128: 1.4e12}
_HEADS = [(32, 8), (64, 8), (8, 2), (4, 2), (16, 4), (28, 4), (32, 32), (16, 1), (12, 4), (8, 1)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        heads = rng.choice(_HEADS)
        D = rng.choice([64, 128, 128])
        kv = rng.choice(["bf16", "bf16", "fp8"])
        sizes = rng.randrange(1, 1 << 30)
        if rng.random() < 0.55:
            hi = _log_int(rng, 16, 32768)
            c = _decode("", _log_int(rng, 1, 512), heads, D, max(1, int(hi * rng.uniform(0.05, 1.0))), hi, kv=kv,
                        rows=rng.choice(["pool", "bf16"]) if kv == "fp8" else "pool",
                        law=rng.choice(["uniform", "uniform", "zipf"]), graph=rng.random() < 0.25, sizes=sizes)
        else:
            hi, ch = _log_int(rng, 4, 12000), _log_int(rng, 16, 12000)
            prefix = rng.random() < 0.6
            c = _prompt("", _log_int(rng, 1, 16), heads, D, (int(ch * rng.random()), ch) if prefix else (0, 0),
                        (max(1, int(hi * rng.random())), hi), kv=kv, sizes=sizes)
        del c["name"]
        if _kv_bytes(c) <= _MAX_KV_BYTES[kv] and work(c)["flops"] <= _MAX_FLOPS[D]:
            return c


# ------------------------------------------------------------------- sizes --

def _lengths(case):
    """(cached, new) tokens of every request before the call, int64 [B] each."""
    rng = np.random.default_rng(np.random.SeedSequence([case["sizes"], 11]))
    B = case["B"]
    if case["kind"] == "decode":
        if case["law"] == "zipf":       # P(L = k) proportional to k^-1.2
            ks = np.arange(case["lo"], case["hi"] + 1, dtype=np.int64)
            p = ks.astype(np.float64) ** -1.2
            total = rng.choice(ks, size=B, p=p / p.sum())
        else:
            total = rng.integers(case["lo"], case["hi"], size=B, endpoint=True)
        return total.astype(np.int64) - 1, np.ones(B, dtype=np.int64)
    cached = rng.integers(case["cached_lo"], case["cached_hi"], size=B, endpoint=True)
    new = rng.integers(case["new_lo"], case["new_hi"], size=B, endpoint=True)
    return cached.astype(np.int64), new.astype(np.int64)


def _kv_bytes(case):
    cached, new = _lengths(case)
    return int((cached + new).sum()) * case["H_kv"] * case["D"] * 2 * (1 if case["kv"] == "fp8" else 2)


def work(case):
    """Every K/V row read once by the attention; new rows read and written
    once; queries read, outputs written; block table, lengths and scales."""
    cached, new = _lengths(case)
    total = cached + new
    eb = 1 if case["kv"] == "fp8" else 2
    rb = 2 if case.get("rows") == "bf16" else eb
    T, D, H_kv = int(new.sum()), case["D"], case["H_kv"]
    pages = int(((total + PAGE - 1) // PAGE).sum())
    nbytes = _kv_bytes(case) + 2 * T * H_kv * D * (rb + eb) + 2 * T * case["H_q"] * D * 2
    nbytes += 4 * pages + 8 * case["B"] + (8 * case["B"] * H_kv if eb == 1 else 0)
    # query i of a request sees its cached tokens and the new ones up to its own
    pairs = int((new * cached + new * (new + 1) // 2).sum())
    return {"bytes": nbytes, "flops": 4 * D * case["H_q"] * pairs}


# ------------------------------------------------------------------ inputs --

def _inputs(case, seed):
    """Buffers of one call on the GPU: pools with every request's pages
    scattered over them, tables, lengths, queries and new rows."""
    dev = "cuda"
    cached, new = _lengths(case)
    B, H_q, H_kv, D = case["B"], case["H_q"], case["H_kv"], case["D"]
    fp8 = case["kv"] == "fp8"
    need = (cached + new + PAGE - 1) // PAGE
    NP = int(need.sum()) + 8
    rng = np.random.default_rng(np.random.SeedSequence([seed, 12]))
    perm = rng.permutation(NP).astype(np.int32)
    bt = np.full((B, int(need.max())), -1, dtype=np.int32)
    live = np.arange(bt.shape[1])[None, :] < need[:, None]
    bt[live] = perm[:int(need.sum())]
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(rng.integers(1 << 62)))

    def values(shape, as_codes=False):
        """N(0, 1) values as bf16, or as e4m3fn codes of scale about 5 / 448."""
        out = torch.empty(shape, dtype=torch.uint8 if as_codes else torch.bfloat16, device=dev)
        per = max(1, (1 << 26) // max(1, math.prod(shape[1:])))
        for i in range(0, shape[0], per):
            part = torch.randn((min(per, shape[0] - i),) + tuple(shape[1:]), generator=gen, device=dev)
            if as_codes:
                out[i:i + per] = (part * (FP8_MAX / 5)).clamp_(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn).view(torch.uint8)
            else:
                out[i:i + per] = part.to(torch.bfloat16)
        return out

    x = 16 if fp8 else 8
    T = int(new.sum())
    row_codes = fp8 and case.get("rows", "pool") == "pool"
    s = {"case": dict(case), "scale": float(np.float32(1.0 / math.sqrt(D))),
         "k_pages": values((NP, H_kv, D // x, PAGE, x), fp8), "v_pages": values((NP, H_kv, D, PAGE), fp8),
         "q": values((T, H_q, D)), "k_new": values((T, H_kv, D), row_codes), "v_new": values((T, H_kv, D), row_codes),
         "block_table": torch.from_numpy(bt).to(dev),
         "lens0": torch.from_numpy(cached.astype(np.int32)).to(dev),
         "q_start": torch.from_numpy(np.concatenate([[0], np.cumsum(new)]).astype(np.int32)).to(dev),
         "k_scale": None, "v_scale": None}
    s["seq_lens"] = s["lens0"].clone()
    s["out"] = torch.empty((T, H_q, D), dtype=torch.bfloat16, device=dev)
    if fp8:
        for n in ("k_scale", "v_scale"):
            s[n] = (torch.rand((B, H_kv), generator=gen, device=dev) * 0.4 + 0.8) * (5 / FP8_MAX)
    return s


def _call(s):
    # every layer of a model steps from the scheduler's lengths
    s["seq_lens"].copy_(s["lens0"])
    if s["case"]["kind"] == "decode":
        quant = s["case"]["rows"] == "bf16"
        bl.kv_append(s["k_new"], s["v_new"], s["k_pages"], s["v_pages"], s["block_table"], s["seq_lens"],
                     k_scale=s["k_scale"] if quant else None, v_scale=s["v_scale"] if quant else None)
        bl.decode_attention(s["q"], s["k_pages"], s["v_pages"], s["block_table"], s["seq_lens"], s["scale"],
                            s["out"], k_scale=s["k_scale"], v_scale=s["v_scale"])
    else:
        bl.kv_write(s["k_new"], s["v_new"], s["k_pages"], s["v_pages"], s["block_table"], s["seq_lens"], s["q_start"])
        bl.prefill_attention(s["q"], s["k_pages"], s["v_pages"], s["block_table"], s["seq_lens"], s["q_start"],
                             s["scale"], s["out"], k_scale=s["k_scale"], v_scale=s["v_scale"])


def prepare(case, seed):
    s = _inputs(case, seed)
    s["graph"] = None
    if case.get("graph"):
        _call(s)                        # the workspace grows outside the capture
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _call(s)
    return s


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _call(state)
    return {n: state[n] for n in ("out", "seq_lens", "k_pages", "v_pages")}


def tolerance(case):
    """Against the binary64 result the output shows 1.6e-3 to 1.8e-3: nearly
    all of it the rounding of the output itself to bf16, over fp8 pools too.
    The pools and lengths are copies: they agree exactly."""
    return {"rel": 7e-3}


# ------------------------------------------------------------------- exact --

def exact(case, seed):
    """Attention in binary64 over each request's rows, gathered from its
    pages; nothing for the pools and lengths."""
    s = _inputs(case, seed)
    cached, new = _lengths(case)
    H_q, H_kv, D, G = case["H_q"], case["H_kv"], case["D"], case["H_q"] // case["H_kv"]
    fp8 = case["kv"] == "fp8"

    def dense(pool, pages, is_k):       # [H_kv, tokens, D] in binary64
        t = pool.index_select(0, pages)
        t = (t.view(torch.float8_e4m3fn) if fp8 else t).float().double()
        if is_k:                        # [pages, H_kv, D/x, 16, x]
            return t.permute(1, 0, 3, 2, 4).reshape(H_kv, -1, D)
        return t.permute(1, 0, 3, 2).reshape(H_kv, -1, D)

    def new_rows(rows, scale):          # the rows as the pool holds them, scales aside
        if not fp8:
            return rows.double()
        if rows.dtype == torch.uint8:
            return rows.view(torch.float8_e4m3fn).float().double()
        y = (rows.float() / scale[None, :, None]).clamp(-FP8_MAX, FP8_MAX)
        return y.to(torch.float8_e4m3fn).float().double()

    out = torch.empty((int(new.sum()), H_q, D), dtype=torch.float64, device="cuda")
    t0 = 0
    for b in range(case["B"]):
        c, n = int(cached[b]), int(new[b])
        pages = s["block_table"][b, :(c + n + PAGE - 1) // PAGE].long()
        ks = s["k_scale"][b] if fp8 else None
        vs = s["v_scale"][b] if fp8 else None
        k, v = dense(s["k_pages"], pages, True)[:, :c + n], dense(s["v_pages"], pages, False)[:, :c + n]
        k[:, c:] = new_rows(s["k_new"][t0:t0 + n], ks).transpose(0, 1)
        v[:, c:] = new_rows(s["v_new"][t0:t0 + n], vs).transpose(0, 1)
        if fp8:
            k, v = k * ks.double()[:, None, None], v * vs.double()[:, None, None]
        pos = torch.arange(c, c + n, device="cuda")
        hidden = torch.arange(c + n, device="cuda")[None, :] > pos[:, None]
        for g in range(H_kv):
            if n == 1:                  # all query heads of the group at once
                q = s["q"][t0, g * G:(g + 1) * G].double()
                out[t0, g * G:(g + 1) * G] = torch.softmax(q @ k[g].T * s["scale"], dim=-1) @ v[g]
                continue
            for h in range(g * G, (g + 1) * G):
                w = s["q"][t0:t0 + n, h].double() @ k[g].T
                w.mul_(s["scale"]).masked_fill_(hidden, -math.inf)
                out[t0:t0 + n, h] = torch.softmax(w, dim=-1) @ v[g]
        t0 += n
    return {"out": out, "seq_lens": None, "k_pages": None, "v_pages": None}
