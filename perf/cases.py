"""The calls a user of this library makes, at the sizes they are made: what is timed when the library is timed.

Three kinds of work, each through the helpers of `paper_2508_15806_amd.api`:

  prefill     one layer's KV compression after a prefill (LayerCall), one prompt or a ragged batch
  recompress  the same selection on a compacted cache that grew during generation (RaggedCall)
  rows, qk    Stage 1, the counting of attention mass over a needle: from attention rows
              (score_heads, score_heads_ex) or from decode queries and context keys (score_heads_qk)

Inputs are synthetic tensors with the shapes and the statistics of the workloads in
`paper_2508_15806_amd.workloads` (N(0,1), a few per cent of the keys pulled towards a window query; decode
rows that are mostly diffuse with a few surface and logic rows), drawn on the GPU from the seed.  The
capacities belong to the case, not to the seed: they come from a model's INF_sc map, which a program
measures once.
"""

import math

import numpy as np
import torch

from paper_2508_15806_amd import api
from paper_2508_15806_amd import binding as B
from paper_2508_15806_amd import workloads as wl

POOLS = {"max": B.SLKV_POOL_MAX, "avg": B.SLKV_POOL_AVG, "none": B.SLKV_POOL_NONE}
ELT_BYTES = {"f32": 4, "bf16": 2, "f16": 2, "bf16_kv8": 1}      # of a key or value element
Q_BYTES = {"f32": 4, "bf16": 2, "f16": 2, "bf16_kv8": 2}        # of a query element
BITS = {4: torch.int32, 2: torch.int16, 1: torch.uint8}
MAP_LAYERS = 32
SPIKE_LAYER = wl.config5_layer_row(wl.config3_inf())            # a layer with a high head: capacities from small to large


def _prefill(name, lens, **kw):
    c = dict(name=name, kind="prefill", lens=lens, dtype="bf16", Hq=32, Hkv=8, d=128, w=64, avg=256, fixed=16,
             layer=SPIKE_LAYER, pool="max", pool_kernel=7, layout="head")
    c.update(kw)
    return c


def _recompress(name, **kw):
    c = dict(name=name, kind="recompress", dtype="bf16", batch=32, Hq=32, Hkv=8, d=128, w=64, avg=256, fixed=16,
             layer=SPIKE_LAYER, new=128, pool="max", pool_kernel=7)
    c.update(kw)
    return c


def listed():
    return [
        # a small model or a unit test: fp32, 1024 tokens; launches and latencies are all there is
        _prefill("fp32_1k", "1024", dtype="f32", Hq=4, Hkv=4, d=64, w=32, avg=128, fixed=32, layer=-1),
        # an ordinary prompt, 8 K tokens, small window (the 8-billion-parameter shape: 32 query / 8 KV heads)
        _prefill("bf16_8k", "8192", w=32, avg=128, fixed=32, layer=-1),
        # the headline: one layer of a 32 K prefill, the capacities of a layer with a high head
        _prefill("bf16_32k", "32768"),
        # the same prompt class with an 8-bit cache
        _prefill("kv8_32k", "32768", dtype="bf16_kv8"),
        # a length of no particular form, half precision, token-major cache, average pooling, large budgets
        _prefill("f16_21k_token_major", "21347", dtype="f16", layout="token", pool="avg", pool_kernel=5, avg=1024),
        # a serving batch of short prompts: more segments than fit one launch's argument table
        _prefill("bf16_batch_short", "611,3020,1777,902,4096,350,2503,1234,5011,777,1600,2048,430,3333,1024,150",
                 w=32, avg=128, fixed=32),
        # a batch of long documents of different lengths
        _prefill("bf16_batch_long", "131072,65536,100000,20000", avg=512, fixed=64),
        # decode of one sequence: its heads are cut back to their capacities once in a while
        _recompress("recompress_one", batch=1, w=32, avg=128, new=64),
        # decode of a batch: all heads of 32 sequences at once, their lengths different
        _recompress("recompress_batch"),
        # Stage 1 over attention rows: all heads of a model, 16 decode steps, 16 K context
        dict(name="rows_16k", kind="rows", L=32, H=32, T=16, n=16384, needle=32, topk=32, ex=False),
        # the same with a prompt length of no particular form, macro-averaged, some layers
        dict(name="rows_ragged_macro", kind="rows", L=8, H=32, T=16, n=13867, needle=27, topk=27, ex=True),
        # Stage 1 from queries and keys, the rows never written
        dict(name="qk_16k", kind="qk", L=32, Hq=32, Hkv=8, T=16, n=16384, d=128, needle=32, topk=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "recompress", "rows", "qk"])
    if kind in ("prefill", "recompress"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "bf16_kv8", "f32"])
        Hq, Hkv = rng.choice([(32, 8), (32, 8), (32, 8), (32, 32), (8, 2), (28, 4)])
        w = rng.choice([16, 32, 64])
        d = rng.choice([128, 128, 64])
        avg = _log_int(rng, 64, 1024)
        c = dict(dtype=dtype, Hq=Hq, Hkv=Hkv, d=d, w=w, avg=avg, fixed=rng.randint(8, avg // 2),
                 layer=rng.choice([SPIKE_LAYER, rng.randrange(MAP_LAYERS)]))
        c["pool"] = rng.choice(["max", "max", "max", "avg", "none"])
        c["pool_kernel"] = 1 if c["pool"] == "none" else rng.choice([3, 5, 7, 7, 13])
    if kind == "prefill":
        # total tokens: up to those of the long listed batch (fp32 and 32 KV heads: as much less as they cost more)
        most = 300000 * 8 // max(Hkv, 8) if dtype != "f32" else 32768 // Hkv
        total = _log_int(rng, 1000, most)
        B_ = 1 if total < 2000 else rng.choice([1, 1, 2, 4, rng.randint(5, 24)])
        if total < 200 * B_:
            B_ = 1
        cuts = [math.exp(rng.uniform(0.0, 2.0)) for _ in range(B_)]
        lens = [max(64, int(total * x / sum(cuts))) for x in cuts]
        lens = [min(x, 140000) for x in lens]
        return dict(c, kind=kind, lens=",".join(map(str, lens)), layout=rng.choice(["head", "head", "token"]))
    if kind == "recompress":
        rows = 64 if dtype != "f32" else 8
        return dict(c, kind=kind, batch=_log_int(rng, 1, max(2, rows * 8 // Hkv)), new=_log_int(rng, 16, 1024))
    if kind == "rows":
        n = _log_int(rng, 512, 40000)
        T = rng.randint(1, 32)
        heads = _log_int(rng, 8, min(1024, (1 << 28) // (n * T)))
        needle = rng.randint(8, 64)
        L = rng.choice([x for x in range(1, 33) if heads // x >= 1])
        return dict(kind=kind, L=L, H=heads // L, T=T, n=n, needle=needle, topk=rng.choice([needle, rng.randint(1, 64)]),
                    ex=rng.random() < 0.4)
    n = _log_int(rng, 512, 40000)
    Hq, Hkv = rng.choice([(32, 8), (32, 8), (8, 2), (28, 4), (32, 32)])
    d = rng.choice([128, 128, 64])
    T = rng.randint(1, 32)
    L = _log_int(rng, 1, max(1, min(32, (1 << 29) // (n * Hkv * d), (1 << 35) // (n * Hq * T * d))))
    needle = rng.randint(8, 64)
    return dict(kind="qk", L=L, Hq=Hq, Hkv=Hkv, T=T, n=n, d=d, needle=needle, topk=rng.choice([needle, rng.randint(1, 64)]))


# ---------------------------------------------------------------- what a case fixes besides the seed

def _capacities(c):
    """This layer's capacities: Algorithm 2 on the model's INF_sc map (32 layers, a few high heads; layer -1: a
    one-layer model with evenly spread scores)."""
    if c["layer"] < 0:
        inf, row = wl.inf_uniform((wl.BASE_SEED, 9), 1, c["Hq"]), 0
    else:
        inf, row = wl.inf_spiky((wl.BASE_SEED + 3, 1000), MAP_LAYERS, c["Hq"]), c["layer"]
    return B.slkv_allocate_budgets(inf, c["Hkv"], c["avg"], c["fixed"])[row]


def _lens(c):
    return [int(x) for x in c["lens"].split(",")]


def _cache_lens(c):
    """Rows per (sequence, KV head) of a cache that has grown since its last compression: what the head's capacity
    kept, and the tokens since, of which a sequence that joined the batch later has fewer."""
    cap = _capacities(c)
    rng = np.random.Generator(np.random.Philox(20250815 + c["batch"]))
    since = rng.integers(max(1, c["new"] // 2), c["new"] + 1, size=c["batch"])
    since[0] = c["new"]
    return [int(max(x, c["w"]) + t) for t in since for x in cap]


def _segments(c):
    """(length, capacity) of every segment."""
    cap = [int(x) for x in _capacities(c)]
    if c["kind"] == "prefill":
        return [(n, x) for n in _lens(c) for x in cap]
    return [(n, cap[i % len(cap)]) for i, n in enumerate(_cache_lens(c))]


# ---------------------------------------------------------------- inputs

def _pull_keys(k_rows, row_seq, row_head, history, qwin, G, gen, frac=0.02, sigma=4.0):
    """2 % of the history keys (rows of k_rows) move towards one random window query of their group."""
    dev = k_rows.device
    pick = (torch.rand(k_rows.shape[0], generator=gen, device=dev) < frac) & history
    rows = pick.nonzero().flatten()
    if rows.numel() == 0:
        return
    hq = row_head[rows] * G + torch.randint(0, G, (rows.numel(),), generator=gen, device=dev)
    qi = torch.randint(0, qwin.shape[2], (rows.numel(),), generator=gen, device=dev)
    q = qwin[row_seq[rows], hq, qi]
    k_rows[rows] += sigma * q / q.norm(dim=1, keepdim=True)


def _cast(x, dtype, cache):
    if dtype == "bf16_kv8" and cache:
        return x.to(torch.float8_e4m3fn).view(torch.uint8)
    return x.to({"f32": torch.float32, "f16": torch.float16}.get(dtype, torch.bfloat16))


def _prepare_prefill(c, gen):
    lens, Hq, Hkv, d, w, dt = _lens(c), c["Hq"], c["Hkv"], c["d"], c["w"], c["dtype"]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    T = int(cu[-1])
    q = torch.randn(len(lens), Hq, w, d, generator=gen, device="cuda")
    k = torch.randn(Hkv, T, d, generator=gen, device="cuda")
    ends = torch.tensor(cu[1:], device="cuda")
    tok = torch.arange(T, device="cuda")
    seq = torch.searchsorted(ends, tok, right=True)
    history = tok < ends[seq] - w
    _pull_keys(k.view(Hkv * T, d), seq.repeat(Hkv), torch.arange(Hkv, device="cuda").repeat_interleave(T),
               history.repeat(Hkv), q, Hq // Hkv, gen)
    k = _cast(k, dt, True)
    v = _cast(torch.randn(Hkv, T, d, generator=gen, device="cuda"), dt, True)
    strides = None
    if c["layout"] == "token":      # a cache that appends tokens: [T][Hkv][d]
        k, v = k.transpose(0, 1).contiguous(), v.transpose(0, 1).contiguous()
        strides = (Hkv * d, d)
    call = api.LayerCall(dt, len(lens), Hq, Hkv, d, w, cu, _capacities(c), c["pool_kernel"], POOLS[c["pool"]],
                         k_strides=strides, v_strides=strides)
    bits = BITS[ELT_BYTES[dt]]
    out = dict(k=call.k_out.view(bits), v=call.v_out.view(bits), kept=call.kept_idx, offsets=call.out_offsets)
    return dict(kind="prefill", call=call, q=_cast(q, dt, False), k=k, v=v, out=out)


def _prepare_recompress(c, gen):
    Hq, Hkv, d, w, dt, n_seq = c["Hq"], c["Hkv"], c["d"], c["w"], c["dtype"], c["batch"]
    lens = _cache_lens(c)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rows = int(offs[-1])
    q = torch.randn(n_seq, Hq, w, d, generator=gen, device="cuda")
    k = torch.randn(rows, d, generator=gen, device="cuda")
    ends = torch.tensor(offs[1:], device="cuda")
    row = torch.arange(rows, device="cuda")
    seg = torch.searchsorted(ends, row, right=True)
    left = ends[seg] - row          # rows from here to the segment's end
    _pull_keys(k, seg // Hkv, seg % Hkv, left > w, q, Hq // Hkv, gen)
    # original positions: the newest w tokens end the sequence, the older ones are spread before them
    pos = torch.where(left > w, (1 << 20) - 8 * left, (1 << 20) - left).to(torch.int32)
    call = api.RaggedCall(dt, n_seq, Hq, Hkv, d, w, offs, _capacities(c), c["pool_kernel"], POOLS[c["pool"]])
    bits = BITS[ELT_BYTES[dt]]
    out = dict(k=call.k_out.view(bits), v=call.v_out.view(bits), kept=call.kept_idx, positions=call.pos_out,
               offsets=call.out_offsets)
    return dict(kind="recompress", call=call, q=_cast(q, dt, False), k=_cast(k, dt, True),
                v=_cast(torch.randn(rows, d, generator=gen, device="cuda"), dt, True), pos=pos, out=out)


def _needle_places(rows, start, needle, n, gen):
    """8 of the needle's tokens and the 16 tokens on either side, for each of `rows` rows."""
    lo, hi = max(0, start - 16), min(n, start + needle + 16)
    r = torch.rand(rows, hi - lo, generator=gen, device="cuda")
    return lo + r.topk(min(8, hi - lo), dim=1).indices


def _prepare_rows(c, gen):
    L, H, T, n, needle = c["L"], c["H"], c["T"], c["n"], c["needle"]
    start = int(torch.randint(0, n - needle + 1, (1,), generator=gen, device="cuda"))
    rows = torch.empty(L, H, T, n, device="cuda")
    step = torch.arange(T, device="cuda").repeat(H)
    for l in range(L):
        z = torch.randn(H * T, n, generator=gen, device="cuda")
        kind = torch.rand(H * T, generator=gen, device="cuda")
        surface = (kind < 0.005).nonzero().flatten()
        z[surface, start + step[surface] % needle] += 12.0
        logic = ((kind >= 0.005) & (kind < 0.02)).nonzero().flatten()
        z[logic.unsqueeze(1), _needle_places(logic.numel(), start, needle, n, gen)] += 6.0
        rows[l] = torch.softmax(z, dim=1).view(H, T, n)
    return dict(kind="rows", ex=c["ex"], rows=rows, start=start, needle=needle, topk=c["topk"])


def _prepare_qk(c, gen):
    L, Hq, Hkv, T, n, d, needle = c["L"], c["Hq"], c["Hkv"], c["T"], c["n"], c["d"], c["needle"]
    G = Hq // Hkv
    start = int(torch.randint(0, n - needle + 1, (1,), generator=gen, device="cuda"))
    k = torch.empty(L, Hkv, n, d, dtype=torch.bfloat16, device="cuda")
    q = torch.randn(L, Hkv, G * T, d, generator=gen, device="cuda")
    step = torch.arange(T, device="cuda").repeat(G).repeat(Hkv)
    head = torch.arange(Hkv, device="cuda").repeat_interleave(G * T)
    for l in range(L):
        kf = torch.randn(Hkv, n, d, generator=gen, device="cuda")
        ql = q[l].view(Hkv * G * T, d)
        kind = torch.rand(Hkv * G * T, generator=gen, device="cuda")
        surface = (kind < 0.005).nonzero().flatten()
        logic = ((kind >= 0.005) & (kind < 0.02)).nonzero().flatten()
        for rows, pull, to in ((surface, 12.0, kf[head[surface], start + step[surface] % needle]),
                               (logic, 6.0, kf[head[logic].unsqueeze(1),
                                               _needle_places(logic.numel(), start, needle, n, gen)].mean(dim=1))):
            ql[rows] += pull * math.sqrt(d) * to / to.square().sum(dim=1, keepdim=True)
        k[l] = kf
    return dict(kind="qk", q=q.view(L, Hq, T, d).to(torch.bfloat16), k=k, start=start, needle=needle, topk=c["topk"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return {"prefill": _prepare_prefill, "recompress": _prepare_recompress, "rows": _prepare_rows,
            "qk": _prepare_qk}[case["kind"]](case, gen)


# ---------------------------------------------------------------- the calls

def run(s):
    if s["kind"] == "prefill":
        s["call"].run(s["q"], s["k"], s["v"])
        return s["out"]
    if s["kind"] == "recompress":
        s["call"].run(s["q"], s["k"], s["v"], s["pos"])
        return s["out"]
    if s["kind"] == "qk":
        return api.score_heads_qk(s["q"], s["k"], s["start"], s["needle"], s["topk"])
    if s["ex"]:
        return api.score_heads_ex(s["rows"], s["start"], s["needle"], s["topk"], aggregation=B.SLKV_AGG_MACRO)
    return api.score_heads(s["rows"], s["start"], s["needle"], s["topk"])


def work(case):
    c = case
    if c["kind"] in ("prefill", "recompress"):
        row = c["d"] * ELT_BYTES[c["dtype"]]
        R = c["Hq"] // c["Hkv"] * c["w"]
        n_bytes = flops = 0
        for n, cap in _segments(c):
            kept = n if n <= c["w"] or n <= cap else max(cap, c["w"])
            ranked = n > c["w"] and n > cap and cap > c["w"]
            # keys of a ranked segment once (the kept ones are among them), kept values, both kept copies, positions
            n_bytes += (n if ranked else kept) * row + kept * (3 * row + 4 + (8 if c["kind"] == "recompress" else 0)) + 8
            if ranked:
                n_bytes += R * c["d"] * Q_BYTES[c["dtype"]]
                flops += 2 * R * c["d"] * (n - c["w"])      # each logit of the window once
        return {"bytes": n_bytes, "flops": flops}
    if c["kind"] == "rows":
        heads, rows = c["L"] * c["H"], c["L"] * c["H"] * c["T"]
        return {"bytes": rows * c["n"] * 4 + heads * (64 if c["ex"] else 40) + heads * 24, "flops": rows * c["n"]}
    rows = c["L"] * c["Hq"] * c["T"]
    return {"bytes": c["L"] * c["Hkv"] * c["n"] * c["d"] * 2 + rows * c["d"] * 2 + c["L"] * c["Hq"] * 64,
            "flops": 2 * rows * c["n"] * c["d"]}


def tolerance(case):
    if case["kind"] == "rows":
        return {"rel": 1e-12}       # fp32 inputs summed in double: the order of the sums is free
    if case["kind"] == "qk":
        return {"rel": 1e-5}        # fp32 logits and weights
    # kept rows are copies, compared bit for bit; two pooled scores closer than fp32 rounding may change places at
    # the capacity of a head, which moves the kept positions between them by one
    return {"rel": 0.0, "differ": 0.005}
