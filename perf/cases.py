"""The calls this framework is used for, as cases to time and to compare.

Five kinds of call, each through the public sessions of
paper_2606_06302_amd.runner (tables, plans and buffers are made once, as a
serving program does at admission; a pass only enqueues):

  decode    one decode step over the ragged cache (tg_decode per layer)
  append    one decode step that also stores the step's new token in the same
            launch (open-ended plans, tg_decode with append_k / append_v);
            the live lengths are first set back to the accepted prefix, as
            after a rejected speculative token, so a pass can be repeated
  prefill   one chunk's attention over its compressed history (tg_prefill)
  compress  one chunk's selection and scatter into its pages (tg_compress)

A case is a dict of plain values.  Its head budgets, per-request ratios and
context lengths come from its "profile" number (the retention structure of
workloads.custom: a share of high heads, the rest low, a narrow per-request
band); tensor values and page placement come from the seed.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2606_06302_amd import tangram as tg
from paper_2606_06302_amd.runner import CompressSession, DecodeSession, PrefillSession, Tables
from workloads import S_CTX, S_K, S_SCORE, S_V, Geometry, custom, device_normal_

PAGE = 16


def listed():
    return [
        # two short requests in fp32: the smallest call, bound by launches and latency (the benchmark's tiny config)
        dict(name="decode-tiny-f32-d64", kind="decode", dtype="f32", L=1, B=2, H=4, gqa=2, d=64, Hp=2,
             ctx_lo=512, ctx_hi=512, frac_hi=0.25, profile=11),
        # one user with a long context at one decode token: few units, each cut into many pieces
        dict(name="decode-one-long-bf16", kind="decode", dtype="bf16", L=2, B=1, H=8, gqa=8, d=128, Hp=2,
             ctx_lo=49152, ctx_hi=49152, frac_hi=0.2, profile=12),
        # an ordinary serving batch, one layer (the benchmark's 32-request, 8192-token decode config)
        dict(name="decode-batch32-bf16", kind="decode", dtype="bf16", L=1, B=32, H=8, gqa=4, d=128, Hp=2,
             ctx_lo=8192, ctx_hi=8192, frac_hi=0.25, profile=13),
        # two layers of the benchmark's largest decode step: 64 requests, lognormal contexts, 8 queries per KV head
        dict(name="decode-batch64-bf16", kind="decode", dtype="bf16", L=2, B=64, H=8, gqa=8, d=128, Hp=2,
             ctx_lo=2048, ctx_hi=65536, frac_hi=0.2, profile=14),
        # head_dim 64, as small models have
        dict(name="decode-batch32-bf16-d64", kind="decode", dtype="bf16", L=2, B=32, H=8, gqa=4, d=64, Hp=2,
             ctx_lo=2048, ctx_hi=16384, frac_hi=0.25, profile=15),
        # fp32 cache (the exact-arithmetic option), ragged contexts
        dict(name="decode-batch16-f32-d128", kind="decode", dtype="f32", L=1, B=16, H=8, gqa=4, d=128, Hp=2,
             ctx_lo=1000, ctx_hi=12000, frac_hi=0.25, profile=16),
        # a served step of several layers with the token appended in the launch: 28 query heads on 4 KV heads
        dict(name="append-batch9-bf16", kind="append", dtype="bf16", L=4, B=9, H=4, gqa=7, d=128, Hp=2,
             ctx_lo=700, ctx_hi=9001, frac_hi=0.2, profile=17),
        # the benchmark's prefill config: 16 requests, a 512-token chunk over the history of 16384 tokens
        dict(name="prefill-batch16-d128", kind="prefill", dtype="bf16", L=1, B=16, H=8, gqa=4, d=128, Hp=2,
             ctx_lo=16384, ctx_hi=16384, C=512, frac_hi=0.25, profile=18),
        # one request being prefilled alone: a chunk of a long prompt
        dict(name="prefill-one-d128", kind="prefill", dtype="bf16", L=1, B=1, H=8, gqa=4, d=128, Hp=2,
             ctx_lo=16384, ctx_hi=16384, C=512, frac_hi=0.25, profile=19),
        # a few requests, odd chunk, odd group size, head_dim 64
        dict(name="prefill-batch5-d64-odd", kind="prefill", dtype="bf16", L=1, B=5, H=8, gqa=5, d=64, Hp=4,
             ctx_lo=900, ctx_hi=7001, C=333, frac_hi=0.25, profile=20),
        # the compression of the benchmark's prefill chunk
        dict(name="compress-512-bf16", kind="compress", dtype="bf16", L=1, B=16, H=8, gqa=4, d=128, Hp=2,
             ctx_lo=16384, ctx_hi=16384, C=512, frac_hi=0.25, profile=18),
        # the longest ordinary chunk
        dict(name="compress-8192-bf16", kind="compress", dtype="bf16", L=1, B=16, H=8, gqa=4, d=128, Hp=2,
             ctx_lo=16384, ctx_hi=16384, C=8192, frac_hi=0.25, profile=22),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges: any of the kinds, the types and head sizes they support, 1 to 64
    requests, contexts of 200 to 49152 tokens and chunks of 16 to 8192, odd values among them."""
    kind = rng.choice(["decode", "decode", "decode", "append", "prefill", "prefill", "compress"])
    H = rng.choice([2, 4, 8, 8])
    case = dict(kind=kind, dtype="bf16", L=1, H=H, d=rng.choice([64, 128]),
                Hp=rng.choice([x for x in (1, 2, 4) if H % x == 0]),
                frac_hi=rng.choice([0.1, 0.2, 0.25, 0.5]), profile=rng.randrange(100, 1 << 20))
    if kind in ("decode", "append"):
        case.update(dtype=rng.choice(["bf16", "bf16", "f32"]), gqa=rng.choice([1, 2, 3, 4, 5, 7, 8, 16]),
                    L=rng.choice([1, 2]), B=_log_int(rng, 1, 64), ctx_lo=_log_int(rng, 200, 8192))
        case["ctx_hi"] = min(49152, _log_int(rng, case["ctx_lo"], 8 * case["ctx_lo"]))
    elif kind == "prefill":
        case.update(gqa=rng.choice([1, 2, 3, 4, 5, 7, 8, 16]), B=_log_int(rng, 1, 16), C=_log_int(rng, 16, 1024),
                    ctx_lo=_log_int(rng, 200, 8192))
        case["ctx_hi"] = min(16384, _log_int(rng, case["ctx_lo"], 4 * case["ctx_lo"]))
    else:
        case.update(dtype=rng.choice(["bf16", "bf16", "f32"]), gqa=4, B=_log_int(rng, 1, 16),
                    C=_log_int(rng, 64, 8192), ctx_lo=_log_int(rng, 200, 8192))
        case["ctx_hi"] = min(16384, _log_int(rng, case["ctx_lo"], 4 * case["ctx_lo"]))
    # no dearer than the largest listed case: fewer requests until the bytes and operations fit
    top = [work(c) for c in listed() if c["kind"] == kind]
    while case["B"] > 1:
        w = work(case)
        if all(w[k] <= max(t[k] for t in top) for k in ("bytes", "flops")):
            break
        case["B"] -= max(1, case["B"] // 8)
    return case


# ------------------------------------------------------------------ lengths
def _workload(case, seed):
    """The case's shapes, budgets and lengths (its profile) with the seed's tensors and page placement."""
    g = Geometry(case["L"], case["H"], case["H"] * case["gqa"], case["d"], PAGE, case["Hp"])
    lo, hi = case["ctx_lo"], case["ctx_hi"]
    z = np.random.default_rng([case["profile"], S_CTX]).standard_normal(case["B"])
    # lognormal contexts around the middle of the range, as request mixes have
    ctx = np.clip(np.round(math.sqrt(lo * hi) * np.exp(0.75 * z)), lo, hi).astype(np.int32)
    wl = custom(case["profile"], g, case["B"], case["dtype"], ctx, frac_hi=case["frac_hi"],
                chunk_len=case.get("C", 0))
    if case["kind"] == "compress":      # the reservation covers the history and the chunk
        wl = dataclasses.replace(wl, ctx_len=(ctx + case["C"]).astype(np.int32))
    return dataclasses.replace(wl, seed=seed), ctx


def _kept(ratio, n):
    return np.ceil(ratio * n).astype(np.int64)


def _lengths(case):
    """Retained entries [B][L][H] (for compress: before the chunk, and after it)."""
    wl, ctx = _workload(case, 0)
    if case["kind"] == "compress":
        return _kept(wl.ratio, ctx[:, None, None]), _kept(wl.ratio, wl.ctx_len[:, None, None])
    return _kept(wl.ratio, ctx[:, None, None])


def work(case):
    esz = 4 if case["dtype"] == "f32" else 2
    B, L, H, d, gqa = case["B"], case["L"], case["H"], case["d"], case["gqa"]
    q = B * H * gqa * d * esz
    if case["kind"] in ("decode", "append"):
        n = int(_lengths(case).sum())
        new = B * L * H * 2 * d * esz * 2 if case["kind"] == "append" else 0   # the token's rows, read and stored
        return {"bytes": n * 2 * d * esz + L * 2 * q + L * B * H * gqa * 4 + new, "flops": n * 4 * d * gqa}
    if case["kind"] == "prefill":
        C = case["C"]
        n = int(_lengths(case)[:, 0].sum())
        keys = n * C + B * H * C * (C + 1) // 2
        return {"bytes": (n * 2 * d + 2 * B * C * H * d) * esz + 2 * C * q, "flops": keys * 4 * d * gqa}
    before, after = _lengths(case)
    kept = int((after - before).sum())
    return {"bytes": kept * 2 * d * esz * 2 + B * H * case["C"] * 4 + kept * 4, "flops": 0}


# ------------------------------------------------------------------ passes
def prepare(case, seed):
    wl, ctx = _workload(case, seed)
    kind = case["kind"]
    if kind == "decode":
        return dict(kind=kind, s=DecodeSession(wl, mode=tg.TG_PLAN_AOT_FILL))
    if kind == "append":
        tables = Tables(wl, headroom=np.full(case["B"], 16, dtype=np.int32))
        s = DecodeSession(wl, tables=tables, mode=tg.TG_PLAN_AOT_FILL, open_end=True)
        shape = (case["L"], case["B"], case["H"], case["d"])
        k = device_normal_(torch.empty(shape, dtype=s.dtype, device="cuda"), wl, S_K, 1.0)
        v = device_normal_(torch.empty(shape, dtype=s.dtype, device="cuda"), wl, S_V, 1.0)
        s.enable_append(k, v, fused=True)
        return dict(kind=kind, s=s, accepted=s.live_len.clone())
    if kind == "prefill":
        return dict(kind=kind, s=PrefillSession(wl))
    tables = Tables(wl)
    elems = case["Hp"] * 2 * PAGE * case["d"]
    pool = torch.zeros(tables.pool_pages * elems, dtype={"f32": torch.float32, "bf16": torch.bfloat16}[case["dtype"]],
                       device="cuda").view(tables.pool_pages, 2, case["Hp"], PAGE, case["d"])
    scores = device_normal_(torch.empty(case["B"], case["H"], case["C"], device="cuda"), wl, S_SCORE, 1.0)
    s = CompressSession(wl, tables, pool, ctx, np.full(case["B"], case["C"], dtype=np.int32), scores=scores)
    return dict(kind=kind, s=s)


def run(state):
    s = state["s"]
    stream = torch.cuda.current_stream()
    if state["kind"] == "decode":
        s.run_step(stream)
        return s.out, s.lse
    if state["kind"] == "append":
        s.live_len.copy_(state["accepted"])
        s.run_decode_step(stream)
        return s.out, s.lse, s.live_len, s.pool
    s.run(stream)
    return s.out if state["kind"] == "prefill" else (s.kept, s.pool)


def tolerance(case):
    if case["kind"] == "compress":
        return "exact"                       # whole rows and indices are moved
    # bf16: the output's own rounding and the rounding of the probabilities (2.3e-3 against 64 bits);
    # f32: fp32 sums in another order (2e-7 against 64 bits, more over the longest contexts)
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 2e-6}


# ------------------------------------------------------------ 64-bit values
def _rows(s, b, layer, h, n):
    """K and V rows [n][d] of the first n entries of head (b, layer, h), in 64 bits."""
    g, t = s.wl.geom, s.t
    base = int(t.pt_offsets[(b * g.num_layers + layer) * g.num_groups + int(t.group_of[layer, h])])
    ids = t.d_pt_pages[base: base + (n + PAGE - 1) // PAGE].long()
    kv = s.pool[ids, :, int(t.slot_of[layer, h])].double()           # [pages][2][P][d]
    return kv[:, 0].reshape(-1, g.head_dim)[:n], kv[:, 1].reshape(-1, g.head_dim)[:n]


def exact(case, seed):
    if case["kind"] == "compress":
        return None                          # bytes and indices: nothing is computed
    state = prepare(case, seed)
    s = state["s"]
    n_of = _lengths(case)
    H, gqa, d = case["H"], case["gqa"], case["d"]
    scale = 1.0 / math.sqrt(d)
    out = torch.zeros(s.out.shape, dtype=torch.float64, device="cuda")
    if case["kind"] == "prefill":
        C = case["C"]
        future = torch.ones(C, C, dtype=torch.bool, device="cuda").triu(1)
        for b in range(case["B"]):
            for h in range(H):
                n = int(n_of[b, 0, h])
                k, v = _rows(s, b, 0, h, n)
                k = torch.cat([k, s.k_new[b, :, h].double()])
                v = torch.cat([v, s.v_new[b, :, h].double()])
                for j in range(h * gqa, (h + 1) * gqa):
                    sc = (s.q[b, :, j].double() @ k.T) * scale
                    sc[:, n:].masked_fill_(future, -math.inf)
                    out[b, :, j] = torch.softmax(sc, dim=1) @ v
        return out
    lse = torch.zeros(s.lse.shape, dtype=torch.float64, device="cuda")
    for l in range(case["L"]):
        for b in range(case["B"]):
            for h in range(H):
                k, v = _rows(s, b, l, h, int(n_of[b, l, h]))
                if case["kind"] == "append":
                    k = torch.cat([k, s.k_tok[l, b, h].double()[None]])
                    v = torch.cat([v, s.v_tok[l, b, h].double()[None]])
                q = slice(h * gqa, (h + 1) * gqa)
                sc = (s.q[l, b, q].double() @ k.T) * scale
                out[l, b, q] = torch.softmax(sc, dim=1) @ v
                lse[l, b, q] = torch.logsumexp(sc, dim=1)
    return (out, lse) if case["kind"] == "decode" else (out, lse, None, None)
