"""What the library's speed is measured on: one pass of each device entry point over the steps a serving
engine hands it, from a handful of short requests to the largest steps of the synthetic configurations.

A case is a dict of plain values:
  entry            which public calls a pass makes (see `run`)
  hq, hkv, d       q-heads, kv-heads, head dimension (page size is always 16)
  decodes, ctx_lo, ctx_hi, log
                   that many decode requests, contexts spread over [ctx_lo, ctx_hi], evenly over the
                   logarithm if `log`
  prompts          prompt chunks as "chunk+prior" tokens, comma separated
  per_task         additionally this many requests for each of six short-prompt tasks (prompt lengths
                   N(mean, std)), half of them prefilling the whole prompt, half decoding
  lengths          the seed the lengths are drawn with (they belong to the case, values to `prepare`'s seed)

All values are N(0, 1) rounded to bf16; page ids are a random permutation of a pool a quarter larger than
needed.  Pages and slots that no request owns hold stale data of the same kind, as in a running engine.
"""
from __future__ import annotations

import functools
import math
import random

import numpy as np
import torch

from paper_2508_15919_amd import binding as hb

PAGE = 16
# (mean, std) of the prompt length and mean output length of the six tasks
TASKS = ((32.6, 10.3, 38.9), (44.4, 6.6, 96.0), (121.8, 35.0, 13.6),
         (643.2, 337.0, 27.8), (51.4, 15.8, 90.1), (259.2, 324.9, 207.8))
# head layouts (q-heads, kv-heads, head dimension) of the drawn cases: grouped-query layers whole and as one
# tensor-parallel share, one kv-head per q-head, 64-wide heads
LAYOUTS = ((32, 8, 128), (32, 8, 128), (8, 1, 128), (8, 2, 128), (8, 8, 128), (24, 8, 128), (32, 8, 64), (32, 4, 64))


def _case(entry, hq, hkv, d, decodes=0, ctx_lo=0, ctx_hi=0, log=False, prompts="", per_task=0, lengths=0, name=None):
    c = dict(entry=entry, hq=hq, hkv=hkv, d=d, decodes=decodes, ctx_lo=ctx_lo, ctx_hi=ctx_hi, log=log,
             prompts=prompts, per_task=per_task, lengths=lengths)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest step there is: plan, append, attend; launches and host latency are all that counts
        _case("step", 4, 2, 64, 3, 37, 129, prompts="32+0", name="tiny_step"),
        # one layer of a lightly loaded instance: a few decodes, latency again
        _case("attention", 32, 8, 128, 4, 100, 2000, log=True, lengths=1, name="decode_few"),
        # one layer of an ordinary mixed step: heavy-tailed decode contexts, a first and a later prompt chunk
        _case("attention", 32, 8, 128, 64, 100, 8192, log=True, prompts="512+0,512+1536", lengths=2, name="mixed"),
        # one layer of a large decode batch: bound by HBM
        _case("attention", 32, 8, 128, 256, 2048, 16384, lengths=3, name="decode_heavy"),
        # one layer of a step that carries long prompt chunks on grown contexts: bound by the matrix cores
        _case("attention", 32, 8, 128, 32, 1792, 2304, prompts="2048+0,2048+4096,2048+8192,2048+12288", lengths=4,
              name="prefill_heavy"),
        # one tensor-parallel share of a large layer at long contexts: a single kv-head for 8 q-heads
        _case("attention", 8, 1, 128, 16, 32768, 131072, prompts="4096+61440", lengths=5, name="long_context"),
        # a whole step of hundreds of short prompts and decodes: planning, appending, many short items
        _case("step", 32, 8, 128, per_task=64, lengths=6, name="short_prompts_step"),
        # the prefill of a single odd-sized prompt
        _case("attention", 32, 8, 128, prompts="777+0", lengths=7, name="one_prompt"),
        # 64-wide heads, odd lengths of both kinds
        _case("attention", 32, 8, 64, 48, 150, 6000, log=True, prompts="301+0,1029+700,130+63", lengths=8, name="mixed_d64"),
        # the new keys and values of a step with long chunks go into their pages
        _case("append", 32, 8, 128, 32, 1792, 2304, prompts="2048+0,2048+4096,2048+8192,2048+12285", lengths=4,
              name="append_chunks"),
        # prefilled requests are handed from one instance's pool to another's
        _case("copy", 32, 8, 128, 0, prompts="2048+0,2048+4096,2048+8192,2048+12285", lengths=4, name="copy_pages"),
        # one request's cache leaves the pool in token order
        _case("gather", 32, 8, 128, 1, 12345, 12345, lengths=9, name="gather_request"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    hq, hkv, d = rng.choice(LAYOUTS)
    entry = rng.choice(("attention",) * 6 + ("step", "step", "append", "copy", "gather"))
    seed = rng.randrange(1 << 30)
    if entry == "gather":
        n = _log_int(rng, 100, 40000)
        return _case(entry, hq, hkv, d, 1, n, n, lengths=seed)
    kind = rng.choice(("decode", "prefill", "mixed", "mixed", "short"))
    if entry in ("append", "copy") and kind == "decode":
        kind = "mixed"
    if kind == "short":
        return _case(entry, hq, hkv, d, per_task=_log_int(rng, 2, 64), lengths=seed)
    decodes = ctx_lo = ctx_hi = 0
    if kind != "prefill":
        decodes = _log_int(rng, 1, 200)
        ctx_hi = _log_int(rng, 40, min(131072, (2300000 if kind == "decode" else 700000) // decodes))
        ctx_lo = _log_int(rng, 20, ctx_hi)
    chunks = []
    if kind != "decode":
        room = 3e11            # multiply-adds of all chunks together: with the decodes, below the largest listed case
        for _ in range(rng.randint(1, 6)):
            q, prior = _log_int(rng, 5, 4096), rng.choice((0, 0, _log_int(rng, 16, 16384), _log_int(rng, 16, 65536)))
            work = 2 * d * hq * (q * prior + q * (q + 1) / 2)
            if work <= room:
                chunks.append(f"{q}+{prior}")
                room -= work
        if not chunks:
            chunks = ["333+100"]
    return _case(entry, hq, hkv, d, decodes, ctx_lo, ctx_hi, rng.random() < 0.5, ",".join(chunks), lengths=seed)


@functools.lru_cache(maxsize=64)
def _lengths_of(decodes, ctx_lo, ctx_hi, log, prompts, per_task, lengths):
    g = np.random.default_rng(lengths)
    kind, q, c = [], [], []
    if decodes:
        if log:
            ctx = np.rint(np.exp(g.uniform(math.log(ctx_lo), math.log(ctx_hi), decodes))).astype(np.int64)
        else:
            ctx = g.integers(ctx_lo, ctx_hi + 1, decodes)
        for n in ctx:
            kind.append(hb.HFX_DECODE); q.append(1); c.append(int(n))
    for item in prompts.split(",") if prompts else ():
        chunk, prior = item.split("+")
        kind.append(hb.HFX_PREFILL); q.append(int(chunk)); c.append(int(chunk) + int(prior))
    for mean, std, out in TASKS if per_task else ():
        lens = np.maximum(4, np.rint(g.normal(mean, std, per_task))).astype(np.int64)
        for i, n in enumerate(lens):
            if i % 2 == 0:
                kind.append(hb.HFX_PREFILL); q.append(int(n)); c.append(int(n))
            else:
                kind.append(hb.HFX_DECODE); q.append(1); c.append(int(n + g.integers(1, max(2, int(out)) + 1)))
    return tuple(np.array(a, np.int32) for a in (kind, q, c))


def _lengths(case):
    """kind, q_len, ctx_len of the step's requests."""
    return _lengths_of(*(case[k] for k in ("decodes", "ctx_lo", "ctx_hi", "log", "prompts", "per_task", "lengths")))


def _normal(gen, *shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)


def _inputs(case, seed):
    """The step's arrays: lengths and block table on the host, values on the GPU."""
    kind, q_len, ctx_len = _lengths(case)
    g = np.random.default_rng([seed, 1])
    n_pages = (ctx_len.astype(np.int64) + PAGE - 1) // PAGE
    indptr = np.zeros(len(kind) + 1, np.int32)
    indptr[1:] = np.cumsum(n_pages)
    need = int(indptr[-1])
    num_pages = max(1, -(-need * 5 // 4))
    pages = g.permutation(num_pages)[:need].astype(np.int32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"case": case, "kind": kind, "q_len": q_len, "ctx_len": ctx_len, "indptr": indptr, "pages": pages,
         "shape": hb.make_shape(case["hq"], case["hkv"], case["d"], num_pages)}
    tokens = int(q_len.sum())
    s["pool"] = _normal(gen, num_pages, case["hkv"], 2, PAGE * case["d"])
    if case["entry"] in ("attention", "step"):
        s["q"] = _normal(gen, tokens, case["hq"], case["d"])
    if case["entry"] in ("append", "step"):
        s["k_new"] = _normal(gen, tokens, case["hkv"], case["d"])
        s["v_new"] = _normal(gen, tokens, case["hkv"], case["d"])
    if case["entry"] == "copy":
        s["dst_pages"] = g.permutation(num_pages)[:need].astype(np.int32)
        s["dst"] = _normal(gen, num_pages, case["hkv"], 2, PAGE * case["d"])
    return s


class _Slot:
    """Staging buffers of one host upload in flight, and the event behind the pass that uses them."""

    def __init__(self, host_bytes, device_bytes):
        self.host = torch.empty(host_bytes, dtype=torch.uint8, pin_memory=True)
        self.device = torch.empty(device_bytes, dtype=torch.uint8, device="cuda")
        self.event = None


def _next_slot(s):
    """The next slot of the ring.  A staging buffer may be written again once the stream has passed the
    pass that uploaded it, so an engine that plans ahead keeps a few of them."""
    slot = s["ring"][s["turn"] % len(s["ring"])]
    s["turn"] += 1
    if slot.event is None:
        slot.event = torch.cuda.Event()
    else:
        slot.event.synchronize()
    return slot


def _build(s, slot, stream):
    hb.hfx_build_batch_desc(s["shape"], s["kind"], s["q_len"], s["ctx_len"], s["indptr"], s["pages"], slot.host,
                            slot.device, stream)


def prepare(case, seed):
    s = _inputs(case, seed)
    stream = torch.cuda.current_stream()
    if case["entry"] == "copy":
        n = 8 * len(s["pages"])
        s["ring"] = [_Slot(n, n) for _ in range(4)]
        s["turn"] = 0
        return s
    host_bytes, device_bytes, ws_bytes = hb.hfx_batch_desc_sizes(s["shape"], s["kind"], s["q_len"], s["ctx_len"])
    if case["entry"] in ("attention", "step"):
        s["workspace"] = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda") if ws_bytes else None
        s["out"] = torch.empty_like(s["q"])
    if case["entry"] == "gather":
        n = int(s["ctx_len"][0])
        s["k_out"] = torch.empty((n, case["hkv"], case["d"]), dtype=torch.bfloat16, device="cuda")
        s["v_out"] = torch.empty_like(s["k_out"])
    if case["entry"] == "step":
        s["ring"] = [_Slot(host_bytes, device_bytes) for _ in range(4)]
        s["turn"] = 0
    else:
        # one descriptor serves every layer of the step
        s["desc"] = _Slot(host_bytes, device_bytes)
        _build(s, s["desc"], stream)
    return s


def run(s):
    entry, stream = s["case"]["entry"], torch.cuda.current_stream()
    if entry == "attention":       # one layer of a step whose descriptor is on the GPU
        hb.hfx_mixed_paged_attention(s["shape"], s["q"], s["pool"], s["desc"].host, s["desc"].device, s["workspace"],
                                     s["out"], stream)
        return s["out"]
    if entry == "step":            # plan and upload the step, then its (first) layer
        slot = _next_slot(s)
        _build(s, slot, stream)
        hb.hfx_append_kv(s["shape"], s["k_new"], s["v_new"], s["pool"], slot.host, slot.device, stream)
        hb.hfx_mixed_paged_attention(s["shape"], s["q"], s["pool"], slot.host, slot.device, s["workspace"], s["out"],
                                     stream)
        slot.event.record(stream)
        return s["out"], s["pool"]
    if entry == "append":
        hb.hfx_append_kv(s["shape"], s["k_new"], s["v_new"], s["pool"], s["desc"].host, s["desc"].device, stream)
        return s["pool"]
    if entry == "copy":
        slot = _next_slot(s)
        hb.hfx_copy_pages(s["shape"], s["pool"], s["dst"], s["shape"].num_pages, s["pages"], s["dst_pages"], slot.host,
                          slot.device, stream)
        slot.event.record(stream)
        return s["dst"]
    hb.hfx_gather_kv(s["shape"], s["pool"], s["desc"].host, s["desc"].device, 0, s["k_out"], s["v_out"], stream)
    return s["k_out"], s["v_out"]


def work(case):
    kind, q, c = (a.astype(np.int64) for a in _lengths(case))
    kv_token = 2 * case["hkv"] * case["d"] * 2            # K and V of one token
    tokens = int(q.sum())
    if case["entry"] == "append":
        return {"bytes": 2 * tokens * kv_token, "flops": 0}
    if case["entry"] == "copy":
        return {"bytes": 2 * int(((c + PAGE - 1) // PAGE).sum()) * PAGE * kv_token, "flops": 0}
    if case["entry"] == "gather":
        return {"bytes": 2 * int(c[0]) * kv_token, "flops": 0}
    pairs = int((q * (c - q) + q * (q + 1) // 2).sum())   # visible (row, key) pairs
    nbytes = int(c.sum()) * kv_token + 2 * tokens * case["hq"] * case["d"] * 2
    if case["entry"] == "step":
        nbytes += 2 * tokens * kv_token
    return {"bytes": nbytes, "flops": 4 * case["d"] * case["hq"] * pairs}


def tolerance(case):
    if case["entry"] in ("append", "copy", "gather"):
        return "exact"
    # Softmax weights and results are rounded to bf16; measured against `exact`: 1.8e-3 to 2.4e-3 in the 2-norm.
    # The first rows of a prompt are of order 1 where rows deep in a context are of order 0.01, so the largest
    # single difference over the rms of all is larger with prompts (up to 0.05) than without (0.014).
    return {"rel": 9e-3, "max": 0.2 if case["prompts"] or case["per_task"] else 0.06}


def _token_major(s, r):
    """Keys and values of request r as [kv-head, token, dimension] in 64 bits."""
    case, n = s["case"], int(s["ctx_len"][r])
    hkv, d = case["hkv"], case["d"]
    ids = torch.from_numpy(s["pages"][s["indptr"][r]:s["indptr"][r + 1]].astype(np.int64)).cuda()
    blocks = s["pool"][ids]                                                   # [pages, hkv, 2, 16 d]
    k = blocks[:, :, 0].reshape(-1, hkv, d // 16, PAGE, 16).permute(1, 0, 3, 2, 4).reshape(hkv, -1, d)[:, :n]
    v = blocks[:, :, 1].reshape(-1, hkv, d, PAGE).permute(1, 0, 3, 2).reshape(hkv, -1, d)[:, :n]
    return k.double(), v.double()


def exact(case, seed):
    if case["entry"] in ("append", "copy", "gather"):
        return None                                                           # bytes are moved, not computed
    s = _inputs(case, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    starts = np.concatenate([[0], np.cumsum(s["q_len"])])
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    for r in range(len(s["kind"])):
        n, q_len, t0 = int(s["ctx_len"][r]), int(s["q_len"][r]), int(starts[r])
        k, v = _token_major(s, r)
        if case["entry"] == "step":       # the chunk's own keys and values are the appended ones
            k[:, n - q_len:] = s["k_new"][t0:t0 + q_len].permute(1, 0, 2).double()
            v[:, n - q_len:] = s["v_new"][t0:t0 + q_len].permute(1, 0, 2).double()
        rows = max(1, (1 << 26) // n)     # chunk rows at a time, so that the scores stay below a few GB
        for a in range(0, q_len, rows):
            b = min(q_len, a + rows)
            m = n - q_len + b             # keys the last of these rows sees
            hidden = torch.arange(m, device="cuda")[None, :] > torch.arange(n - q_len + a, m, device="cuda")[:, None]
            for g in range(hkv):
                qg = s["q"][t0 + a:t0 + b, g * (hq // hkv):(g + 1) * (hq // hkv)].double()
                for h in range(hq // hkv):
                    score = (qg[:, h] @ k[g, :m].T) / math.sqrt(d)
                    if b - a > 1:
                        score.masked_fill_(hidden, -math.inf)
                    out[t0 + a:t0 + b, g * (hq // hkv) + h] = torch.softmax(score, dim=1) @ v[g, :m]
    return (out, None) if case["entry"] == "step" else out
