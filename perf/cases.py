"""The library's calls as a serving program makes them, with their inputs, work and tolerances.

A case is one attention layer (or a few layers) of a serving step: the token phase over dense
caches and block pools, the prompt phase, a mixed batch, and the hand-off of a cache from a
prompt machine to a token machine.  Shapes are the workloads of `workloads.py` and of the tests;
context lengths are the quantiles of a workload's length distribution, dealt to the requests in
an order drawn from the seed, so that every seed costs the same.

`listed()` names the cases, `draw()` gives further ones of the same ranges, `prepare()` makes a
case's inputs on the GPU, `run()` is one pass, `exact()` the same result in 64 bits by plain torch.
"""
import math
import random
from statistics import NormalDist

import torch

from paper_2311_18677_amd import binding as sw

DEV = "cuda:0"


# ---- cases --------------------------------------------------------------------------------

def _case(name, kind, n_req, n_qh, n_kvh, head_dim, max_len, lens, lo, hi, **more):
    """lens: "uniform" over [lo, hi], "lognormal" with `median` and `sigma` clipped to [lo, hi],
    or "fixed" (every request hi positions)."""
    c = {"name": name, "kind": kind, "n_req": n_req, "n_qh": n_qh, "n_kvh": n_kvh, "head_dim": head_dim,
         "max_len": max_len, "lens": lens, "lo": lo, "hi": hi, "median": 0.0, "sigma": 0.0,
         "layers": 1, "block": 0, "k_scaled": 0.0, "prompts": 0, "piece": 0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest calls: four short chats on a small multi-head model of two layers; what
        # counts is the launch and the latency
        _case("decode_layers_tiny_mha", "append", 4, 8, 8, 64, 128, "uniform", 1, 127, layers=2),
        # the token machine's inner loop: eight layers of a Llama-2-70B share (8 query heads on one
        # key/value head), batch 64, each layer storing the newest rows and attending over its cache
        _case("decode_layers_llama70b", "append", 64, 8, 1, 128, 4096, "uniform", 1000, 2600, layers=8),
        # the same step on a BLOOM-176B share: multi-head, no sharing of rows between query heads
        _case("decode_bloom176b", "decode", 32, 14, 14, 128, 8192, "lognormal", 16, 8192, median=1000.0, sigma=0.8),
        # a large batch with contexts of very different lengths and some large keys
        _case("decode_skewed_256", "decode", 256, 8, 1, 128, 8192, "lognormal", 16, 8192, median=1020.0, sigma=1.0,
              k_scaled=0.1),
        # few requests over a long context
        _case("decode_longctx_8x32k", "decode", 8, 8, 1, 128, 32768, "fixed", 1, 32768),
        # a token machine that keeps its cache in blocks of 16 positions; 12 heads on 4, odd batch
        _case("decode_paged_16", "paged", 37, 12, 4, 128, 3008, "uniform", 3, 3000, block=16),
        # 64-wide heads with shared keys, the library's other head size
        _case("decode_d64_gqa", "decode", 64, 12, 4, 64, 3000, "uniform", 200, 3000),
        # a prompt machine's usual batch (about 2048 tokens): store the rows, attend
        _case("prompt_2048_batch", "prompt", 2, 8, 1, 128, 2048, "uniform", 72, 1976),
        # one long document
        _case("prompt_8k", "prompt", 1, 8, 1, 128, 8192, "fixed", 1, 8192),
        # the longest prompt, where the quadratic part is all that counts
        _case("prompt_32k", "prompt", 1, 8, 1, 128, 32768, "fixed", 1, 32768),
        # a mixed machine: 63 requests in their token phase and one prompt, cache in blocks
        _case("mixed_paged_llama70b", "mixed", 64, 8, 1, 128, 4096, "uniform", 1000, 2600, block=16,
              prompts=1, piece=1500),
        # a prompt batch's cache handed over: pools to dense, the spans to send, dense to pools
        _case("handoff_32x2k", "handoff", 32, 8, 8, 128, 2048, "uniform", 500, 2048, block=16),
    ]


HEADS = ((1, 1), (2, 1), (4, 2), (6, 2), (8, 1), (8, 8), (12, 4), (14, 14), (16, 1), (5, 5), (7, 1), (32, 8))


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("decode", "decode", "append", "paged", "prompt", "prompt", "mixed", "handoff"))
    n_qh, n_kvh = rng.choice(HEADS)
    head_dim = 128 if kind in ("prompt", "mixed") else rng.choice((64, 128, 128))
    block = rng.choice((4, 16, 32, 128)) if kind in ("paged", "handoff") else 0
    if kind == "mixed":
        block = rng.choice((0, 16, 64))
    if kind == "prompt":
        n_req = _log(rng, 1, 16)
        longest = _log(rng, 32, 32768)
        # no more query-key pairs than the largest listed prompt has
        while n_req * n_qh * longest * longest > 8 * 32768 * 32768:
            longest = max(32, longest * 2 // 3)
        lens, lo = ("fixed", longest) if n_req == 1 else ("uniform", max(1, longest // rng.randint(2, 20)))
        return _drawn(kind, n_req, n_qh, n_kvh, head_dim, longest + rng.randint(0, 64), lens, lo, longest, block=block)
    n_req = _log(rng, 1, 256)
    longest = _log(rng, 64, 32768)
    layers = rng.randint(1, 8) if kind == "append" else 1
    # at most 300 MB of cached rows in a pass, 600 MB with the unused part of the caches
    while layers * n_req * n_kvh * longest * head_dim * 4 > 6e8:
        longest = max(64, longest * 2 // 3)
        n_req = max(1, n_req * 4 // 5)
    max_len = longest + rng.randint(0, 100)
    lens, lo, more = "uniform", rng.randint(1, max(1, longest // 2)), {}
    if kind in ("decode", "append") and longest >= 512 and rng.random() < 0.5:
        lens, lo, more = "lognormal", 16, {"median": longest / 5.0, "sigma": round(rng.uniform(0.4, 1.0), 2)}
    if kind == "mixed":
        more = {"prompts": rng.randint(1, min(2, n_req)), "piece": rng.randint(2, max(2, min(longest, 1500)))}
    if kind == "decode":
        more["k_scaled"] = rng.choice((0.0, 0.0, 0.1))
    return _drawn(kind, n_req, n_qh, n_kvh, head_dim, max_len, lens, lo, longest,
                  layers=layers, block=block, **more)


def _drawn(*a, **more):
    c = _case("", *a, **more)
    del c["name"]
    return c


# ---- a case's lengths ------------------------------------------------------------------------

def _lens(case):
    """The batch's context lengths in rising order (the same for every seed)."""
    n, lo, hi = case["n_req"], case["lo"], case["hi"]
    if case["lens"] == "fixed":
        got = [hi] * n
    elif case["lens"] == "uniform":
        got = [int(lo + (hi - lo) * (i + 0.5) / n + 0.5) for i in range(n)]
    else:
        z = NormalDist()
        got = [int(math.exp(math.log(case["median"]) + case["sigma"] * z.inv_cdf((i + 0.5) / n)) + 0.5) for i in range(n)]
    return [min(hi, max(min(lo, hi), x)) for x in got]


def _queries(case):
    """(length, query tokens) of every request, in the order of _lens.  A mixed batch's prompts
    are pieces of at most `piece` tokens, the others have one query token."""
    lens = _lens(case)
    if case["kind"] == "prompt":
        return [(L, L) for L in lens]
    if case["kind"] == "mixed":
        k = case["prompts"]
        # the prompts have no cached tokens before the piece where it is as long as they are
        return [(max(L, case["piece"]) if i < k else L, min(case["piece"], max(L, case["piece"])) if i < k else 1)
                for i, L in enumerate(lens)]
    return [(L, 1) for L in lens]


def _order(case, seed):
    order = list(range(case["n_req"]))
    random.Random(1000003 * seed + 17).shuffle(order)
    pairs = _queries(case)
    return [pairs[i] for i in order]


# ---- inputs ----------------------------------------------------------------------------------

def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 13)

    def rand(*shape):
        return torch.randn(*shape, generator=gen, dtype=torch.float16, device=DEV)

    c = case
    pairs = _order(c, int(seed))
    lens = [L for L, _ in pairs]
    n_req, n_qh, n_kvh, d, layers = c["n_req"], c["n_qh"], c["n_kvh"], c["head_dim"], c["layers"]
    s = {"case": c, "lens": lens, "nq": [q for _, q in pairs], "stream": torch.cuda.current_stream()}
    # the append form counts the positions cached before the newest token
    s["seq_lens"] = _i32([L - 1 for L in lens] if c["kind"] == "append" else lens)
    bs = c["block"]
    if bs:
        per = [-(-L // bs) for L in lens]
        s["max_blocks"] = -(-c["max_len"] // bs)
        s["n_blocks"] = sum(per) + 3
        lay = sw.sw_kv_paged_layout(s["n_blocks"], n_kvh, d, bs)
        ids = torch.randperm(s["n_blocks"], generator=gen, device=DEV).to(torch.int32)
        table = torch.zeros(n_req, s["max_blocks"], dtype=torch.int32, device=DEV)
        at = 0
        for r, n in enumerate(per):
            if c["kind"] == "handoff":      # a prompt's blocks come mostly in runs
                table[r, :n] = torch.arange(at, at + n, dtype=torch.int32, device=DEV)
            else:
                table[r, :n] = ids[at:at + n]
            at += n
        s["table"] = table
    else:
        lay = sw.sw_kv_layout(n_req, n_kvh, d, c["max_len"])
    s["lay"] = lay
    s["k"] = rand(layers, lay.total_elems)
    s["v"] = rand(layers, lay.total_elems)
    if c["k_scaled"]:
        # a share of the key rows is eight times as large, which stresses the softmax's range
        for layer in s["k"]:
            rows = layer.view(-1, d)
            rows *= 1 + 7 * (torch.rand(rows.shape[0], 1, generator=gen, device=DEV) < c["k_scaled"]).to(torch.float16)
    if c["kind"] in ("decode", "append", "paged"):
        s["q"] = rand(layers, n_req, n_qh, d)
        s["out"] = torch.zeros_like(s["q"])
        if c["kind"] == "append":
            s["k_new"], s["v_new"] = rand(layers, n_req, n_kvh, d), rand(layers, n_req, n_kvh, d)
            s["per_layer"] = list(zip(*(s[x].unbind(0) for x in ("q", "k_new", "v_new", "k", "v", "out"))))
    elif c["kind"] in ("prompt", "mixed"):
        nq = s["nq"]
        starts = [sum(nq[:r]) for r in range(n_req)]
        s["starts"], s["q_starts"], s["q_lens"] = starts, _i32(starts), _i32(nq)
        s["n_tokens"], s["max_q"] = sum(nq), max(nq)
        s["q"] = rand(s["n_tokens"], n_qh, d)
        s["out"] = torch.zeros_like(s["q"])
        s["k_rows"], s["v_rows"] = rand(s["n_tokens"], n_kvh, d), rand(s["n_tokens"], n_kvh, d)
    else:                                   # hand-off: the dense caches in between, the receiver's pools
        dense = sw.sw_kv_layout(n_req, n_kvh, d, c["max_len"])
        s["dense"] = dense
        for name in ("k_dense", "v_dense"):
            s[name] = torch.zeros(dense.total_elems, dtype=torch.float16, device=DEV)
        s["k_there"], s["v_there"] = torch.zeros_like(s["k"][0]), torch.zeros_like(s["v"][0])
        s["span_first"] = torch.zeros(n_req, s["max_blocks"], dtype=torch.int32, device=DEV)
        s["span_blocks"] = torch.zeros_like(s["span_first"])
        s["n_spans"] = torch.zeros(n_req, dtype=torch.int32, device=DEV)
        ids = ids.flip(0).contiguous()      # the receiver's blocks lie scattered
        table = torch.zeros_like(s["table"])
        at = 0
        for r, n in enumerate(per):
            table[r, :n] = ids[at:at + n]
            at += n
        s["table_there"] = table
    # what a pass leaves behind: results, and the caches where it writes them (as bytes)
    if c["kind"] == "handoff":
        s["result"] = [s[x].view(torch.int16) for x in ("k_dense", "v_dense", "k_there", "v_there")]
        s["result"] += [s["n_spans"], s["span_first"], s["span_blocks"]]
    elif c["kind"] in ("append", "prompt", "mixed"):
        s["result"] = [s["out"], s["k"].view(torch.int16), s["v"].view(torch.int16)]
    else:
        s["result"] = [s["out"]]
    return s


# ---- one pass --------------------------------------------------------------------------------

def run(s):
    c, st = s["case"], s["stream"]
    n_req, n_qh, n_kvh, d, L = c["n_req"], c["n_qh"], c["n_kvh"], c["head_dim"], c["max_len"]
    kind = c["kind"]
    if kind == "decode":
        sw.sw_decode_attn(s["q"], s["k"], s["v"], s["seq_lens"], s["out"], n_req, n_qh, n_kvh, d, L, st)
        return s["result"]
    if kind == "append":
        for q, k_new, v_new, k, v, out in s["per_layer"]:
            sw.sw_decode_attn_append(q, k_new, v_new, k, v, s["seq_lens"], out, n_req, n_qh, n_kvh, d, L, st)
        return s["result"]
    if kind == "paged":
        sw.sw_decode_attn_paged(s["q"], s["k"], s["v"], s["table"], s["seq_lens"], s["out"], n_req, n_qh, n_kvh, d,
                                c["block"], s["max_blocks"], s["n_blocks"], st)
        return s["result"]
    if kind == "prompt":
        sw.sw_kv_store(s["k_rows"], s["v_rows"], s["k"], s["v"], s["seq_lens"], s["q_starts"], None, s["n_tokens"],
                       n_req, n_kvh, d, L, L, st)
        sw.sw_prefill_attn(s["q"], s["k"], s["v"], s["seq_lens"], s["q_starts"], s["out"], s["n_tokens"], n_req, n_qh,
                           n_kvh, d, L, st)
        return s["result"]
    if kind == "mixed" and c["block"]:
        geom = (c["block"], s["max_blocks"], s["n_blocks"], s["max_q"], st)
        sw.sw_kv_store_paged(s["k_rows"], s["v_rows"], s["k"], s["v"], s["table"], s["seq_lens"], s["q_starts"],
                             s["q_lens"], s["n_tokens"], n_req, n_kvh, d, *geom)
        sw.sw_mixed_attn_paged(s["q"], s["k"], s["v"], s["table"], s["seq_lens"], s["q_starts"], s["q_lens"], s["out"],
                               s["n_tokens"], n_req, n_qh, n_kvh, d, *geom)
        return s["result"]
    if kind == "mixed":
        sw.sw_kv_store(s["k_rows"], s["v_rows"], s["k"], s["v"], s["seq_lens"], s["q_starts"], s["q_lens"],
                       s["n_tokens"], n_req, n_kvh, d, L, s["max_q"], st)
        sw.sw_mixed_attn(s["q"], s["k"], s["v"], s["seq_lens"], s["q_starts"], s["q_lens"], s["out"], s["n_tokens"],
                         n_req, n_qh, n_kvh, d, L, s["max_q"], st)
        return s["result"]
    geom = (n_req, n_kvh, d, L, c["block"], s["max_blocks"], s["n_blocks"], st)
    sw.sw_kv_pack(s["k"], s["v"], s["table"], s["seq_lens"], s["k_dense"], s["v_dense"], *geom)
    sw.sw_kv_span_plan(s["table"], s["seq_lens"], s["span_first"], s["span_blocks"], s["n_spans"], n_req, c["block"],
                       s["max_blocks"], s["n_blocks"], st)
    sw.sw_kv_unpack(s["k_dense"], s["v_dense"], s["table_there"], s["seq_lens"], s["k_there"], s["v_there"], *geom)
    return s["result"]


# ---- what a pass cannot do without -------------------------------------------------------------

def work(case):
    c = case
    pairs = _queries(c)
    row = c["n_kvh"] * c["head_dim"] * 2
    cached = sum(L for L, _ in pairs)
    new = sum(q for _, q in pairs)
    if c["kind"] == "handoff":
        return {"bytes": 4 * 2 * cached * row, "flops": 0}      # K and V, in and out, packed and unpacked
    seen = sum(q * (L - q) + q * (q + 1) // 2 for L, q in pairs)
    rows = 2 * c["n_qh"] * c["head_dim"] * 2 * new              # queries in, results out
    stored = 2 * 2 * new * row if c["kind"] in ("append", "prompt", "mixed") else 0
    return {"bytes": c["layers"] * (2 * cached * row + rows + stored),
            "flops": c["layers"] * 4 * c["head_dim"] * c["n_qh"] * seen}


def tolerance(case):
    """A result is a weighted mean, rounded once to binary16.  The token phase keeps 32 bits up to
    that rounding: with its sums in another order (other chunks, other kernel) a few values round
    the other way, 1.7e-5 in the 2-norm and 1e-3 of a value at most.  The prompt phase takes its
    weights in binary16, relative to a maximum that depends on the order of the keys: 2.9e-4 in the
    2-norm, 9e-3 of the root mean square at most over the listed and two dozen drawn cases."""
    if case["kind"] == "handoff":
        return "exact"
    if case["kind"] in ("prompt", "mixed"):
        return {"rel": 1.2e-3, "max": 3.5e-2}
    return {"rel": 1e-4, "max": 4e-3}


# ---- the same in 64 bits -----------------------------------------------------------------------

def _attend(q, k, v, first):
    """Causal attention of one request, 64 bits: q [n, n_qh, d] at positions first ..., k and v
    [n_kvh, L, d]."""
    n, n_qh, d = q.shape
    n_kvh = k.shape[0]
    group = n_qh // n_kvh
    out = torch.empty(n, n_qh, d, dtype=torch.float64, device=q.device)
    k, v, q = k.double(), v.double(), q.double() / math.sqrt(d)
    pos = torch.arange(k.shape[1], device=q.device)
    step = max(1, int(2e8) // (k.shape[1] * group))
    for g in range(n_kvh):
        kt = k[g].t().contiguous()
        for i in range(0, n, step):
            qq = q[i:i + step, g * group:(g + 1) * group].reshape(-1, d)
            m = min(step, n - i)
            scores = (qq @ kt).view(m, group, -1)
            late = pos[None, :] > (first + i + torch.arange(m, device=q.device))[:, None]
            scores.masked_fill_(late[:, None, :], -math.inf)
            w = torch.softmax(scores, dim=-1).view(m * group, -1)
            out[i:i + m, g * group:(g + 1) * group] = (w @ v[g]).view(m, group, d)
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "handoff":
        return None
    s = prepare(case, seed)
    n_req, n_kvh, d, lay = c["n_req"], c["n_kvh"], c["head_dim"], s["lay"]
    if c["kind"] in ("prompt", "mixed"):
        q, starts = s["q"], s["starts"]
        out = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    else:
        out = torch.zeros(s["q"].shape, dtype=torch.float64, device=DEV)

    def cached(pool, r, L):
        """[n_kvh, L, d] of request r from a cache or pool"""
        if c["block"]:
            ids = s["table"][r, :-(-L // c["block"])].long()
            blocks = pool.view(s["n_blocks"], n_kvh, c["block"], d)[ids]
            return blocks.transpose(0, 1).reshape(n_kvh, -1, d)[:, :L].clone()
        return pool.as_strided((n_kvh, L, d), (lay.stride_kvh, lay.stride_tok, 1),
                               pool.storage_offset() + r * lay.stride_req).clone()

    for i in range(c["layers"]):
        for r in range(n_req):
            L, nq = s["lens"][r], s["nq"][r]
            k, v = cached(s["k"][i], r, L), cached(s["v"][i], r, L)
            if c["kind"] == "append":
                k[:, L - 1], v[:, L - 1] = s["k_new"][i, r], s["v_new"][i, r]
            if c["kind"] in ("prompt", "mixed"):
                rows = slice(starts[r], starts[r] + nq)
                k[:, L - nq:] = s["k_rows"][rows].transpose(0, 1)
                v[:, L - nq:] = s["v_rows"][rows].transpose(0, 1)
                out[rows] = _attend(q[rows], k, v, L - nq)
            else:
                out[i, r] = _attend(s["q"][i, r][None], k, v, L - 1)[0]
    return [out, None, None] if c["kind"] in ("append", "prompt", "mixed") else [out]
