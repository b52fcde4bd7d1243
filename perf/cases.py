"""The work a user of this package has it do, as cases that can be timed and compared.

A case is a dict of plain values.  `listed()` names the standing ones, `draw(rng)` gives one more of the same
ranges, `prepare` / `run` make and run one pass through the package's calls, `work` says what a pass cannot do
without, `exact` gives the result in 64 bits from plain torch, `tolerance` how far a correct implementation may be
from another.

Fields: kind ("step" = cast + append of the current token and attention in one call, "attend" = attention alone,
"multi" = several query tokens per sequence, "rotate" = keys cached before the rotary embedding and rotated at read,
"cast" = bulk cast into the cache, "read" = cached rows back to numbers), batch, q_heads, kv_heads, tokens (of the
longest sequence), ragged (lengths spread log-uniformly below that), dtype, block, bits (mantissa bits of the
cache), page (tokens per page, 0 = one region per sequence), q_bits (query cast to that many bits, 0 = as it is),
q_tokens, perm (channel permutations applied at run time; otherwise the weights carry them).
"""
import math
import random

import numpy as np
import torch

from paper_2403_20137_amd import kvbfp

D = 128
DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
ELT = {"bf16": 2, "f16": 2, "f32": 4}
SCALE = float(np.float32(D ** -0.5))
K_ROWS, V_ROWS, QUERY, K_NEW, V_NEW, GAINS, ORDER, LENGTHS, PAGES = range(9)
BASE = {"kind": "step", "batch": 1, "q_heads": 32, "kv_heads": 8, "tokens": 1024, "ragged": False, "dtype": "bf16",
        "block": 32, "bits": 4, "page": 0, "q_bits": 0, "q_tokens": 1, "perm": True}
# the dearest pass in either measure: bytes of attend_8bit_8k, operations of chunk_64
MOST_BYTES = 1.1e9
MOST_FLOPS = 4.0e10


def listed():
    cases = [
        # one user's chat, a short context: a decode step is launches and latency
        dict(name="step_900", tokens=900),
        # one user on the 7B shape (one query head per kv-head, fp16), context full
        dict(name="step_7b_4k", tokens=4096, kv_heads=32, dtype="f16"),
        # the 32k-context configuration the package is quoted on, one decode step of a layer
        dict(name="step_32k", batch=8, tokens=32769),
        # a serving engine's step: sequences of every length in a pool of 16-token pages
        dict(name="step_paged_ragged", batch=48, tokens=16384, ragged=True, page=16),
        # the batched 8k configuration with 8-bit mantissas: the largest cache
        dict(name="attend_8bit_8k", kind="attend", batch=16, kv_heads=32, tokens=8192, block=16, bits=8),
        # one very long context
        dict(name="attend_128k", kind="attend", tokens=131072, block=16),
        # speculative decoding: the current token and four drafted ones verified at once
        dict(name="verify_5", kind="multi", batch=8, tokens=12000, q_tokens=5),
        # a chunk of a prompt attends to what is cached of it
        dict(name="chunk_64", kind="multi", batch=4, tokens=8192, q_tokens=64),
        # fp32 activations
        dict(name="attend_f32", kind="attend", batch=4, tokens=8192, dtype="f32", block=16),
        # keys cached before the rotary embedding
        dict(name="rotate_16k", kind="rotate", batch=8, tokens=16384),
        # a prompt's rows cast into 32 layers' caches at once, reordered on the way
        dict(name="cast_prefill", kind="cast", batch=32, tokens=4096, block=16),
        # those caches' keys read back, for another store or a check
        dict(name="read_back", kind="read", batch=32, tokens=4096, block=16),
    ]
    return [dict(BASE, **c) for c in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = dict(BASE)
    c["kind"] = rng.choice(["step", "step", "step", "attend", "attend", "multi", "multi", "rotate", "cast", "read"])
    # one query head per kv-head, groups of four and eight, and the share of one GPU of four or eight
    c["q_heads"], c["kv_heads"] = rng.choice([(32, 32), (32, 8), (32, 8), (64, 8), (8, 2), (8, 1)])
    c["dtype"] = rng.choice(["bf16", "bf16", "f16"])
    c["block"] = rng.choice([16, 32, 32, 64, 128])
    c["bits"] = rng.choice([4, 4, 8])
    c["perm"] = rng.random() < 0.7
    if c["kind"] in ("attend", "rotate", "cast", "read") and rng.random() < 0.2:
        c["dtype"] = "f32"
    if c["kind"] in ("step", "attend", "multi"):
        c["page"] = rng.choice([0, 0, 16, 64, 256])
        c["ragged"] = rng.random() < 0.5
        c["q_bits"] = rng.choice([0, 0, 0, 8])
    if c["kind"] == "multi":
        c["q_tokens"] = _log_int(rng, 2, 64)
    c["tokens"] = _log_int(rng, 64, 131072 if c["kind"] in ("step", "attend", "rotate") else 32768)
    c["batch"] = 1
    most = 1
    while most < 128 and _fits(dict(c, batch=most + 1)):
        most += 1
    c["batch"] = min(most, _log_int(rng, 1, 128))
    while c["tokens"] > 64 and not _fits(c):
        c["tokens"] = c["tokens"] * 3 // 4
    return c


def _fits(c):
    w = work(dict(c, ragged=False))
    return w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS


# ---- inputs, from the seed alone -----------------------------------------------------------------------

def _gen(seed, *ids):
    g = torch.Generator(device="cuda")
    s = int(seed)
    for i in ids:
        s = (s * 1000003 + int(i) * 7919 + 12345) % (2 ** 62)
    g.manual_seed(s)
    return g


def _lengths(c, seed):
    """Cached tokens of every sequence after the call (the longest one has all of them): ragged ones are spread
    log-uniformly, the same lengths for every seed in another order."""
    if not c["ragged"]:
        return [c["tokens"]] * c["batch"]
    lo = max(c["q_tokens"], 64)
    got = [int(lo * (c["tokens"] / lo) ** ((b + 1) / c["batch"])) for b in range(c["batch"])]
    got[-1] = c["tokens"]
    random.Random(int(seed) * 31 + LENGTHS).shuffle(got)
    return got


def _gains(c, seed, which):
    """fp32 [kv_heads][D]: 1, and 10 to 50 in the two to six outlier channels of each head."""
    rng = np.random.default_rng([int(seed), GAINS, which])
    g = np.ones((c["kv_heads"], D), np.float32)
    for h in range(c["kv_heads"]):
        ch = rng.permutation(D)[:rng.integers(2, 7)]
        g[h, ch] = np.exp(rng.uniform(math.log(10), math.log(50), len(ch)))
    return g


def _order(c, seed, which):
    """int32 [kv_heads][D]: channels by their gain, as a calibration orders them."""
    if not c["perm"]:
        return None
    rng = np.random.default_rng([int(seed), ORDER, which])
    near = _gains(c, seed, which) * rng.uniform(0.9, 1.1, (c["kv_heads"], D))
    return np.argsort(near, axis=1, kind="stable").astype(np.int32)


def _rows(c, seed, which, b, n, gains):
    """[n][kv_heads][D] rows of sequence b, n of them, in the case's type."""
    x = torch.randn((n, c["kv_heads"], D), generator=_gen(seed, which, b), device="cuda", dtype=DTYPES[c["dtype"]])
    return x.mul_(gains)


def _all_rows(c, seed, which, gains, counts, room):
    x = torch.zeros((c["batch"], room, c["kv_heads"], D), device="cuda", dtype=DTYPES[c["dtype"]])
    for b, n in enumerate(counts):
        x[b, :n] = _rows(c, seed, which, b, n, gains)
    return x


def _gain_tensors(c, seed):
    return [torch.as_tensor(_gains(c, seed, w), device="cuda").to(DTYPES[c["dtype"]]) for w in (0, 1)]


def _query(c, seed):
    shape = (c["batch"], c["q_tokens"], c["q_heads"], D) if c["kind"] == "multi" else (c["batch"], c["q_heads"], D)
    return torch.randn(shape, generator=_gen(seed, QUERY), device="cuda").to(DTYPES[c["dtype"]])


def _theta():
    return (10000.0 ** (-np.arange(0, D, 2, dtype=np.float64) / D)).astype(np.float32)


def prepare(case, seed):
    c = dict(BASE, **case)
    lens, room = _lengths(c, seed), c["tokens"]
    before = [n - 1 for n in lens] if c["kind"] == "step" else lens
    gk, gv = _gain_tensors(c, seed)
    pk, pv = _order(c, seed, 0), _order(c, seed, 1)
    s = {"c": c, "perm_k": None if pk is None else torch.as_tensor(pk, device="cuda"),
         "perm_v": None if pv is None else torch.as_tensor(pv, device="cuda")}
    perms = {"perm_k": s["perm_k"], "perm_v": s["perm_v"]}
    if c["page"]:
        need = [-(-n // c["page"]) for n in lens]
        order = np.random.default_rng([int(seed), PAGES]).permutation(sum(need)).astype(np.int32)
        table = np.zeros((c["batch"], max(need)), np.int32)
        for b, n in enumerate(need):
            table[b, :n] = order[sum(need[:b]):sum(need[:b]) + n]
        s["table"] = torch.as_tensor(table, device="cuda")
        layout = kvbfp.make_layout(D, c["block"], c["bits"], c["kv_heads"], sum(need), c["page"])
        s["cache"] = kvbfp.alloc_cache(layout, "cuda", fill=0)
        for b, n in enumerate(before):
            if n:
                kvbfp.quantize_append_paged(s["cache"], s["table"][b:b + 1], _rows(c, seed, K_ROWS, b, n, gk)[None],
                                            _rows(c, seed, V_ROWS, b, n, gv)[None], **perms)
    else:
        layout = kvbfp.make_layout(D, c["block"], c["bits"], c["kv_heads"], c["batch"], room)
        s["cache"] = kvbfp.alloc_cache(layout, "cuda", fill=0)
        k, v = (_all_rows(c, seed, w, g, before, room) for w, g in ((K_ROWS, gk), (V_ROWS, gv)))
        if c["kind"] == "cast":
            s["k"], s["v"] = k, v
            return s
        kvbfp.quantize_append(s["cache"], k, v, **perms)
    if c["kind"] == "read":
        s["out"] = torch.empty((c["batch"], room, c["kv_heads"], D), dtype=DTYPES[c["dtype"]], device="cuda")
        return s
    s["q"] = _query(c, seed)
    s["out"] = torch.empty_like(s["q"])
    s["lens"] = torch.as_tensor(np.asarray(lens, np.int32), device="cuda")
    heads = c["q_heads"] * c["q_tokens"]
    if c["page"]:
        size = kvbfp.decode_workspace_bytes_paged(layout, s["table"].shape[1], c["batch"], heads, room)
    else:
        size = kvbfp.decode_workspace_bytes(layout, heads, room)
    s["workspace"] = torch.empty((size,), dtype=torch.uint8, device="cuda")
    if c["kind"] == "step":
        s["k"] = torch.stack([_rows(c, seed, K_NEW, b, 1, gk) for b in range(c["batch"])])
        s["v"] = torch.stack([_rows(c, seed, V_NEW, b, 1, gv) for b in range(c["batch"])])
    if c["kind"] == "rotate":
        order = pk if pk is not None else np.tile(np.arange(D, dtype=np.int32), (c["kv_heads"], 1))
        s["rope"] = [torch.as_tensor(x, device="cuda") for x in kvbfp.permute_rope(_theta(), order, kvbfp.ROPE_PAIRS_HALF_SPLIT)]
    return s


def run(state):
    s, c = state, state["c"]
    kind, cache = c["kind"], s["cache"]
    if kind == "cast":
        kvbfp.quantize_append(cache, s["k"], s["v"], perm_k=s["perm_k"], perm_v=s["perm_v"])
        return list(cache.planes())
    if kind == "read":
        return kvbfp.dequantize(cache, 0, 0, c["tokens"], perm=s["perm_k"], out=s["out"])
    more = {"seq_len_dev": s["lens"], "perm_k": s["perm_k"], "perm_v": s["perm_v"], "out": s["out"],
            "workspace": s["workspace"]}
    if kind == "rotate":
        return kvbfp.decode_attention_rope(cache, s["q"], c["tokens"], SCALE, *s["rope"], **more)
    where = (cache, s["table"]) if c["page"] else (cache,)
    if kind == "step":
        call = kvbfp.append_decode_attention_paged if c["page"] else kvbfp.append_decode_attention
        out = call(*where, s["k"], s["v"], s["q"], c["tokens"], SCALE, q_mant_bits=c["q_bits"], **more)
        return [out, *cache.planes()]
    if kind == "multi":
        call = kvbfp.decode_attention_multi_paged if c["page"] else kvbfp.decode_attention_multi
        return call(*where, s["q"], c["tokens"], SCALE, q_mant_bits=c["q_bits"], **more)
    if c["page"]:
        return kvbfp.decode_attention_paged(*where, s["q"], c["tokens"], SCALE, q_mant_bits=c["q_bits"], **more)
    if c["q_bits"]:
        return kvbfp.decode_attention_qbfp(cache, s["q"], c["tokens"], SCALE, c["q_bits"], **more)
    return kvbfp.decode_attention(cache, s["q"], c["tokens"], SCALE, **more)


def work(case):
    """Packed rows read (or written) once, dense rows written (or read) once, query and output once; two
    multiply-adds per cached element and query head."""
    c = dict(BASE, **case)
    row = D * c["bits"] // 8 + D // c["block"]
    rows = c["kv_heads"] * sum(_lengths(c, 0))
    if c["kind"] == "cast":
        return {"bytes": 2 * rows * (row + D * ELT[c["dtype"]]), "flops": 4 * rows * D}
    if c["kind"] == "read":
        return {"bytes": rows * (row + D * ELT[c["dtype"]]), "flops": rows * D}
    heads = c["q_heads"] * c["q_tokens"]
    total = 2 * rows * row + 2 * c["batch"] * heads * D * ELT[c["dtype"]]
    if c["kind"] == "step":
        total += 2 * c["batch"] * c["kv_heads"] * (D * ELT[c["dtype"]] + row)
    return {"bytes": total, "flops": 4 * rows * D * (heads // c["kv_heads"])}


# Measured: an output against the 64-bit result is one rounding to its type off (bf16 1.7e-3, fp16 2.1e-4 of its
# norm, fp32 some 1e-7 to 1e-6 of sums); two correct results differ by at most their two roundings.
REL = {"bf16": 7e-3, "f16": 9e-4, "f32": 1e-5}


def tolerance(case):
    c = dict(BASE, **case)
    if c["kind"] in ("cast", "read"):
        return "exact"
    return {"rel": REL[c["dtype"]], "max": 4 * REL[c["dtype"]]}


# ---- the result in 64 bits ------------------------------------------------------------------------------

def _bfp(x, block, bits):
    """x [..][D] after the cast to Block Floating Point and back, in float64: the shared exponent is the finest
    at which the block's largest magnitude still rounds into the symmetric range."""
    f = x.to(torch.float32).reshape(*x.shape[:-1], D // block, block)
    top = f.abs().amax(-1, keepdim=True)
    e = ((top.view(torch.int32) + (1 << (24 - bits))) >> 23).clamp(min=1).to(torch.float64) - 127 - (bits - 2)
    unit = torch.exp2(e)
    return (torch.round(f.to(torch.float64) / unit) * unit).reshape(x.shape)


def _in_order(x, order, h):
    return x if order is None else x[..., torch.as_tensor(order[h].astype(np.int64), device=x.device)]


def exact(case, seed):
    c = dict(BASE, **case)
    if c["kind"] == "cast":
        return None
    lens = _lengths(c, seed)
    gk, gv = _gain_tensors(c, seed)
    pk, pv = _order(c, seed, 0), _order(c, seed, 1)
    group = c["q_heads"] // c["kv_heads"]
    if c["kind"] == "read":
        out = torch.empty((c["batch"], c["tokens"], c["kv_heads"], D), dtype=torch.float64, device="cuda")
        for b, n in enumerate(lens):
            rows = _rows(c, seed, K_ROWS, b, n, gk)
            for h in range(c["kv_heads"]):
                got = _bfp(_in_order(rows[:, h], pk, h), c["block"], c["bits"])
                if pk is None:
                    out[b, :, h] = got
                else:
                    out[b, :, h, torch.as_tensor(pk[h].astype(np.int64), device="cuda")] = got
        return out
    q = _query(c, seed)
    q4 = q.reshape(c["batch"], c["q_tokens"], c["q_heads"], D)
    out = torch.zeros(q4.shape, dtype=torch.float64, device="cuda")
    if c["kind"] == "rotate":
        angle = torch.arange(c["tokens"], device="cuda", dtype=torch.float64)[:, None] * \
            torch.as_tensor(_theta().astype(np.float64), device="cuda")
        cos, sin = torch.cos(angle), torch.sin(angle)
    for b, n in enumerate(lens):
        rows = []
        for which, new, g in ((K_ROWS, K_NEW, gk), (V_ROWS, V_NEW, gv)):
            if c["kind"] == "step":
                rows.append(torch.cat([_rows(c, seed, which, b, n - 1, g), _rows(c, seed, new, b, 1, g)]))
            else:
                rows.append(_rows(c, seed, which, b, n, g))
        for h in range(c["kv_heads"]):
            k = _bfp(_in_order(rows[0][:, h], pk, h), c["block"], c["bits"])
            v = _bfp(_in_order(rows[1][:, h], pv, h), c["block"], c["bits"])
            qh = _in_order(q4[b, :, h * group:(h + 1) * group], pk, h)           # [q_tokens][group][D]
            qh = _bfp(qh, c["block"], c["q_bits"]) if c["q_bits"] else qh.to(torch.float64)
            if c["kind"] == "rotate":                                              # back to the original order, pairs (i, i + D/2)
                if pk is not None:
                    back = torch.as_tensor(np.argsort(pk[h]).astype(np.int64), device="cuda")
                    k, qh = k[:, back], qh[..., back]
                x, y = k[:, :D // 2], k[:, D // 2:]
                k = torch.cat([x * cos[:n] - y * sin[:n], y * cos[:n] + x * sin[:n]], 1)
            qh = qh.reshape(-1, D)
            s = torch.mm(qh, k.t().contiguous()) * SCALE                          # [q_tokens * group][n]
            if c["q_tokens"] > 1:
                seen = n - (c["q_tokens"] - 1 - torch.arange(c["q_tokens"], device="cuda"))
                hidden = torch.arange(n, device="cuda")[None] >= seen[:, None]
                s.masked_fill_(hidden.repeat_interleave(group, 0), -math.inf)
            o = torch.mm(torch.softmax(s, 1), v).reshape(c["q_tokens"], group, D)
            if pv is not None:
                o = o[..., torch.as_tensor(np.argsort(pv[h]).astype(np.int64), device="cuda")]
            out[b, :, h * group:(h + 1) * group] = o
    out = out.reshape(q.shape)
    return [out, None, None, None, None] if c["kind"] == "step" else out
