"""Cases that stand for what a program does with this library, for timing it and comparing its results.

A program fills a quantised KV cache from a prompt (in one call with the key-norm calibration, or chunk by
chunk) and then decodes: one query per sequence attends to the cache, the new token joins it, and what leaves
the recent window is quantised.  `listed()` names twelve such pieces of work, `draw(rng)` gives more of the same
ranges; `prepare` makes the inputs and the cache a program holds before the call, `run` makes the call once.

A decode step moves its cache on by one token.  `run` takes that token back afterwards (the two host counters
of the cache), as a program does with a rejected speculative token: the next pass writes the same slots and rows
again, so a pass can be repeated on the same state.
"""
from __future__ import annotations

import math

import torch

from paper_2602_23200_amd import binding as iq

D = 128
SINK = 4
PAGE = 64
STORE = ("k_codes", "k_scales", "k_zeros", "v_codes", "v_scales", "v_zeros")

# Cost bound of a drawn case, in (sequence, kv head, token) units: the largest listed decode case has 4 x 8 x 131072.
MOST_UNITS = 4 * 8 * 131072
# ... and of a drawn prompt, which costs more per token: the largest listed one has 8 x 8 x 32768.
MOST_PROMPT_UNITS = 8 * 8 * 32768


def _case(name, op, batch, q_heads, kv_heads, tokens, bits, group, recent, **more):
    c = dict(op=op, batch=batch, q_heads=q_heads, kv_heads=kv_heads, tokens=tokens, bits=bits, v_bits=0, group=group,
             recent=recent, k_mode=iq.HYBRID, v_mode=iq.HYBRID, kind=iq.KIND_INNER, keys="normal", norm=False,
             half_out=True, chunk=0, steps=0)
    c.update(more)
    if name is not None:
        c = dict(name=name, **c)
    return c


def listed():
    return [
        # The smallest decode step: one short sequence, 4 query heads on 1 kv head.  Launches and latency count.
        _case("step_512_4bit", "step", 1, 4, 1, 512, 4, 32, 32, keys="outliers"),
        # A chat turn on a multi-head layer (as many kv heads as query heads) at 4 bits, moderate context.
        _case("step_4k_mha_4bit", "step", 1, 32, 32, 4096, 4, 32, 128, keys="outliers"),
        # The headline: a batch of long contexts on a grouped-query layer, 2-bit codes, heavy-tailed key channels.
        _case("step_32k_2bit", "step", 8, 32, 8, 32768, 2, 32, 128, keys="heavy"),
        # A serving batch: many sequences of medium length, wide groups.
        _case("step_8k_batch32_g64", "step", 32, 32, 8, 8192, 2, 64, 128),
        # The longest contexts, with the key-norm factors applied to the query by the call.
        _case("step_128k_key_norm", "step", 4, 32, 8, 131072, 2, 32, 128, keys="heavy", norm=True, half_out=False),
        # The paper's Base preset: 3-bit symmetric keys and values.
        _case("step_32k_base_preset", "step", 8, 32, 8, 32768, 3, 32, 128, k_mode=iq.SYM, v_mode=iq.SYM, keys="heavy"),
        # The paper's Hybrid preset (3-bit symmetric keys, 2-bit hybrid values) with 8 query heads per kv head and an
        # odd length, through the separate attention call (append and attention apart, as in a first integration).
        _case("attend_odd_16k_hybrid_preset", "attend", 4, 64, 8, 16001, 3, 32, 128, v_bits=2, k_mode=iq.SYM,
              keys="heavy", half_out=False),
        # Continuous batching: sequences of 1k to 16k tokens in one batch, token counts on the device, paged store.
        _case("step_ragged_paged", "ragged", 16, 32, 8, 16384, 2, 32, 128, keys="heavy"),
        # The end of a long prefill: calibration of the key factors and quantisation of the whole prompt.
        _case("prefill_32k_2bit", "prefill", 8, 32, 8, 32768, 2, 32, 128, keys="heavy"),
        # Chunked prefill of a 4k prompt, 512 tokens a chunk, keys and values at 4 bits.
        _case("prefill_chunked_4k_4bit", "chunks", 1, 32, 32, 4096, 4, 32, 128, keys="outliers", chunk=512),
        # A whole short conversation from an empty cache: a 100-token prompt, then 64 decode steps; the first ones
        # find no quantised token yet.
        _case("generate_100_plus_64", "generate", 2, 32, 8, 100, 4, 32, 128, steps=64),
        # The layout the method is compared with (groups across the inner dimension), behind the same calls.
        _case("attend_8k_outer", "attend", 8, 32, 8, 8192, 2, 32, 128, kind=iq.KIND_OUTER, keys="heavy"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ranges: any of the operations at a size between the smallest and the largest."""
    op = rng.choice(["step", "step", "step", "step", "attend", "ragged", "prefill", "chunks", "generate"])
    kv_heads = rng.choice([1, 2, 4, 8, 8, 16, 32])
    q_heads = kv_heads * rng.choice([1, 2, 4, 4, 8])
    bits, v_bits, k_mode, v_mode = rng.choice([
        (2, 0, iq.HYBRID, iq.HYBRID), (2, 0, iq.SYM, iq.HYBRID), (2, 0, iq.SYM, iq.SYM), (4, 0, iq.HYBRID, iq.HYBRID),
        (4, 0, iq.SYM, iq.ASYM), (3, 0, iq.SYM, iq.SYM), (3, 2, iq.SYM, iq.HYBRID), (3, 2, iq.SYM, iq.SYM)])
    batch = _log_int(rng, 1, 32)
    most = (MOST_PROMPT_UNITS if op in ("prefill", "chunks") else MOST_UNITS) // (batch * kv_heads)
    tokens = _log_int(rng, 300, max(301, min(131072, most)))
    more = dict(v_bits=v_bits, k_mode=k_mode, v_mode=v_mode, keys=rng.choice(["normal", "outliers", "heavy"]),
                half_out=rng.random() < 0.5)
    if op == "attend" and rng.random() < 0.5:
        bits = rng.choice([2, 4])
        more.update(kind=iq.KIND_OUTER, v_bits=0)
    if op in ("step", "attend"):
        more["norm"] = rng.random() < 0.3
    if op == "chunks":
        more["chunk"] = max(64, rng.randint(tokens // 12, tokens // 3))
    if op == "generate":
        batch, tokens = min(batch, 4), rng.randint(20, 400)
        more["steps"] = rng.randint(24, 64)
    return _case(None, op, batch, q_heads, kv_heads, tokens, bits, rng.choice([32, 32, 64]), rng.choice([32, 64, 128]), **more)


# ------------------------------------------------------------------------------------------------ inputs


def _config(c, capacity, pages=0):
    return iq.make_config(c["batch"], c["q_heads"], c["kv_heads"], D, c["bits"], c["group"], SINK, c["recent"],
                          c["k_mode"], c["v_mode"], 0, c["kind"], capacity, c["v_bits"], 0, pages)


def _lengths(c):
    """Tokens per sequence of a ragged batch: spread evenly over the logarithm from tokens / 16 to tokens."""
    B, n = c["batch"], c["tokens"]
    return [max(SINK + c["recent"] + 2, int(n * 16.0 ** (-(B - 1 - i) / max(1, B - 1)))) for i in range(B)]


class _Inputs:
    """fp16 keys, values and queries from the seed alone: keys are normal draws times a spread per channel."""

    def __init__(self, c, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(1000003 * (seed % (1 << 40)) + 17)
        B, H = c["batch"], c["kv_heads"]
        sigma = torch.ones(H, D, device="cuda")
        if c["keys"] == "outliers":       # one channel in a hundred (at least one a head) eight times larger
            pick = torch.rand(H, D, generator=self.gen, device="cuda")
            sigma = torch.where(pick <= torch.clamp(pick.min(dim=1, keepdim=True).values, min=0.01), 8.0, 1.0)
        elif c["keys"] == "heavy":        # 1 + |Student-t with 3 degrees of freedom|
            z = torch.randn(4, H, D, generator=self.gen, device="cuda")
            sigma = 1.0 + (z[0] / ((z[1] ** 2 + z[2] ** 2 + z[3] ** 2) / 3.0).sqrt()).abs()
        self.sigma = sigma
        n = c["tokens"] + c["steps"]
        self.k = self._rows(B, H, n, sigma[None, :, None, :])
        self.v = self._rows(B, H, n, None)
        self.k_new = self._rows(B, H, 1, sigma[None, :, None, :])
        self.v_new = self._rows(B, H, 1, None)
        shape = (max(1, c["steps"]), B, c["q_heads"], D)
        self.q = torch.randn(shape, generator=self.gen, device="cuda").half()

    def _rows(self, B, H, n, scale):
        out = torch.empty(B, H, n, D, dtype=torch.float16, device="cuda")
        for b in range(B):
            x = torch.randn(1, H, n, D, generator=self.gen, device="cuda")
            out[b:b + 1] = x if scale is None else x.mul_(scale)
        return out


def _one_sequence(cache, b):
    """Sequence b of a paged cache as a cache of its own: its row of the page table, its windows, the shared pool."""
    cfg = iq.innerq_config_t.from_buffer_copy(bytes(cache.cfg))
    B, cfg.batch = cfg.batch, 1
    bufs, c = dict(cache.buffers), iq.innerq_cache_t()
    for name in iq.BUFFER_NAMES:
        t = cache.buffers[name]
        if name not in STORE and t is not None:
            bufs[name] = t.view(B, -1)[b]
        setattr(c, name, None if bufs[name] is None else bufs[name].data_ptr())
    c.page_table = cache.buffers["page_table"][b].data_ptr()
    return iq.Cache(cfg, bufs, c)


def prepare(case, seed):
    c, s = case, {}
    s["op"], s["steps"], s["chunk"], s["n"] = c["op"], c["steps"], c["chunk"], c["tokens"]
    x = _Inputs(c, seed)
    capacity = -(-(c["tokens"] + c["steps"] + 2) // PAGE) * PAGE
    out_type = torch.float16 if c["half_out"] else torch.float32
    s["out"] = torch.empty(x.q.shape if c["op"] == "generate" else x.q.shape[1:], dtype=out_type, device="cuda")
    s["q"] = x.q if c["op"] == "generate" else x.q[0]
    s["q_scale"] = None
    if c["op"] == "ragged":
        lengths = _lengths(c)
        blocks = [-(-(n + 2) // PAGE) for n in lengths]
        pool = sum(blocks) + 8
        ids = torch.randperm(pool, generator=x.gen, device="cuda").to(torch.int32)
        table = torch.zeros(c["batch"], capacity // PAGE, dtype=torch.int32, device="cuda")
        at = 0
        for b, n in enumerate(blocks):
            table[b, :n] = ids[at:at + n]
            at += n
        cache = iq.allocate_cache(_config(c, capacity, pool), page_table=table)
        for b, n in enumerate(lengths):
            one = _one_sequence(cache, b)
            iq.innerq_quantize_append(one, x.k[b:b + 1, :, :n].contiguous(), x.v[b:b + 1, :, :n].contiguous())
            iq.innerq_quantize_ahead(one)
        s["lengths"] = torch.tensor(lengths, dtype=torch.int32, device="cuda")
        s["counts"] = torch.empty_like(s["lengths"])
        s["max_tokens"] = max(lengths) + 1
        s["k_new"], s["v_new"] = x.k_new, x.v_new
    else:
        cache = iq.allocate_cache(_config(c, capacity))
        if c["op"] in ("step", "attend"):
            inv = None
            if c["norm"]:
                # the factors divide the keys on their way in; the new key comes from a folded projection
                s["q_scale"], inv = iq.innerq_calibrate_key_norm(cache.cfg, x.k)
                x.k_new = (x.k_new.float() * inv[None, :, None, :]).half()
            iq.innerq_quantize_append(cache, x.k, x.v, inv)
            if c["op"] == "step":
                iq.innerq_quantize_ahead(cache)
                s["k_new"], s["v_new"] = x.k_new, x.v_new
        elif c["op"] == "prefill":
            s["k"], s["v"] = x.k, x.v
        elif c["op"] == "chunks":
            cut = lambda t: [t[:, :, i:i + c["chunk"]].contiguous() for i in range(0, c["tokens"], c["chunk"])]  # noqa: E731
            s["k"], s["v"] = cut(x.k), cut(x.v)
        else:
            n = c["tokens"]
            s["k"], s["v"] = x.k[:, :, :n].contiguous(), x.v[:, :, :n].contiguous()
            s["k_new"] = [x.k[:, :, n + i:n + i + 1].contiguous() for i in range(c["steps"])]
            s["v_new"] = [x.v[:, :, n + i:n + i + 1].contiguous() for i in range(c["steps"])]
    s["cache"] = cache
    s["ws"] = iq.allocate_workspace(cache.cfg)
    s["buffers"] = {n: t for n, t in cache.buffers.items() if t is not None and n != "page_table"}
    return s


def run(s):
    op, cache = s["op"], s["cache"]
    if op == "step":
        iq.innerq_decode_step(cache, s["k_new"], s["v_new"], s["q"], s["ws"], out=s["out"], q_scale=s["q_scale"])
        cache.c.n_tokens -= 1
        cache.c.store_ahead_tokens -= 1
        return {"out": s["out"], **s["buffers"]}
    if op == "attend":
        iq.innerq_decode_attention(cache, s["q"], s["ws"], out=s["out"], q_scale=s["q_scale"])
        return {"out": s["out"]}
    if op == "ragged":
        s["counts"].copy_(s["lengths"])          # the scheduler's lengths of this step; the call advances them
        iq.innerq_decode_step_ragged(cache, s["counts"], s["max_tokens"], s["k_new"], s["v_new"], s["q"], s["ws"], out=s["out"])
        return {"out": s["out"], "counts": s["counts"], **s["buffers"]}
    cache.c.n_tokens = cache.c.store_ahead_tokens = 0
    if op == "prefill":
        norm, inv = iq.innerq_prefill(cache, s["k"], s["v"])
        return {"norm": norm, "inv_norm": inv, **s["buffers"]}
    if op == "chunks":
        for k, v in zip(s["k"], s["v"]):
            iq.innerq_quantize_append(cache, k, v)
        return dict(s["buffers"])
    iq.innerq_quantize_append(cache, s["k"], s["v"])
    iq.innerq_quantize_ahead(cache)
    for i in range(s["steps"]):
        iq.innerq_decode_step(cache, s["k_new"][i], s["v_new"][i], s["q"][i], s["ws"], out=s["out"][i])
    return {"out": s["out"], **s["buffers"]}


# ------------------------------------------------------------------------------------------------ the least work


def _partition(c, which, n):
    """(sink, quantised, recent) tokens of keys (0) or values (1) when n are cached."""
    mid = max(0, n - SINK - c["recent"])
    if (which == 1) == (c["kind"] == iq.KIND_INNER):        # groups along tokens: whole groups only
        mid -= mid % c["group"]
    return min(n, SINK), mid, n - min(n, SINK) - mid


def _row_bytes(c, which):
    """Bytes of one quantised (token, kv head) of one tensor: codes, scales, zero-points."""
    bits = c["v_bits"] if which == 1 and c["v_bits"] else c["bits"]
    mode = c["k_mode"] if which == 0 else c["v_mode"]
    return D * bits / 8 + D / c["group"] * (2 if mode == iq.SYM else 4)


def _attention_work(c, n, sequences):
    """One query per sequence over n tokens: the cache once, query in, output out."""
    heads, b = c["kv_heads"] * sequences, 0.0
    for w in (0, 1):
        sink, mid, recent = _partition(c, w, n)
        b += heads * (mid * _row_bytes(c, w) + (sink + recent) * D * 2)
    b += sequences * c["q_heads"] * D * (2 + (2 if c["half_out"] else 4))
    return b, 4.0 * sequences * c["q_heads"] * n * D


def _append_work(c, n, sequences):
    """n tokens into the cache: fp16 rows in, packed rows out; about eight operations a value for a group's range,
    code and error, twice where both variants compete."""
    heads, b, f = c["kv_heads"] * sequences, 0.0, 0.0
    for w, mode in ((0, c["k_mode"]), (1, c["v_mode"])):
        b += heads * n * (D * 2 + _row_bytes(c, w))
        f += heads * n * D * (16 if mode == iq.HYBRID else 8)
    return b, f


def work(case):
    c, B, n = case, case["batch"], case["tokens"]
    parts = []
    if c["op"] in ("step", "attend"):
        step = c["op"] == "step"
        parts.append(_attention_work(c, n + step, B))
        if step:
            parts.append(_append_work(c, 1, B))
    elif c["op"] == "ragged":
        parts += [_attention_work(c, m + 1, 1) for m in _lengths(c)] + [_append_work(c, 1, B)]
    elif c["op"] in ("prefill", "chunks"):
        parts.append(_append_work(c, n, B))
    else:
        parts.append(_append_work(c, n, B))
        for i in range(c["steps"]):
            parts += [_attention_work(c, n + i + 1, B), _append_work(c, 1, B)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # Packed codes, scales, zero-points, windows and counts are whole values: the same bits.  A decode output is a
    # weighted mean whose fp16 weights are rounded (relative 2^-12 each, nearly independent); where the weights are
    # flat the mean itself is small against its terms.  Measured against 64 bits over 100 drawn cases: 1e-4 to 1.6e-3
    # in the 2-norm, up to 5.6e-3 of the root mean square in one element, the fp16 outputs' own rounding included.
    if case["op"] in ("prefill", "chunks"):
        return {"rel": 1e-6, "max": 1e-6}       # the fp32 square root and reciprocal of the key factors
    return {"rel": 4e-3, "max": 0.02}


# ------------------------------------------------------------------------------------------------ the reference


def _decoded(groups, bits, mode):
    """The values, in 64 bits, that a cache holds for fp16 groups [G, M] (one group a column): quantised by the
    method's rule with every 32-bit operation rounded on its own, and decoded exactly."""
    x = groups.float()
    top, half = (1 << bits) - 1, 1 << (bits - 1)
    one = torch.ones((), device=x.device)
    low, high, most = x.amin(0), x.amax(0), x.abs().amax(0)

    def scale_of(r, den):
        return (r / torch.full_like(r, float(den))).half()

    sa, ss = scale_of(high - low, top), scale_of(most, half - 1)
    quotient = lambda a, s: torch.where(s == 0, torch.zeros((), device=x.device), a / torch.where(s == 0, one, s))  # noqa: E731
    ca = quotient(x - low, sa.float()).round_().clamp_(0, top)
    cs = quotient(x, ss.float()).round_().clamp_(-half, half - 1)
    if mode == iq.HYBRID:
        ea, es = torch.zeros_like(low), torch.zeros_like(low)
        for i in range(x.shape[0]):                        # summed in index order, multiply and add rounded apart
            ra = sa.float() * ca[i]
            ra = ra + low
            ea = ea + (x[i] - ra).abs()
            rs = ss.float() * cs[i]
            es = es + (x[i] - rs).abs()
        asym = ea < es
    else:
        asym = torch.full_like(low, mode == iq.ASYM, dtype=torch.bool)
    zero = low.half().double()
    return torch.where(asym, sa.double() * ca.double() + zero, ss.double() * cs.double())


def _store_values(c, which, x, rows):
    """64-bit values of store rows 0 .. rows of one (sequence, kv head): x fp16 [tokens, D]."""
    G = c["group"]
    bits = c["v_bits"] if which == 1 and c["v_bits"] else c["bits"]
    mode = c["k_mode"] if which == 0 else c["v_mode"]
    q = x[SINK:SINK + rows]
    if rows == 0:
        return q.double()
    if (which == 1) == (c["kind"] == iq.KIND_INNER):        # G tokens of one channel
        g = q.view(rows // G, G, D).permute(1, 0, 2).reshape(G, -1)
        return _decoded(g, bits, mode).view(G, rows // G, D).permute(1, 0, 2).reshape(rows, D)
    g = q.view(rows, D // G, G).permute(2, 0, 1).reshape(G, -1)
    return _decoded(g, bits, mode).view(G, rows, D // G).permute(1, 2, 0).reshape(rows, D)


def _attended(c, k, v, steps):
    """Attention of one (sequence, kv head): k, v fp16 [tokens, D]; steps: (tokens attended, fp64 queries [r, D])."""
    last = max(n for n, _ in steps)
    ks, vs = (_store_values(c, w, t, _partition(c, w, last)[1]) for w, t in ((0, k), (1, v)))
    out = []
    for n, q in steps:
        kk, vv = k[:n].double(), v[:n].double()
        for w, t, st in ((0, kk, ks), (1, vv, vs)):
            rows = _partition(c, w, n)[1]
            t[SINK:SINK + rows] = st[:rows]
        p = torch.softmax(q @ kk.T / math.sqrt(D), dim=-1)
        out.append(p @ vv)
    return out


def exact(case, seed):
    c, r = case, case["q_heads"] // case["kv_heads"]
    x = _Inputs(c, seed)
    B, H, n = c["batch"], c["kv_heads"], c["tokens"]
    if c["op"] == "chunks":
        return None
    if c["op"] == "prefill":
        most = x.k.abs().amax(dim=(0, 1, 2)).double()
        norm = torch.where(most == 0, torch.ones_like(most), most.sqrt())[None].expand(H, D).contiguous()
        return {"norm": norm, "inv_norm": 1.0 / norm}
    k, v, q = x.k, x.v, x.q
    if c["norm"]:
        most = k.abs().amax(dim=(0, 1, 2)).float()
        norm = torch.where(most == 0, torch.ones_like(most), most.sqrt())
        inv = torch.ones_like(norm) / norm
        for b in range(B):
            k[b] = (k[b].float() * inv).half()
        x.k_new = (x.k_new.float() * inv).half()
        q = (q.float() * norm).half()
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lengths = _lengths(c) if c["op"] == "ragged" else [n] * B
    for b in range(B):
        for h in range(H):
            kb, vb = k[b, h], v[b, h]
            if c["op"] in ("step", "ragged"):
                kb = torch.cat([kb[:lengths[b]], x.k_new[b, h]])
                vb = torch.cat([vb[:lengths[b]], x.v_new[b, h]])
            if c["op"] == "generate":
                steps = [(n + i + 1, q[i, b, h * r:(h + 1) * r].double()) for i in range(c["steps"])]
            else:
                steps = [(kb.shape[0], q[0, b, h * r:(h + 1) * r].double())]
            for i, o in enumerate(_attended(c, kb, vb, steps)):
                out[i, b, h * r:(h + 1) * r] = o
    return {"out": out if c["op"] == "generate" else out[0]}
