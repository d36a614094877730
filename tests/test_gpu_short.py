"""Decode steps and attention calls of short caches, which one launch serves (attention and append): around its 64-token tiles
and the first packed rows of a tensor, with one, two and four query heads a work-group, in every layout, against the oracle.

Everything is fp32, weights included, so the bound is that of fp32 sums: a score is a sum of 128 products (absolute error
up to 128 x 2^-24 of sum |q k| / sqrt(d), below 1e-5 for these inputs), which moves a weight by as much relative to itself.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import assert_cache_equal, gpu_config, max_rel_err, oracle_config

pytestmark = pytest.mark.gpu
TOL = 5e-5


@pytest.mark.parametrize("kind,bits,group,recent,batch,heads,start,steps", [
    (orc.KIND_INNER, 4, 32, 128, 2, (8, 2), 1, 6), (orc.KIND_INNER, 2, 32, 128, 1, (4, 1), 62, 4), (orc.KIND_INNER, 3, 32, 128, 2, (6, 2), 126, 9),
    (orc.KIND_INNER, 4, 32, 128, 1, (8, 1), 158, 8),          # the first value group leaves; the fused kernel after it
    (orc.KIND_INNER, 3, 64, 128, 1, (5, 1), 189, 9), (orc.KIND_INNER, 2, 32, 1, 2, (2, 2), 1, 40), (orc.KIND_INNER, 2, 64, 2, 1, (1, 1), 3, 70),
    (orc.KIND_INNER, 2, 32, 230, 1, (4, 2), 252, 8),          # ... and on to caches that take more than one work-group
    (orc.KIND_INNER, 2, 32, 128, 40, (8, 2), 131, 3), (orc.KIND_INNER, 4, 64, 128, 150, (8, 2), 130, 3), (orc.KIND_INNER, 3, 64, 128, 300, (1, 1), 134, 2),
    (orc.KIND_INNER, 3, 32, 8, 130, (40, 8), 12, 4), (orc.KIND_INNER, 2, 64, 50, 130, (40, 8), 61, 5),     # crowded: two launches up to 64 tokens
    (orc.KIND_OUTER, 2, 32, 128, 2, (8, 2), 130, 6), (orc.KIND_OUTER, 4, 64, 32, 1, (3, 1), 60, 5), (orc.KIND_FP16, 2, 32, 128, 2, (8, 2), 129, 5),
])
def test_steps_of_short_caches(kind, bits, group, recent, batch, heads, start, steps):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    one = batch > 2                                          # (sequences of a large batch are copies of one, which the oracle follows)
    w = wl.Workload("s", 1 if one else batch, heads[0], heads[1], 128, start + steps, bits, group, 4, recent, seed=start + group,
                    k_mode=orc.HYBRID, v_mode=orc.HYBRID)
    o = oracle_config(w, kind=kind)
    K, V = wl.kv_full(w)

    def spread(a):
        t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
        return t.expand(batch, *t.shape[1:]).contiguous() if one else t

    norm, _ = orc.calibrate_key_norm(K, per_head=True)
    g = iq.allocate_cache(gpu_config(oracle_config(w.with_(batch=batch), kind=kind)))
    iq.innerq_quantize_append(g, spread(K[:, :, :start]), spread(V[:, :, :start]))
    iq.innerq_quantize_ahead(g)
    want = orc.cache_init_prefill(o, K[:, :, :start], V[:, :, :start])
    ws = iq.allocate_workspace(g.cfg)
    ws.fill_(0xFF)                                           # (its contents must not matter)
    for i in range(steps):
        q, n = wl.query(w, 0, i), start + i
        scale = norm if i % 2 else None
        qs = torch.from_numpy(np.ascontiguousarray(norm, dtype=np.float32)).cuda() if i % 2 else None
        out = iq.innerq_decode_step(g, spread(K[:, :, n:n + 1]), spread(V[:, :, n:n + 1]), spread(q), ws, q_scale=qs).cpu().numpy()
        orc.quantize_append(o, want, K[:, :, n:n + 1], V[:, :, n:n + 1])
        ref = orc.decode_attention(o, want, q, q_scale=scale)
        fused = min(orc.partition(o, x, n + 1)[1] for x in "kv") > 0            # (a fused kernel: fp16 weights)
        tol = 2e-3 if fused else TOL
        assert max_rel_err(out, np.repeat(ref, batch, 0) if one else ref) <= tol, f"step {i}"
        again = iq.innerq_decode_attention(g, spread(q), ws, q_scale=qs).cpu().numpy()       # the same tokens, now appended
        assert max_rel_err(again, np.repeat(ref, batch, 0) if one else ref) <= tol, f"step {i}"
    assert_cache_equal(g, want, o, bsel=slice(0, 1) if one else slice(None))


def step_us(torch, iq, batch, heads, recent, n):
    """GPU time of a decode step over n tokens, from a replayed graph of ten."""
    cfg = iq.make_config(batch, heads[0], heads[1], 128, 3, 32, 4, recent, capacity_tokens=256)
    c, ws = iq.allocate_cache(cfg), iq.allocate_workspace(cfg)
    x = torch.randn(batch, heads[1], n, 128, device="cuda").half()
    one, q, out = x[:, :, :1].contiguous(), torch.randn(batch, heads[0], 128, device="cuda").half(), torch.empty(batch, heads[0], 128, device="cuda")
    iq.innerq_quantize_append(c, x, x)
    iq.innerq_quantize_ahead(c)

    def again():
        c.c.n_tokens, c.c.store_ahead_tokens = n, n + 1
        iq.innerq_decode_step(c, one, one, q, ws, out=out)

    again()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(10):
            again()
    best = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        best.append(a.elapsed_time(b) * 100)
    return min(best)


@pytest.mark.parametrize("batch,heads,n", [(600, (40, 8), 17), (300, (40, 8), 9)])
def test_packed_rows_of_many_heads(batch, heads, n):
    """A tile of packed key rows over thousands of sequence-heads wants small work-groups: 1.2 times a step over fp16 rows (109 us,
    91), where a work-group that fills its compute unit for each took 1.6 (148)."""
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    packed, plain = step_us(torch, iq, batch, heads, 1, n), step_us(torch, iq, batch, heads, 128, n)
    assert packed < 1.4 * plain, (packed, plain)
