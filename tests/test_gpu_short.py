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
