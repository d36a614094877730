"""The fp32 attention kernel (short caches and the forms no fused kernel serves) against the oracle.

Everything in it is fp32, weights included, so the bound is that of fp32 sums: a score is a sum of 128
products (absolute error up to 128 x 2^-24 of sum |q k| / sqrt(d), below 1e-5 for these inputs), which
moves a weight by as much relative to itself; the weighted sums add the same order again.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import gpu_config, max_rel_err, oracle_config

pytestmark = pytest.mark.gpu
TOL = 5e-5


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    iq.lib()
    return torch, iq


CASES = [
    # nothing quantised in both tensors yet: one 64-token tile per work-group, its edges, packed rows of one tensor
    *[(kind, bits, 0, 32, (8, 2), n) for kind, bits in ((orc.KIND_INNER, 4), (orc.KIND_INNER, 3), (orc.KIND_OUTER, 2),
                                                        (orc.KIND_FP16, 2)) for n in (1, 63, 64, 65, 131, 132, 163)
      if kind != orc.KIND_FP16 or n <= 132],          # (an fp16 store with a row in it has a fused kernel)
    # forms without a fused kernel: several tiles per work-group, both tensors packed, a remainder of heads
    (orc.KIND_INNER, 2, 4, 32, (20, 2), 900), (orc.KIND_INNER, 4, 2, 64, (8, 2), 1111), (orc.KIND_INNER, 2, 3, 32, (2, 1), 777),
    (orc.KIND_OUTER, 3, 0, 32, (8, 2), 900), (orc.KIND_OUTER, 3, 4, 64, (12, 1), 1500), (orc.KIND_FP16, 2, 0, 32, (10, 1), 2100),
]


@pytest.mark.parametrize("kind,bits,v_bits,group,heads,n_tokens", CASES)
@pytest.mark.parametrize("scaled", [False, True])
def test_fp32_attention(env, kind, bits, v_bits, group, heads, n_tokens, scaled):
    torch, iq = env
    w = wl.Workload("g", 2, heads[0], heads[1], 128, n_tokens, bits, group, 4, 128, seed=n_tokens + bits,
                    k_mode=orc.HYBRID, v_mode=orc.HYBRID)
    o = oracle_config(w, kind=kind, v_bits=v_bits)
    K, V = wl.kv_full(w)
    q = wl.query(w)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    norm = inv = None
    if scaled:
        norm, inv = orc.calibrate_key_norm(K, per_head=True)
    want = orc.decode_attention(o, orc.cache_init_prefill(o, K, V, k_inv_norm=inv),
                                q if norm is None else (q.astype(np.float32).reshape(2, heads[1], -1, 128)
                                                        * norm[None, :, None, :].astype(np.float32)).astype(np.float16).reshape(q.shape))
    g = iq.allocate_cache(gpu_config(o))
    iq.innerq_quantize_append(g, dev(K), dev(V), None if inv is None else dev(inv.astype(np.float32)))
    out = iq.innerq_decode_attention(g, dev(q), iq.allocate_workspace(g.cfg),
                                     q_scale=None if norm is None else dev(norm.astype(np.float32)))
    assert max_rel_err(out.cpu().numpy(), want) <= TOL


@pytest.mark.parametrize("batch,n_tokens", [(128, 1), (129, 1), (128, 64), (64, 65), (65, 65), (300, 3)])
@pytest.mark.parametrize("heads", [(2, 2), (8, 2)])
def test_more_work_groups_than_compute_units(env, batch, n_tokens, heads):
    """Short caches of many sequences: up to 256 work-groups take a row a thread, more take four."""
    torch, iq = env
    w = wl.Workload("g", batch, heads[0], heads[1], 128, n_tokens, 2, 32, 4, 128, seed=batch)
    o = oracle_config(w)
    K, V = wl.kv_full(w)
    q = wl.query(w)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    g = iq.allocate_cache(gpu_config(o))
    iq.innerq_quantize_append(g, dev(K), dev(V))
    out = iq.innerq_decode_attention(g, dev(q), iq.allocate_workspace(g.cfg))
    assert max_rel_err(out.cpu().numpy(), orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)) <= TOL
