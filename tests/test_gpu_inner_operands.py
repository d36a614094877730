"""Precision of the fused inner-grouped kernel's integer products.

Where many weights are alike, the output is about 1 / sqrt(N) of the values' size, and so is what the rounding of the weights to
fp16 adds: each weight is off by up to 2^-11 of itself, uniformly, independently of the others, so the output's 2-norm is
off by 2^-11 / sqrt(12) to 2^-10 / sqrt(12) of itself (1.4e-4 to 2.8e-4, by where the weights' mantissas lie).  Sums of
products that lose bits do not shrink with 1 / sqrt(N), so they would show here first.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import gpu_config, oracle_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,v_bits,group,mode", [(2, 0, 32, orc.HYBRID), (2, 0, 64, orc.ASYM), (3, 0, 32, orc.SYM),
                                                    (3, 2, 64, orc.HYBRID), (4, 0, 32, orc.HYBRID), (4, 0, 64, orc.SYM)])
@pytest.mark.parametrize("heads", [4, 8, 3])
def test_flat_weights_over_a_long_context(bits, v_bits, group, mode, heads):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    w = wl.Workload("m", 1, heads, 1, 128, 16001, bits, group, 4, 128, k_mode=mode, v_mode=mode, seed=bits)
    o = oracle_config(w, v_bits=v_bits)
    K, V = wl.kv_full(w)
    q = (wl.query(w) * np.float16(0.5)).astype(np.float16)
    g = iq.allocate_cache(gpu_config(o))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    iq.innerq_quantize_append(g, dev(K), dev(V))
    out = iq.innerq_decode_attention(g, dev(q), iq.allocate_workspace(g.cfg)).cpu().numpy().astype(np.float64)
    want = orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)
    err = np.linalg.norm(out - want) / np.linalg.norm(want)
    assert err <= 3e-4, err
