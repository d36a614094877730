"""The log-sum-exp merge with one and with four wavefronts per head: partial counts around every boundary.

One sequence on one kv head gets a wavefront per 64-token tile, so the length sets the number of partials: a few, the
count at which four wavefronts take over (25 with up to 64 heads, 49 with up to 256), shares that do not divide
evenly, a wavefront's first 32 partials and its second load (4 x 32), and head counts on both sides of the rule.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import gpu_config, max_rel_err, oracle_config

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.mark.parametrize("kind", [orc.KIND_INNER, orc.KIND_FP16])
@pytest.mark.parametrize("heads,tiles", [((1, 1), t) for t in (1, 2, 5, 7, 9, 10, 11, 12, 13, 15, 16, 17, 18, 19, 20, 31, 40, 42, 43, 44, 45, 46, 47,
                                                               120, 130, 300)] + [((4, 1), 20), ((64, 16), 20), ((68, 17), 20), ((256, 64), 46), ((264, 66), 46)])
def test_partial_counts(kind, heads, tiles):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    n = 4 + 32 + 64 * tiles
    w = wl.Workload("p", 1, heads[0], heads[1], 128, n + 1, 2, 32, 4, 32, seed=tiles)
    o = oracle_config(w, kind=kind)
    K, V = wl.kv_full(w)
    q = wl.query(w)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    g = iq.allocate_cache(gpu_config(o))
    iq.innerq_quantize_append(g, dev(K[:, :, :n]), dev(V[:, :, :n]))
    iq.innerq_quantize_ahead(g)
    ws = iq.allocate_workspace(g.cfg)
    ws.fill_(0xFF)                                        # (NaN everywhere: what is not written must not be read)
    step = iq.innerq_decode_step(g, dev(K[:, :, n:]), dev(V[:, :, n:]), dev(q), ws)
    want = orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)
    assert max_rel_err(step.cpu().numpy(), want) <= TOL
    ws.fill_(0xFF)
    assert max_rel_err(iq.innerq_decode_attention(g, dev(q), ws).cpu().numpy(), want) <= TOL
