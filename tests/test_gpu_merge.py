"""The log-sum-exp merge with one and with four wavefronts per head: partial counts around every boundary.

One sequence on one kv head gets a wavefront per 64-token tile, so the length sets the number of partials: a few, shares
that do not divide evenly, a wavefront's first 32 partials and its second load (4 x 32).  The counts and heads at which
four wavefronts take over (33 partials on 4 to 128 heads, 49 on up to 256) have a test of their own, which reads the number
of partials back from the workspace: it depends on the planner, and sizes that miss the line would prove nothing.
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
    run(kind, heads, 32, tiles)


@pytest.mark.parametrize("kind,heads,recent,tiles,partials,four", [
    (orc.KIND_INNER, (3, 1), 32, 30, 36, False), (orc.KIND_INNER, (3, 1), 32, 46, 52, True), (orc.KIND_FP16, (3, 1), 32, 45, 49, True),
    (orc.KIND_INNER, (4, 1), 32, 26, 32, False), (orc.KIND_INNER, (4, 1), 32, 28, 34, True), (orc.KIND_FP16, (4, 1), 32, 29, 33, True),
    (orc.KIND_INNER, (128, 32), 32, 28, 32, False), (orc.KIND_INNER, (128, 32), 32, 30, 34, True),
    (orc.KIND_INNER, (132, 33), 32, 30, 33, False), (orc.KIND_FP16, (132, 33), 32, 45, 49, True),
    (orc.KIND_INNER, (256, 64), 900, 4, 59, True), (orc.KIND_FP16, (256, 32), 1000, 20, 48, False),
    (orc.KIND_INNER, (264, 33), 900, 4, 60, False), (orc.KIND_FP16, (264, 33), 900, 4, 58, False),
])
def test_lines_of_the_rule(kind, heads, recent, tiles, partials, four):
    import torch
    assert four == ((partials >= 33 and 4 <= heads[0] <= 128) or (partials >= 49 and heads[0] <= 256))
    ws = run(kind, heads, recent, tiles)
    written = int((ws[256:].view(torch.int32) != -1).sum())       # (m, l) and 128 channels per partial and head
    assert written == partials * heads[0] * 130


def run(kind, heads, recent, tiles):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    n = 4 + recent + 64 * tiles
    w = wl.Workload("p", 1, heads[0], heads[1], 128, n + 1, 2, 32, 4, recent, seed=tiles)
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
    return ws
