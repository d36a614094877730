"""The outer-grouped kernel around its tiles (16 half-words: 128 tokens of 2 bits, 64 of 4): quantised ranges that end inside one,
token groups and channel groups of 32 and 64, one to eight query heads, every combination of zero-point arrays, several
tiles a wavefront, scales whose magnitudes force another normalisation in every tile, and tiles of zero and tiny ones, against the oracle.

Softmax weights and their products with the value scales are fp16 numbers (relative 2^-12 each), the bound that the other parity tests use.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import gpu_config, max_rel_err, oracle_config

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.mark.parametrize("bits,group,batch,heads,quantised,modes,ramp", [
    (2, 32, 1, (4, 1), 32, (orc.HYBRID, orc.HYBRID), False), (2, 32, 2, (3, 1), 96, (orc.ASYM, orc.SYM), False), (2, 32, 1, (8, 2), 128, (orc.SYM, orc.ASYM), False),
    (2, 32, 1, (5, 1), 160, (orc.HYBRID, orc.HYBRID), False), (2, 32, 1, (8, 1), 2016, (orc.SYM, orc.SYM), True), (2, 64, 2, (6, 3), 64, (orc.HYBRID, orc.ASYM), False),
    (2, 64, 1, (8, 1), 192, (orc.HYBRID, orc.HYBRID), True), (2, 64, 1, (1, 1), 1984, (orc.SYM, orc.SYM), False), (4, 32, 1, (4, 1), 32, (orc.HYBRID, orc.HYBRID), False),
    (4, 32, 2, (7, 1), 96, (orc.SYM, orc.HYBRID), False), (4, 32, 1, (2, 1), 1056, (orc.ASYM, orc.ASYM), True), (4, 64, 1, (8, 1), 64, (orc.HYBRID, orc.SYM), False),
    (4, 64, 1, (4, 2), 2112, (orc.HYBRID, orc.HYBRID), False),
    (2, 32, 130, (8, 2), 1376, (orc.HYBRID, orc.HYBRID), True), (4, 32, 300, (5, 1), 736, (orc.HYBRID, orc.SYM), True),       # several tiles a wavefront
])
def test_outer_attention(bits, group, batch, heads, quantised, modes, ramp):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    one = batch > 2                                          # (sequences of a large batch are copies of one)
    n = 4 + 32 + quantised + 5                               # (the values keep five tokens more than whole groups of keys)
    w = wl.Workload("o", 1 if one else batch, heads[0], heads[1], 128, n, bits, group, 4, 32, seed=quantised + bits, k_mode=modes[0], v_mode=modes[1])
    o = oracle_config(w, kind=orc.KIND_OUTER)
    K, V = wl.kv_full(w)
    if ramp:                                                 # magnitudes that grow along the tokens, and back
        f = np.exp2(np.round(6 * np.sin(np.arange(n) / 90.0))).astype(np.float16)
        K, V = K * (f ** np.float16(0.25))[:, None], V * f[:, None]
    q = wl.query(w)

    def spread(a):
        t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
        return t.expand(batch, *t.shape[1:]).contiguous() if one else t

    g = iq.allocate_cache(gpu_config(oracle_config(w.with_(batch=batch), kind=orc.KIND_OUTER)))
    iq.innerq_quantize_append(g, spread(K), spread(V))
    assert min(orc.partition(o, x, n)[1] for x in "kv") == quantised
    out = iq.innerq_decode_attention(g, spread(q), iq.allocate_workspace(g.cfg)).cpu().numpy()
    want = orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)
    assert max_rel_err(out, np.repeat(want, batch, 0) if one else want) <= TOL


@pytest.mark.parametrize("what", ["keys all zero", "a tile of zero keys", "keys x 2^-12", "keys x 2^-16", "a tile of zero values", "values x 2^-12"])
@pytest.mark.parametrize("k_mode", [orc.SYM, orc.ASYM, orc.HYBRID])
@pytest.mark.parametrize("group,heads", [(32, (4, 1)), (64, (8, 1))])
@pytest.mark.parametrize("bits", [2, 4])
def test_zero_and_tiny_groups(bits, group, heads, k_mode, what):
    """Tiles whose scales are all zero, or fp16 denormals: the power of two that normalises them is at its upper end (2^14, and
    2^14 times the level 2^(b-1) is no fp16 number at 4 bits)."""
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    n = 4 + 32 + 512 + 5
    w = wl.Workload("z", 1, heads[0], heads[1], 128, n, bits, group, 4, 32, seed=bits + group, k_mode=k_mode, v_mode=orc.HYBRID)
    o = oracle_config(w, kind=orc.KIND_OUTER)
    K, V = wl.kv_full(w)
    if what == "keys all zero":
        K[:] = 0
    elif what == "a tile of zero keys":
        K[:, :, 4 + 128:4 + 256] = 0                         # one tile of 128 tokens, two of 64
    elif what == "a tile of zero values":
        V[:, :, 4 + 128:4 + 256] = 0
    else:
        x, shift = what.split(" x 2^")
        (K if x == "keys" else V)[:] *= np.float16(2.0 ** int(shift))
    q = wl.query(w)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    g = iq.allocate_cache(gpu_config(o))
    iq.innerq_quantize_append(g, dev(K), dev(V))
    out = iq.innerq_decode_attention(g, dev(q), iq.allocate_workspace(g.cfg)).cpu().numpy()
    assert np.isfinite(out).all()
    assert max_rel_err(out, orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)) <= TOL


def test_window_of_a_million_tokens():
    """68754 window chunks of a sequence-head: more than the second dimension of a grid.  (The quantised tokens are zeros, which every
    width holds exactly, so that the inputs themselves are what is attended to.)"""
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    recent, quantised = 1_100_000, 64
    n = 4 + quantised + recent
    cfg = iq.make_config(1, 2, 1, 128, 4, 32, 4, recent, kind=orc.KIND_OUTER, capacity_tokens=-(-n // 64) * 64)
    gen = torch.Generator(device="cuda").manual_seed(8)
    K, V = (torch.randn(1, 1, n, 128, device="cuda", generator=gen).half() for _ in range(2))
    K[:, :, 4:4 + quantised] = 0
    V[:, :, 4:4 + quantised] = 0
    q = 2 * torch.randn(1, 2, 128, device="cuda", generator=gen).half()
    g = iq.allocate_cache(cfg)
    iq.innerq_quantize_append(g, K, V)
    assert iq.innerq_partition(cfg, 0, n)[1] == quantised
    out = iq.innerq_decode_attention(g, q, iq.allocate_workspace(cfg))
    s = (K[0, 0].double() @ q[0].double().T) / 128 ** 0.5
    want = torch.softmax(s, 0).T @ V[0, 0].double()
    assert ((out[0].double() - want).abs().amax(-1) / want.abs().amax(-1)).max().item() <= TOL
