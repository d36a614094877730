"""Launches that join their own partial results: one work-group per sequence-head and two to eight, of few and of eight
wavefronts, for two to eight query heads and all widths, more of them than fit the chip at once, and windows of many chunks;
steps at which a value group leaves its ring; a workspace of any content; replays from a graph.

Which launch ran is read back from the workspace, since it depends on the planner and sizes that miss a path would prove nothing: a
work-group by itself writes none of it, joined work-groups leave the words that they published cleared, and a launch that keeps
the merge leaves its partial results.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import assert_cache_equal, gpu_config, max_rel_err, oracle_config

pytestmark = pytest.mark.gpu
TOL = 2e-3
MERGE = 0                                                # (else: work-groups of a sequence-head; a pair: before and after the value group leaves)


def joined_groups(ws, batch, heads):
    """Work-groups of a sequence-head that joined in the last call, from a workspace that held nothing but 0xFF before it."""
    import torch
    words = ws[-(-4 * batch // 256) * 256:].view(torch.int32)
    written = words != -1
    n = int(written.sum())
    if n == 0:
        return 1
    if int((words[written] != 0).sum()) > 0:
        assert n % (130 * batch * heads) == 0
        return MERGE
    assert n % (264 * batch * heads) == 0                # (a half head: 64 channels, a level and a sum of 64 bits)
    return n // (264 * batch * heads)


@pytest.mark.parametrize("batch,q_heads,kv_heads,tokens,recent,group,bits,groups", [
    (1, 4, 1, 200, 32, 32, 4, 1), (2, 8, 2, 440, 48, 64, 2, 1), (64, 8, 1, 440, 64, 32, 3, 1),      # one work-group
    (1, 3, 1, 900, 32, 32, 2, (4, 3)), (1, 32, 8, 1500, 128, 32, 4, (7, 6)), (1, 4, 1, 6000, 128, 32, 2, 8), (1, 4, 1, 9000, 128, 32, 2, 8),
    (1, 4, 1, 1500, 900, 32, 2, 8),                                                  # window chunks for most of the wavefronts
    (64, 4, 1, 9000, 128, 32, 2, 4), (64, 8, 1, 9000, 128, 32, 2, 4), (64, 5, 1, 9000, 48, 64, 2, 4),       # a full chip
    (64, 4, 1, 9000, 48, 32, 3, 4), (64, 8, 1, 9000, 128, 64, 3, 4), (128, 8, 1, 5000, 32, 32, 4, 2),
    (40, 4, 1, 3000, 128, 32, 2, 6), (256, 2, 1, 2500, 32, 32, 2, 1), (300, 1, 1, 700, 32, 32, 2, 1), (1024, 1, 1, 3700, 500, 32, 2, 2),              # ... and more than fit it at once
    (2, 16, 2, 3000, 128, 64, 2, MERGE), (3, 15, 3, 2000, 48, 32, 3, MERGE), (1, 4, 1, 12000, 128, 32, 2, MERGE),
    (2100, 2, 1, 250, 40, 32, 2, MERGE), (72, 4, 1, 6000, 128, 32, 2, MERGE),
])
def test_steps(batch, q_heads, kv_heads, tokens, recent, group, bits, groups):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    steps = 3
    n = tokens - (tokens - 4 - recent) % group + group - 3       # a value group leaves its ring within the steps
    # (sequences of a large batch are copies of one, which the oracle follows)
    one = batch > 8
    w = wl.Workload("j", 1 if one else batch, q_heads, kv_heads, 128, n + steps, bits, group, 4, recent, seed=tokens)
    o = oracle_config(w)
    K, V = wl.kv_full(w)

    def spread(a):
        t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
        return t.expand(batch, *t.shape[1:]).contiguous() if one else t

    g = iq.allocate_cache(gpu_config(oracle_config(w.with_(batch=batch))))
    iq.innerq_quantize_append(g, spread(K[:, :, :n]), spread(V[:, :, :n]))
    iq.innerq_quantize_ahead(g)
    want = orc.cache_init_prefill(o, K[:, :, :n], V[:, :, :n])
    ws = iq.allocate_workspace(g.cfg)
    for i in range(steps):
        q = wl.query(w, 0, i)
        k1, v1, qd = spread(K[:, :, n + i:n + i + 1]), spread(V[:, :, n + i:n + i + 1]), spread(q)
        leaves = (n + i + 2 - 4 - recent) % group == 0            # (the merge takes the group along on a chip that is not full)
        out = None
        for content in (0x00, 0x3F, 0xFF):                        # (its contents must not matter)
            ws.fill_(content)
            g.c.n_tokens, g.c.store_ahead_tokens = n + i, n + i + 1
            again = iq.innerq_decode_step(g, k1, v1, qd, ws).cpu().numpy()
            assert out is None or np.array_equal(out, again)
            out = again
        left = (n + i + 1 - 4 - recent) % group <= i              # ... or has left in these steps
        expect = MERGE if leaves and batch * kv_heads < 256 else groups[left] if isinstance(groups, tuple) else groups
        got = joined_groups(ws, batch, q_heads)
        assert got == expect, f"step {i}: {got} work-groups"
        orc.quantize_append(o, want, K[:, :, n + i:n + i + 1], V[:, :, n + i:n + i + 1])
        ref = orc.decode_attention(o, want, q)
        for b in range(0, batch, max(1, batch // 7)):
            assert max_rel_err(out[b:b + 1], ref[:1] if one else ref[b:b + 1]) <= TOL, f"step {i} sequence {b}"
        again = iq.innerq_decode_attention(g, qd, ws).cpu().numpy()   # the same tokens, now appended
        assert max_rel_err(again, out) <= TOL
    assert_cache_equal(g, want, o, bsel=slice(0, 1) if one else slice(None))


@pytest.mark.parametrize("batch,q_heads,kv_heads,recent,quantised", [(1, 4, 1, 8192, 12416), (2, 2, 1, 7168, 12800), (1, 4, 4, 6144, 12352)])
def test_windows_of_more_chunks_than_wavefronts_joined(batch, q_heads, kv_heads, recent, quantised):
    """A recent window as long as the quantised range: the plan has to keep a wavefront without a window chunk."""
    import torch
    from paper_2602_23200_amd import binding as iq
    n = 4 + recent + quantised
    w = wl.Workload("w", batch, q_heads, kv_heads, 128, n + 1, 2, 32, 4, recent, seed=recent)
    o = oracle_config(w)
    K, V = wl.kv_full(w)
    q = wl.query(w)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    g = iq.allocate_cache(gpu_config(o))
    iq.innerq_quantize_append(g, dev(K[:, :, :n]), dev(V[:, :, :n]))
    iq.innerq_quantize_ahead(g)
    out = iq.innerq_decode_step(g, dev(K[:, :, n:]), dev(V[:, :, n:]), dev(q), iq.allocate_workspace(g.cfg)).cpu().numpy()
    assert max_rel_err(out, orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)) <= TOL


def test_kernel_choice_changed_by_another_thread():
    """innerq_select_inner_kernel from a second thread: every step is planned for the kernel that runs it."""
    import threading

    import torch
    from paper_2602_23200_amd import binding as iq
    w = wl.Workload("t", 1, 4, 1, 128, 1500, 2, 32, 4, 128, seed=9)              # joined by the default kernel, not by the other
    o = oracle_config(w)
    K, V = wl.kv_full(w)
    q = wl.query(w)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    n = w.n_tokens - 1
    g = iq.allocate_cache(gpu_config(o))
    iq.innerq_quantize_append(g, dev(K[:, :, :n]), dev(V[:, :, :n]))
    iq.innerq_quantize_ahead(g)
    k1, v1, qd = dev(K[:, :, n:]), dev(V[:, :, n:]), dev(q)
    ws, outs = iq.allocate_workspace(g.cfg), torch.empty(2000, 1, 4, 128, device="cuda")
    done = threading.Event()

    def change():
        while not done.is_set():
            iq.innerq_select_inner_kernel(1)
            iq.innerq_select_inner_kernel(0)

    other = threading.Thread(target=change)
    outs.fill_(float("nan"))
    other.start()
    try:
        for i in range(outs.shape[0]):
            g.c.n_tokens, g.c.store_ahead_tokens = n, n + 1
            iq.innerq_decode_step(g, k1, v1, qd, ws, out=outs[i])
    finally:
        done.set()
        other.join()
        iq.innerq_select_inner_kernel(0)
    want = orc.decode_attention(o, orc.cache_init_prefill(o, K, V), q)
    assert max_rel_err(outs.cpu().numpy(), np.broadcast_to(want, outs.shape)) <= TOL


def test_replays_from_a_graph_start_from_nothing():
    """A recorded launch keeps its tag: what a replay publishes must not be taken for the next one's."""
    import torch
    from paper_2602_23200_amd import binding as iq
    w = wl.Workload("g", 16, 32, 8, 128, 4600, 2, 32, 4, 128, seed=5)            # fills the chip: joined by the call itself
    cfg = gpu_config(oracle_config(w))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    rows = lambda *s: torch.randn(*s, generator=gen, device="cuda").half()  # noqa: E731
    g = iq.allocate_cache(cfg)
    iq.innerq_quantize_append(g, rows(16, 8, 4600, 128), rows(16, 8, 4600, 128))
    ws, other = iq.allocate_workspace(cfg), iq.allocate_workspace(cfg)
    q, out = rows(16, 32, 128), torch.empty(16, 32, 128, device="cuda")
    iq.innerq_decode_attention(g, q, ws, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        iq.innerq_decode_attention(g, q, ws, out=out)
    for i in range(12):
        q.copy_(rows(16, 32, 128))
        out.fill_(float("nan"))
        graph.replay()
        if i % 3 == 0:
            graph.replay()
        ref = iq.innerq_decode_attention(g, q, ws if i % 2 else other)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), f"replay {i}"
