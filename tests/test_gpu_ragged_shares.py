"""innerq_decode_step_ragged: the wavefronts of a launch shared over the sequences by their lengths.

Batches at the edges of the plan: two sequences, 32 (the most that share) and 33 and 65 (every sequence the same number), one long
sequence among short ones (as many wavefronts as it has partial slots), all short (none has a tile), equal lengths, and
a loose bound.  Every sequence against the oracle on its own.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import assert_cache_equal, gpu_config, max_rel_err, oracle_config

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.mark.parametrize("name,lengths,heads,group,bound", [
    ("two", [3000, 17], (4, 1), 32, 0),
    ("32", [5 + 37 * i % 1500 for i in range(32)], (2, 1), 32, 0),
    ("33", [5 + 41 * i % 1500 for i in range(33)], (4, 1), 32, 0),
    ("65", [5 + 37 * i % 900 for i in range(65)], (2, 1), 64, 0),
    ("one long", [40, 12000, 300, 5, 64], (8, 2), 32, 0),
    ("all short", [1, 5, 130, 60, 164, 163], (4, 1), 64, 0),
    ("equal", [1000] * 9, (4, 2), 32, 0),
    ("loose bound", [700, 90, 2100], (8, 1), 64, 9000),
])
def test_every_sequence_of_a_shared_launch(name, lengths, heads, group, bound):
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    B, steps = len(lengths), 3
    n_most = max(lengths) + steps
    w = wl.Workload("r", B, heads[0], heads[1], 128, n_most, 2, group, 4, 128, seed=7)
    cap = -(-max(n_most, bound) // group) * group + group
    o, o1 = oracle_config(w, capacity=cap), oracle_config(w.with_(batch=1), capacity=cap)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    g = iq.allocate_cache(gpu_config(o))
    want, kv = [], []
    for b, n in enumerate(lengths):
        slabs = [wl.kv_slab(w, b, h, n_tokens=n + steps) for h in range(heads[1])]
        K, V = np.stack([s[0] for s in slabs])[None], np.stack([s[1] for s in slabs])[None]
        view = iq.sequence_view(g, b)
        iq.innerq_quantize_append(view, dev(K[:, :, :n]), dev(V[:, :, :n]))
        iq.innerq_quantize_ahead(view)
        want.append(orc.cache_init_prefill(o1, K[:, :, :n], V[:, :, :n]))
        kv.append((K, V))
    counts = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    ws = iq.allocate_workspace(g.cfg)
    ws.fill_(0xA5)                                        # (its contents must not matter)
    for i in range(steps):
        k1 = np.concatenate([K[:, :, n + i:n + i + 1] for (K, _), n in zip(kv, lengths)])
        v1 = np.concatenate([V[:, :, n + i:n + i + 1] for (_, V), n in zip(kv, lengths)])
        q = wl.query(w, step=i)
        out = iq.innerq_decode_step_ragged(g, counts, bound or n_most, dev(k1), dev(v1), dev(q), ws).cpu().numpy()
        assert counts.cpu().tolist() == [n + i + 1 for n in lengths]
        for b in range(B):
            orc.quantize_append(o1, want[b], k1[b:b + 1], v1[b:b + 1])
            if B < 20 or b % 7 == 0:
                assert max_rel_err(out[b:b + 1], orc.decode_attention(o1, want[b], q[b:b + 1])) <= TOL, f"{name} {i} {b}"
    for b in range(B):
        assert_cache_equal(g, want[b], o1, bsel=slice(b, b + 1), what=f"{name} sequence {b}", per_sequence=True)
