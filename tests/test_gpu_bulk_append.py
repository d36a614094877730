"""Appends of prompts and chunks, in each form they run in (a group a lane, a group on eight lanes, owners of ring
slices), against the oracle.

Every byte is compared.  The sizes cross the edges of the forms' units (rows per wavefront: 16 at G = 32, 32 at G = 64;
groups per wavefront of a ring slice), chunks shorter and longer than the windows, a chunk that ends inside a group, and
the lines between the forms.
"""
import numpy as np
import pytest

from oracle import innerq_oracle as orc
from paper_2602_23200_amd import workloads as wl
from tests.helpers import assert_cache_equal, gpu_config, oracle_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    iq.lib()
    return torch, iq


def values(rng, shape, dist):
    x = rng.standard_normal(shape).astype(np.float32)
    if dist == "ties":                                    # quarters: codes on exact halves, both signs of zero
        x = np.round(x * 6) / 4
    elif dist == "denormal":                              # scales that are fp16 denormals: codes are clamped
        x = x * 2.0 ** -17
    elif dist == "wide":                                  # 2^-20 .. 2^14 side by side: differences that fp32 rounds
        x = x * np.exp2(rng.integers(-20, 14, shape))
    return x.clip(-60000, 60000).astype(np.float16)


@pytest.mark.parametrize("dist", ["normal", "ties", "denormal", "wide"])
@pytest.mark.parametrize("kind,bits,group,modes,literal,recent,chunks", [
    (orc.KIND_INNER, 2, 32, (orc.HYBRID, orc.HYBRID), 0, 128, (133, 2, 64, 501, 17, 300)),
    (orc.KIND_INNER, 4, 64, (orc.SYM, orc.ASYM), 0, 32, (300, 65, 64, 63)),
    (orc.KIND_INNER, 3, 32, (orc.HYBRID, orc.HYBRID), 1, 48, (1037, 50, 33)),
    (orc.KIND_INNER, 2, 64, (orc.SYM, orc.HYBRID), 1, 100, (700, 129)),
    (orc.KIND_OUTER, 3, 64, (orc.HYBRID, orc.SYM), 0, 64, (400, 100, 257)),
    (orc.KIND_OUTER, 4, 32, (orc.HYBRID, orc.HYBRID), 0, 300, (1500, 31, 700)),
    (orc.KIND_INNER, 2, 32, (orc.HYBRID, orc.HYBRID), 0, 1500, (1400, 900, 40, 2500)),     # a long ring
])
@pytest.mark.parametrize("norm", [False, True])
def test_bulk_append_bit_exact(env, kind, bits, group, modes, literal, recent, chunks, norm, dist):
    torch, iq = env
    n = sum(chunks)
    w = wl.Workload("b", 2, 3, 3, 128, n, bits, group, 4, recent, k_mode=modes[0], v_mode=modes[1])
    o = oracle_config(w, kind=kind, sym_denominator=literal)
    rng = np.random.default_rng(n + bits)
    K, V = values(rng, (2, 3, n, 128), dist), values(rng, (2, 3, n, 128), dist)
    inv = rng.uniform(0.3, 1.0, (3, 128)).astype(np.float32) if norm else None
    want = orc.cache_init_prefill(o, K, V, k_inv_norm=inv)
    g = iq.allocate_cache(gpu_config(o))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    at = 0
    for c in chunks:
        iq.innerq_quantize_append(g, dev(K[:, :, at:at + c]), dev(V[:, :, at:at + c]), None if inv is None else dev(inv))
        at += c
    assert_cache_equal(g, want, o)


@pytest.mark.parametrize("heads,group,recent,bits,mode,chunks", [
    # both variants, groups of 64: owners of a channel a lane from 8192 groups to 98304 (2 bits) or 163840
    (33, 64, 64, 2, orc.HYBRID, (200, 140, 300)),         # 9240 and 19800 groups
    (31, 64, 64, 2, orc.HYBRID, (200, 140, 300)),         # 8680 and 18600
    (29, 64, 64, 2, orc.HYBRID, (200, 140, 300)),         # 8120: two launches of eight lanes a group, then 17400
    (64, 64, 64, 2, orc.HYBRID, (200, 64, 767, 768)),     # 8192, 98176, and 98304: two launches of a group a lane
    (64, 64, 64, 4, orc.HYBRID, (200, 1279, 1280)),       # 163712, 163840
    # ... where a ring's groups are more than one round: of pairs, from 24 heads on
    (33, 64, 300, 2, orc.HYBRID, (500, 200, 400)),
    (23, 64, 300, 2, orc.HYBRID, (500, 200, 400)),
    # one variant: from 3072 groups on, a channel a lane up to 65536 (131072, 196608), then pairs
    (64, 64, 64, 2, orc.ASYM, (236, 24, 40, 511, 512)),   # 3072, no values, 65408, 65536
    (63, 64, 64, 2, orc.SYM, (236, 24)),                  # 3024: two launches
    (64, 64, 64, 3, orc.SYM, (200, 1023, 1024, 2048)),    # 130944, 131072, 262144: two launches
    (64, 64, 64, 4, orc.ASYM, (200, 1535, 1536)),         # 196480, 196608
    (33, 64, 300, 4, orc.ASYM, (500, 100, 400)),          # more rounds: 6600 groups, 26400
    (2, 32, 416, 2, orc.HYBRID, (900, 448, 449, 447, 480)),   # rings of 448 rows and more, a second round of their groups
    (40, 32, 32, 2, orc.HYBRID, (70, 2, 3, 130, 27, 4)),      # keys only, few groups, 4096 groups and more
])
@pytest.mark.parametrize("kind", [orc.KIND_INNER, orc.KIND_OUTER])
def test_lines_between_the_forms(env, kind, heads, group, recent, bits, mode, chunks):
    torch, iq = env
    n = sum(chunks)
    w = wl.Workload("l", 1, heads, heads, 128, n, bits, group, 4, recent, k_mode=mode, v_mode=mode)
    o = oracle_config(w, kind=kind)
    rng = np.random.default_rng(n)
    K, V = values(rng, (1, heads, n, 128), "normal"), values(rng, (1, heads, n, 128), "ties")
    g = iq.allocate_cache(gpu_config(o))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    at = 0
    for c in chunks:
        iq.innerq_quantize_append(g, dev(K[:, :, at:at + c]), dev(V[:, :, at:at + c]))
        at += c
    assert_cache_equal(g, orc.cache_init_prefill(o, K, V), o)


def device_values(torch, gen, shape, dist):
    x = torch.randn(shape, generator=gen, device="cuda")
    if dist == "ties":
        x = torch.round(x * 6) / 4
    elif dist == "denormal":
        x = x * 2.0 ** -17
    elif dist == "wide":
        x = x * torch.exp2(torch.randint(-20, 14, shape, generator=gen, device="cuda").float())
    elif dist == "offset":                                # differences small against the values: the bound's largest term
        x = x + 1000 * torch.randint(-1, 2, shape[:3] + (1,), generator=gen, device="cuda")
    x = x.clamp(-60000, 60000).half()
    if dist == "special":
        m = torch.rand(shape, generator=gen, device="cuda")
        x[m < 1e-4], x[(m > 1e-4) & (m < 2e-4)], x[(m > 2e-4) & (m < 3e-4)] = float("nan"), float("inf"), float("-inf")
        x[(m > .3) & (m < .4)] = -0.0
    return x


def same_bytes_whole_and_in_parts(torch, iq, cfg, K, V, inv, cuts):
    whole, parts = iq.allocate_cache(cfg), iq.allocate_cache(cfg)
    iq.innerq_quantize_append(whole, K, V, inv)
    for a, b in zip(cuts, cuts[1:]):
        iq.innerq_quantize_append(parts, K[:, :, a:b].contiguous(), V[:, :, a:b].contiguous(), inv)
    for name, buf in whole.buffers.items():
        if buf is not None and not name.endswith("recent"):               # (a ring's spare slots hold older tokens)
            assert torch.equal(buf, parts.buffers[name]), name


@pytest.mark.parametrize("dist", ["normal", "ties", "denormal", "wide", "offset", "special"])
@pytest.mark.parametrize("kind,bits,group,modes", [
    (orc.KIND_INNER, 2, 32, (orc.HYBRID, orc.HYBRID)), (orc.KIND_INNER, 2, 64, (orc.HYBRID, orc.HYBRID)),
    (orc.KIND_INNER, 3, 32, (orc.HYBRID, orc.HYBRID)), (orc.KIND_INNER, 3, 64, (orc.SYM, orc.HYBRID)),
    (orc.KIND_INNER, 4, 32, (orc.HYBRID, orc.ASYM)), (orc.KIND_INNER, 4, 64, (orc.HYBRID, orc.HYBRID)),
    (orc.KIND_INNER, 2, 32, (orc.SYM, orc.HYBRID)), (orc.KIND_INNER, 2, 64, (orc.HYBRID, orc.ASYM)),
    (orc.KIND_OUTER, 2, 32, (orc.HYBRID, orc.HYBRID)), (orc.KIND_OUTER, 2, 64, (orc.SYM, orc.HYBRID)), (orc.KIND_OUTER, 4, 64, (orc.HYBRID, orc.SYM)),
])
def test_shorter_error_sum(env, kind, bits, group, modes, dist):
    """From 2 M groups on (2.1 M here) a prompt of 2 bits, or 4 at G = 64, decides between the variants on a shorter error sum; the same tokens in
    parts below that line, which the tests above hold against the oracle, leave the same bytes, and so they do at other widths."""
    torch, iq = env
    H, n = 8, (1 << 21) // 8 * group // 128 + 200
    cfg = iq.make_config(1, H, H, 128, bits, group, 4, 128, modes[0], modes[1], 0, kind, capacity_tokens=-(-n // 64) * 64)
    gen = torch.Generator(device="cuda").manual_seed(bits * group)
    K, V = (device_values(torch, gen, (1, H, n, 128), dist) for _ in range(2))
    inv = torch.rand(H, 128, device="cuda", generator=gen) + 0.5 if group == 32 else None
    same_bytes_whole_and_in_parts(torch, iq, cfg, K, V, inv, (0, n // 3, n // 3 * 2 - 5, n))


@pytest.mark.parametrize("dist", ["normal", "ties", "denormal", "special"])
@pytest.mark.parametrize("kind,bits,modes", [
    (orc.KIND_INNER, 2, (orc.HYBRID, orc.HYBRID)), (orc.KIND_INNER, 3, (orc.SYM, orc.SYM)), (orc.KIND_INNER, 4, (orc.SYM, orc.HYBRID)),
    (orc.KIND_OUTER, 2, (orc.HYBRID, orc.ASYM)), (orc.KIND_OUTER, 3, (orc.ASYM, orc.HYBRID)),
])
def test_large_chunks_of_groups_of_32(env, kind, bits, modes, dist):
    """A chunk of 2.1 M groups onto 300 tokens: owners of ring slices with two channels a lane."""
    torch, iq = env
    H, n = 8, 66200
    cfg = iq.make_config(1, H, H, 128, bits, 32, 4, 128, modes[0], modes[1], 0, kind, capacity_tokens=-(-n // 64) * 64)
    gen = torch.Generator(device="cuda").manual_seed(bits)
    K, V = (device_values(torch, gen, (1, H, n, 128), dist) for _ in range(2))
    inv = torch.rand(H, 128, device="cuda", generator=gen) + 0.5
    same_bytes_whole_and_in_parts(torch, iq, cfg, K, V, inv, (0, 300, n))


def test_long_prompt_with_key_factors(env):
    """A prompt of 4 M groups, and in parts of at most 1.95 M; they leave the same bytes."""
    torch, iq = env
    n, H = 131400, 8
    cfg = iq.make_config(1, H, H, 128, 2, 32, 4, 128, capacity_tokens=131456)
    gen = torch.Generator(device="cuda").manual_seed(5)
    K, V = (torch.randn(1, H, n, 128, device="cuda", generator=gen).half() for _ in range(2))
    inv = torch.rand(H, 128, device="cuda", generator=gen) + 0.5
    same_bytes_whole_and_in_parts(torch, iq, cfg, K, V, inv, (0, 40000, 70000, 70601, n))


def append_us(torch, iq, heads, group, recent, cached, t, mode=orc.HYBRID):
    """GPU time of one append of t tokens onto `cached` ones, from a replayed graph of ten."""
    cfg = iq.make_config(1, heads, heads, 128, 2, group, 4, recent, mode, mode, capacity_tokens=-(-(cached + t) // 64) * 64)
    c = iq.allocate_cache(cfg)
    x = torch.randn(1, heads, max(cached, t), 128, device="cuda").half()
    if cached:
        iq.innerq_quantize_append(c, x[:, :, :cached].contiguous(), x[:, :, :cached].contiguous())
    x = x[:, :, :t].contiguous()

    def again():
        c.c.n_tokens = c.c.store_ahead_tokens = cached
        iq.innerq_quantize_append(c, x, x)

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


@pytest.mark.parametrize("group", [32, 64])
def test_long_windows_use_the_whole_chip(env, group):
    """The rows of a long ring are no work for one work-group: with a window of 8192 tokens instead of 128 a chunk of
    16384 has to read and copy as much again (12 and 17 us), not 86 (G = 32) and 158 us (G = 64)."""
    torch, iq = env
    short, long = (append_us(torch, iq, 1, group, recent, recent + 1000, 16384) for recent in (128, 8192))
    assert long < 4 * short, (short, long)


def test_many_heads_use_the_whole_chip(env):
    """Two tokens of 2048 heads have work for a few thousand wavefronts: 8 us, where 256 heads take 6; a work-group for
    every slice of every ring took 52."""
    torch, iq = env
    few, many = append_us(torch, iq, 256, 32, 128, 1000, 2), append_us(torch, iq, 2048, 32, 128, 1000, 2)
    assert many < 3 * few, (few, many)


@pytest.mark.parametrize("heads,t,recent,cached,mode", [
    (110, 8583, 16, 64, orc.ASYM), (60, 17635, 16, 64, orc.ASYM), (32, 5226, 128, 285, orc.ASYM), (16, 9040, 128, 611, orc.SYM),
])
def test_chunk_takes_what_a_prompt_takes(env, heads, t, recent, cached, mode):
    """Groups of 64 of one variant: a chunk onto a cache reads and packs what a first prompt of as many tokens does (84 us, 79; 22, 19);
    with a channel of two bytes a lane and load, owners of ring slices took 162, in two launches the smaller ones 29."""
    torch, iq = env
    chunk, prompt = (append_us(torch, iq, heads, 64, recent, c, t, mode) for c in (cached, 0))
    assert chunk < 1.3 * prompt, (chunk, prompt)


@pytest.mark.parametrize("kind,bits,group", [(orc.KIND_INNER, 2, 32), (orc.KIND_INNER, 4, 64), (orc.KIND_OUTER, 3, 32)])
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("chunks", [(300,), (20, 300), (140, 2, 40, 1, 200), (3, 133)])
def test_short_append_bit_exact(env, kind, bits, group, chunks, norm):
    """Calls of few groups: groups of new tokens only, of ring tokens only and of both."""
    torch, iq = env
    n = sum(chunks)
    w = wl.Workload("s", 2, 3, 3, 128, n, bits, group, 4, 32)
    o = oracle_config(w, kind=kind)
    rng = np.random.default_rng(n + bits)
    K, V = values(rng, (2, 3, n, 128), "normal"), values(rng, (2, 3, n, 128), "normal")
    inv = rng.uniform(0.3, 1.0, (3, 128)).astype(np.float32) if norm else None
    g = iq.allocate_cache(gpu_config(o))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    at = 0
    for c in chunks:
        iq.innerq_quantize_append(g, dev(K[:, :, at:at + c]), dev(V[:, :, at:at + c]), None if inv is None else dev(inv))
        at += c
    assert_cache_equal(g, orc.cache_init_prefill(o, K, V, k_inv_norm=inv), o)


@pytest.mark.parametrize("batch,heads,n_tokens", [(1, 1, 1), (2, 3, 255), (1, 5, 257), (3, 2, 1100), (1, 33, 600)])
@pytest.mark.parametrize("per_head", [False, True])
def test_calibration_exact(env, batch, heads, n_tokens, per_head):
    """Slices of one and several passes, fewer and more heads than the finishing threads take at once."""
    torch, iq = env
    rng = np.random.default_rng(heads)
    K = (rng.standard_normal((batch, heads, n_tokens, 128)) * 30).astype(np.float16)
    K[:, :, :, 5] = 0
    w = wl.Workload("c", batch, heads, heads, 128, n_tokens, 2, 32, 4, 32)
    for _ in range(3):
        norm, inv = iq.innerq_calibrate_key_norm(gpu_config(oracle_config(w)), torch.from_numpy(K).cuda(), per_head=per_head)
        norm_o, inv_o = orc.calibrate_key_norm(K, per_head=per_head)
        assert np.array_equal(norm.cpu().numpy(), norm_o.astype(np.float32))
        assert np.array_equal(inv.cpu().numpy(), inv_o.astype(np.float32))


@pytest.mark.parametrize("per_head", [False, True])
def test_calibration_into_one_buffer(env, per_head):
    """A caller that wants 1 / norm only may pass its buffer for both outputs: 1 / norm is what stays in it."""
    import ctypes
    torch, iq = env
    rng = np.random.default_rng(9)
    K = (rng.standard_normal((2, 3, 700, 128)) * 30).astype(np.float16)
    Kd = torch.from_numpy(K).cuda()
    inv = torch.full((3, 128), 7.0, device="cuda")
    cfg = gpu_config(oracle_config(wl.Workload("c", 2, 3, 3, 128, 700, 2, 32, 4, 32)))
    st = iq.lib().innerq_calibrate_key_norm(ctypes.byref(cfg), Kd.data_ptr(), 700, int(per_head), inv.data_ptr(), inv.data_ptr(),
                                            iq._stream(None))
    assert st == iq.OK
    assert np.array_equal(inv.cpu().numpy(), orc.calibrate_key_norm(K, per_head=per_head)[1].astype(np.float32))


@pytest.mark.parametrize("per_head", [False, True])
def test_calibration_passes_over_nan(env, per_head):
    """A NaN among the keys does not count towards its channel's maximum, nor does it hide the others (a channel of
    nothing but NaN is like one of zeros)."""
    torch, iq = env
    rng = np.random.default_rng(11)
    K = (rng.standard_normal((2, 3, 900, 128)) * 30).astype(np.float16)
    K[:, 1, 400, 7] = 6000.0                              # (the maximum of all heads is in the head that has the NaN)
    at = (rng.random(K.shape) < 0.01).astype(bool)
    at[:, 1, 400, 7] = False
    at[:, 2, :, 9] = True
    bad, good = K.copy(), K.copy()
    bad[at] = rng.integers(0x7C01, 0x8000, int(at.sum()), dtype=np.uint16).view(np.float16)    # signalling ones among them
    good[at] = 0
    cfg = gpu_config(oracle_config(wl.Workload("c", 2, 3, 3, 128, 900, 2, 32, 4, 32)))
    norm, inv = iq.innerq_calibrate_key_norm(cfg, torch.from_numpy(bad).cuda(), per_head=per_head)
    norm_o, inv_o = orc.calibrate_key_norm(good, per_head=per_head)
    assert np.array_equal(norm.cpu().numpy(), norm_o.astype(np.float32))
    assert np.array_equal(inv.cpu().numpy(), inv_o.astype(np.float32))


@pytest.mark.parametrize("kind,bits,group,mode", [(orc.KIND_INNER, 2, 32, orc.HYBRID), (orc.KIND_OUTER, 4, 64, orc.HYBRID),
                                                  (orc.KIND_INNER, 3, 64, orc.ASYM), (orc.KIND_OUTER, 2, 32, orc.SYM)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_bytes_do_not_depend_on_the_call(env, kind, bits, group, mode, bad):
    """NaN and infinite values leave the bytes of a group unspecified, but the same in a chunk and token by token."""
    torch, iq = env
    n = 1500                                              # (more than 16384 groups: the bulk form)
    w = wl.Workload("n", 2, 3, 3, 128, n, bits, group, 4, 32, k_mode=mode, v_mode=mode)
    rng = np.random.default_rng(bits)
    KV = []
    for x in wl.kv_full(w):
        x[rng.random(x.shape) < 0.002] = bad
        KV.append(torch.from_numpy(x).cuda())
    cfg = gpu_config(oracle_config(w, kind=kind))
    chunk, steps = iq.allocate_cache(cfg), iq.allocate_cache(cfg)
    iq.innerq_quantize_append(chunk, *KV)
    for t in range(n):
        iq.innerq_quantize_append(steps, *(x[:, :, t:t + 1].contiguous() for x in KV))
    for name, buf in chunk.buffers.items():
        if buf is not None and not name.endswith("recent"):               # (a ring's spare slots hold older tokens)
            assert torch.equal(buf, steps.buffers[name]), name


@pytest.mark.parametrize("kind,bits,heads,chunks", [
    (orc.KIND_INNER, 4, 1, (150, 64, 200)), (orc.KIND_INNER, 3, 9, (200, 70, 131)), (orc.KIND_OUTER, 2, 5, (133, 100, 300)),
    (orc.KIND_INNER, 2, 64, (150, 1024, 1025)),           # 131072 groups and 128 more: owners, then two launches
    (orc.KIND_INNER, 3, 40, (150, 200, 131)), (orc.KIND_OUTER, 4, 48, (133, 100, 300)),                     # owners: 8192 groups and more
])
def test_owners_of_hybrid_groups_of_64(env, kind, bits, heads, chunks):
    torch, iq = env
    n = sum(chunks)
    w = wl.Workload("b", 1, heads, heads, 128, n, bits, 64, 4, 64, k_mode=orc.HYBRID, v_mode=orc.HYBRID)
    o = oracle_config(w, kind=kind)
    rng = np.random.default_rng(n + bits)
    K, V = (rng.standard_normal((1, heads, n, 128)).astype(np.float16) for _ in range(2))
    g = iq.allocate_cache(gpu_config(o))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    at = 0
    for c in chunks:
        iq.innerq_quantize_append(g, dev(K[:, :, at:at + c]), dev(V[:, :, at:at + c]))
        at += c
    assert_cache_equal(g, orc.cache_init_prefill(o, K, V), o)


@pytest.mark.parametrize("kind,bits,group,modes,heads", [
    (orc.KIND_INNER, 2, 32, (orc.HYBRID, orc.HYBRID), 3), (orc.KIND_INNER, 3, 32, (orc.SYM, orc.HYBRID), 192), (orc.KIND_INNER, 4, 64, (orc.HYBRID, orc.ASYM), 64),
    (orc.KIND_INNER, 2, 64, (orc.HYBRID, orc.HYBRID), 256),
    (orc.KIND_INNER, 3, 64, (orc.HYBRID, orc.HYBRID), 257), (orc.KIND_INNER, 2, 32, (orc.HYBRID, orc.SYM), 65),       # beyond the lines: a group a lane
    (orc.KIND_INNER, 3, 32, (orc.SYM, orc.HYBRID), 193), (orc.KIND_INNER, 3, 32, (orc.SYM, orc.HYBRID), 256),
    (orc.KIND_OUTER, 4, 32, (orc.HYBRID, orc.SYM), 5), (orc.KIND_OUTER, 3, 64, (orc.ASYM, orc.HYBRID), 2),
])
@pytest.mark.parametrize("dist", ["normal", "ties", "denormal"])
def test_channel_groups_over_eight_lanes(env, kind, bits, group, modes, heads, dist):
    """Short appends and steps in which per-channel groups leave their ring: the groups spread over eight lanes, and in one."""
    torch, iq = env
    chunks = (4 + 32 + group - 1, 1, 2, group, 1)            # up to a group short of one token, then one at a time and a group at once
    n = sum(chunks)
    w = wl.Workload("c", 1, heads, heads, 128, n, bits, group, 4, 32, k_mode=modes[0], v_mode=modes[1])
    o = oracle_config(w, kind=kind)
    rng = np.random.default_rng(n + bits)
    K, V = (values(rng, (1, heads, n, 128), dist) for _ in range(2))
    inv = rng.uniform(0.3, 1.0, (heads, 128)).astype(np.float32)
    g = iq.allocate_cache(gpu_config(o))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    at = 0
    for c in chunks:
        iq.innerq_quantize_append(g, dev(K[:, :, at:at + c]), dev(V[:, :, at:at + c]), dev(inv))
        at += c
    assert_cache_equal(g, orc.cache_init_prefill(o, K, V, k_inv_norm=inv), o)


@pytest.mark.parametrize("kind,bits,group,mode,heads,recent,chunks", [
    (orc.KIND_INNER, 2, 64, orc.ASYM, 1, 64, (150, 64, 200)), (orc.KIND_INNER, 3, 64, orc.SYM, 9, 64, (200, 70, 131)), (orc.KIND_OUTER, 4, 64, orc.ASYM, 5, 64, (133, 100, 300)),
    (orc.KIND_INNER, 2, 64, orc.SYM, 64, 16, (150, 2048, 2049)),          # 262144 groups and 128 more: owners, then two launches
    (orc.KIND_INNER, 4, 64, orc.ASYM, 2, 384, (700, 320, 447, 64)), (orc.KIND_OUTER, 3, 64, orc.SYM, 1, 300, (600, 400)),       # five groups of a ring and more
    (orc.KIND_INNER, 2, 32, orc.HYBRID, 3, 416, (800, 288, 300, 447)), (orc.KIND_OUTER, 3, 32, orc.HYBRID, 1, 280, (600, 400)),   # nine and more, at G = 32
    (orc.KIND_INNER, 4, 32, orc.ASYM, 2, 256, (300, 287, 513, 40)),
])
@pytest.mark.parametrize("paged", [False, True])
def test_owners_with_a_pair_of_channels_a_lane(env, kind, bits, group, mode, heads, recent, chunks, paged):
    """New groups of one variant at G = 64, and rings with more groups than one round of a work-group takes; the same bytes in a paged store."""
    torch, iq = env
    n = sum(chunks)
    w = wl.Workload("p", 1, heads, heads, 128, n, bits, group, 4, recent, k_mode=mode, v_mode=mode)
    cap = -(-n // 64) * 64
    o = oracle_config(w, kind=kind, capacity=cap)
    rng = np.random.default_rng(n + bits)
    K, V = values(rng, (1, heads, n, 128), "normal"), values(rng, (1, heads, n, 128), "ties")
    inv = rng.uniform(0.3, 1.0, (heads, 128)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    pages, caches = cap // 64, [iq.allocate_cache(gpu_config(o))]
    if paged:
        cfg = gpu_config(o)
        cfg.page_pool_pages = pages
        caches.append(iq.allocate_cache(cfg, page_table=torch.arange(pages - 1, -1, -1, dtype=torch.int32, device="cuda")[None].contiguous()))
    for g in caches:
        at = 0
        for c in chunks:
            iq.innerq_quantize_append(g, dev(K[:, :, at:at + c]), dev(V[:, :, at:at + c]), dev(inv))
            at += c
    if not paged:
        assert_cache_equal(caches[0], orc.cache_init_prefill(o, K, V, k_inv_norm=inv), o)
        return
    # page by page (64 rows of every head): the pages lie in the pool in reverse
    for name in ("k_codes", "k_scales", "k_zeros", "v_codes", "v_scales", "v_zeros"):
        a, b = (c.buffers[name] for c in caches)
        if a is None:
            continue
        rows = a.view(heads, pages, -1)
        got = b.view(pages, heads, -1).flip(0).permute(1, 0, 2)
        full = min(orc.partition(o, x, n)[1] for x in "kv") // 64                # (whole pages of quantised rows)
        assert torch.equal(rows[:, :full], got[:, :full]), name
