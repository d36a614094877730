"""Calls go to the caller's current stream, or to the one that is passed."""
import pytest

pytestmark = pytest.mark.gpu


def test_current_and_given_streams():
    import torch
    from paper_2602_23200_amd import binding as iq
    assert torch.cuda.is_available(), "these tests need the MI355X"
    side = torch.cuda.Stream()
    assert iq._stream(None) == (torch.cuda.current_stream().cuda_stream or None)
    with torch.cuda.stream(side):
        assert iq._stream(None) == side.cuda_stream and iq._stream(None)
    assert iq._stream(side) == side.cuda_stream
    # work is recorded where the stream says: a capture on the side stream takes the step, and its replay writes the output
    cfg = iq.make_config(1, 4, 1, 128, 4, 32, 4, 32, capacity_tokens=256)
    cache, ws = iq.allocate_cache(cfg), iq.allocate_workspace(cfg)
    gen = torch.Generator(device="cuda").manual_seed(3)
    k = torch.randn(1, 1, 100, 128, generator=gen, device="cuda").half()
    q = torch.randn(1, 4, 128, generator=gen, device="cuda").half()
    iq.innerq_quantize_append(cache, k, k)
    want, out = iq.innerq_decode_attention(cache, q, ws), torch.zeros(1, 4, 128, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        iq.innerq_decode_attention(cache, q, ws, out=out)
    assert not out.any()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
