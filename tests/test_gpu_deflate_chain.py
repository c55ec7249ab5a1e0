"""The encoder's chain words stay with the context from call to call: calls of growing and shrinking numbers of links, and a
recorded call that goes on with words the context has outgrown since.  Streams as from a context of their own."""
import pytest
import torch

from paper_2309_06973_amd.pipeline import Codec

pytestmark = pytest.mark.gpu

CHUNK = 32768


def data(chunks, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randn(chunks * CHUNK // 4, generator=g, device="cuda")
    return torch.where(torch.rand(w.numel(), generator=g, device="cuda") < 0.2, w, torch.zeros_like(w)).view(torch.uint8)


def same(a, b, size):
    assert torch.equal(a.stream[:size], b.stream[:size])
    assert torch.equal(a.seg_off, b.seg_off) and torch.equal(a.sub_bits, b.sub_bits) and torch.equal(a.sub_marks, b.sub_marks)


# 768 chunks take a link each, 769 and more share one between two; 1024 links are there from the start
@pytest.mark.parametrize("sizes", [[1, 2, 1, 1, 3, 2], [768, 1, 769, 5, 768, 768], [2047, 2049, 7, 2100, 4100, 2, 2049]])
def test_calls_of_many_sizes(sizes):
    codec = Codec()
    for i, chunks in enumerate(sizes):
        x = data(chunks, i)
        got = codec.deflate(x)
        ref = Codec().deflate(x)
        assert got.stream_bytes == ref.stream_bytes
        same(got, ref, got.stream_bytes)
        assert torch.equal(codec.inflate(got)[:x.numel()], x)


def test_recorded_call_and_growth():
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        codec = Codec()
        x = data(40, 1)
        package = codec.deflate(x)                                        # makes room
        size = package.stream_bytes
        out = torch.empty(size + 5 * 40 + x.numel(), dtype=torch.uint8, device="cuda")
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            recorded = codec.deflate(x, stream=out, sync=False)
        for i in range(4):
            x.copy_(data(40, 10 + i))
            out.zero_()
            graph.replay()
            stream.synchronize()
            ref = Codec().deflate(x)
            same(recorded, ref, ref.stream_bytes)
            codec.deflate(data([3, 3000, 1, 50][i], i))                  # the second one outgrows the words
        del graph
        stream.synchronize()
