"""The encoder's chain words stay with the context from call to call: calls of growing and shrinking numbers of links, and
recorded calls, which have words of their own and go on when the context has outgrown its.  Streams as from a context of their own."""
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


# An eager call of either kind and of that size makes room for a recorded one (40 chunks: a link each; 900: one to two)
@pytest.mark.parametrize("chunks", [40, 900])
@pytest.mark.parametrize("first", ["inflate", "small buffer"])
def test_recorded_behind_another_call(first, chunks):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        x = data(chunks, 2)
        other = Codec()
        package = other.deflate(x)
        codec = Codec()
        codec.work = torch.empty_like(other.work)
        if first == "inflate":
            assert torch.equal(codec.inflate(package)[:x.numel()], x)
        else:
            codec.deflate(x, stream=torch.empty(package.stream_bytes, dtype=torch.uint8, device="cuda"))
        check_recorded(codec, other, stream, x, chunks)


# A recording of the mode in which it may allocate, in a context that has run nothing: what it leaves to be cleared is not taken
# for cleared by an eager call before the first replay
def test_recorded_first():
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        x = data(40, 3)
        other = Codec()
        codec = Codec()
        codec.work = torch.full_like(torch.empty(50 * (CHUNK + 64), dtype=torch.uint8, device="cuda"), 0xEE)
        check_recorded(codec, other, stream, x, 40, mode="relaxed")


# More than 1024 chunks: the decoder has a list of those whose segments are long, which a longer input outgrows
def test_recorded_list_and_growth():
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        x = data(1100, 4)
        codec, other = Codec(), Codec()
        package = other.deflate(x)
        back = torch.empty_like(x)
        codec.inflate(package, out=back)                                  # makes room
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            codec.inflate(package, out=back, sync=False)
        for i in range(3):
            y = data([2100, 4200, 5][i], 40 + i)
            assert torch.equal(codec.inflate(other.deflate(y))[:y.numel()], y)
            back.zero_()
            graph.replay()
            stream.synchronize()
            assert torch.equal(back, x)
        del graph
        stream.synchronize()


def check_recorded(codec, other, stream, x, chunks, mode="global"):
    out = torch.empty(x.numel() + 5 * chunks, dtype=torch.uint8, device="cuda")
    back = torch.empty_like(x)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode=mode):
        recorded = codec.deflate(x, stream=out, sync=False)
        codec.inflate(recorded, out=back, sync=False)
    for i in range(3):
        y = data([chunks, 3, 2500][i], 30 + i)                            # eager, before the first replay too
        got, ref = codec.deflate(y), other.deflate(y)
        same(got, ref, ref.stream_bytes)
        assert torch.equal(codec.inflate(got)[:y.numel()], y)
        x.copy_(data(chunks, 20 + i))
        out.zero_()
        graph.replay()
        stream.synchronize()
        ref = other.deflate(x)
        same(recorded, ref, ref.stream_bytes)
        assert torch.equal(back, x)
    del graph
    stream.synchronize()
