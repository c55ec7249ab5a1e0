"""Deflating with one chunk to a block and with two, on both sides of where it changes and with a last
block that is half empty: segments straight into the stream and segments by slots give the same
stream, offsets, side information and marks, and write nothing behind them."""
import pytest
import torch

from paper_2309_06973_amd import shifter as S

pytestmark = pytest.mark.gpu

CHUNK = S.SHIFTER_CODEC_CHUNK
SUBS = CHUNK // S.SHIFTER_CODEC_SUB


@pytest.mark.parametrize("chunks,last", [(1, 1), (767, CHUNK), (768, 7), (769, CHUNK), (769, 1), (770, CHUNK - 1), (771, 513)])
@pytest.mark.parametrize("zeros", [False, True])
def test_both_forms(chunks, last, zeros):
    n = (chunks - 1) * CHUNK + last
    g = torch.Generator(device="cuda").manual_seed(n)
    data = torch.zeros((n + 3) // 4, device="cuda")
    if not zeros:           # chunks of density 0 to 1 side by side, both ends among them
        density = torch.rand(chunks, generator=g, device="cuda")
        density[::5] = density[::5].round()
        keep = torch.rand(data.numel(), generator=g, device="cuda") < density.repeat_interleave(CHUNK // 4)[:data.numel()]
        data = torch.where(keep, torch.randn(data.numel(), generator=g, device="cuda"), data)
    data = data.view(torch.uint8)[:n].clone()
    n_chunks, work, bound = S.shifter_codec_layout(n)
    assert n_chunks == chunks
    d_work = torch.empty(work, dtype=torch.uint8, device="cuda")
    ctx = S.shifter_create(0, torch.cuda.current_stream().cuda_stream)
    got = []
    try:
        for cap in (bound, bound - 1):          # the stream cannot overflow; it could (but does not: zeros, or sparse chunks)
            full = lambda m, dtype, v: torch.full((m,), v, dtype=dtype, device="cuda")
            stream, off = full(bound + 64, torch.uint8, 0xAA), full(chunks + 9, torch.int64, -7)
            bits, marks = full((chunks + 2) * SUBS, torch.int16, -7), full((chunks + 2) * SUBS, torch.int64, -7)
            if cap < bound and chunks == 1:
                continue                        # a single byte is stored and takes all of the bound
            size = S.shifter_deflate(ctx, data, n, d_work, stream[:cap], off, bits, marks)
            assert (stream[size:] == 0xAA).all() and (off[chunks + 1:] == -7).all()
            assert (bits[chunks * SUBS:] == -7).all() and (marks[chunks * SUBS:] == -7).all()
            assert int(off[chunks]) == size
            got.append((size, stream, off, bits, marks))
        for other in got[1:]:
            assert other[0] == got[0][0]
            assert all(torch.equal(a, b) for a, b in zip(other[1:], got[0][1:]))
        size, stream, off, bits, marks = got[0]
        out = torch.full((n + 16,), 0x55, dtype=torch.uint8, device="cuda")
        S.shifter_inflate(ctx, stream, size, off, bits, marks, n, out)
        assert torch.equal(out[:n], data) and (out[n:] == 0x55).all()
    finally:
        S.shifter_destroy(ctx)
