"""Inflating with one instance for all chunks and with three by segment size, on both sides of where
it changes: chunks of zeros, sparse, half-full and incompressible side by side, a ragged end."""
import pytest
import torch
import zlib

from paper_2309_06973_amd.pipeline import Codec

pytestmark = pytest.mark.gpu

CHUNK = 32768


@pytest.mark.parametrize("chunks,last", [(1, CHUNK), (3, 5), (1024, CHUNK), (1024, 1), (1025, 1), (1026, 4097)])
def test_round_trip(chunks, last):
    n = (chunks - 1) * CHUNK + last
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.randn((n + 3) // 4, generator=g, device="cuda")
    density = torch.rand((chunks, 1), generator=g, device="cuda")
    density = torch.where(torch.arange(chunks, device="cuda")[:, None] % 4 == 0, density.round(), density)   # 0 and 1 too
    w = torch.where(torch.rand(w.numel(), generator=g, device="cuda") < density.expand(-1, CHUNK // 4).reshape(-1)[:w.numel()],
                    w, torch.zeros_like(w))
    data = w.view(torch.uint8)[:n].clone()
    codec = Codec()
    package = codec.deflate(data)
    for _ in range(2):
        out = torch.full((n + 16,), 0xAA, dtype=torch.uint8, device="cuda")
        codec.inflate(package, out=out[:n])
        assert torch.equal(out[:n], data)
        assert (out[n:] == 0xAA).all()
    if chunks <= 3:
        raw = package.stream[:package.stream_bytes].cpu().numpy().tobytes()
        assert zlib.decompress(raw, wbits=-15) == data.cpu().numpy().tobytes()
