"""What a decoder's lane takes from its part of the segment: as many tokens as 128 bytes can make, one to each byte, parts
that start at every bit of a dword, matches that cover what several lanes write, and sub-chunks on either side of
where they are stored instead (49 literals of nine bits), read at any byte."""
import pytest
import torch
import zlib

from paper_2309_06973_amd.pipeline import Codec

pytestmark = pytest.mark.gpu


def data(kind, n):
    g = torch.Generator().manual_seed(n + len(kind))
    at = torch.arange(n)
    x = torch.randint(1, 144, (n,), generator=g, dtype=torch.uint8)       # a literal of eight bits each
    if kind == "eight":
        x = torch.where((at > 0) & (x == x.roll(1)), x ^ 1, x).clamp(1, 143)
    elif kind in ("coded", "stored"):                                     # 48 or 49 of nine bits in a sub-chunk
        x = torch.where(at % 512 < (48 if kind == "coded" else 49), torch.randint(144, 255, (n,), generator=g, dtype=torch.uint8), x)
    elif kind == "mixed":                                                 # every other sub-chunk stored, at any byte
        x = torch.where(((at // 512) % 2 == 0) & (at % 512 < 60 + at // 512 % 7), x | 0x90, x)
        x = torch.where((at // 512) % 8 == 3, torch.zeros_like(x), x)
    elif kind == "runs":                                                  # runs of 1 to 300 of one value, not only zero
        ends = torch.cumsum(torch.randint(1, 300, (n // 100 + 8,), generator=g), 0)
        x = (torch.searchsorted(ends, at, right=True) * 37 % 251).to(torch.uint8)
    return x


@pytest.mark.parametrize("kind", ["eight", "coded", "stored", "mixed", "runs"])
@pytest.mark.parametrize("n", [130, 511, 32768, 3 * 32768 + 1025, 1025 * 32768 + 77])
def test_lanes(kind, n):
    host = data(kind, n)
    x = host.cuda()
    codec = Codec()
    package = codec.deflate(x)
    out = torch.full((n + 16,), 0xAA, dtype=torch.uint8, device="cuda")
    codec.inflate(package, out=out[:n])
    assert torch.equal(out[:n], x)
    assert (out[n:] == 0xAA).all()
    if n <= 4 * 32768:
        raw = package.stream[:package.stream_bytes].cpu().numpy().tobytes()
        assert zlib.decompress(raw, wbits=-15) == host.numpy().tobytes()
