"""The multi-pass select at the sizes where its windows change kind: runs of exactly a list's room
and beyond, runs of equal weights that only their index separates, weights outside
the binned range, weights sorted by size (one block meets a whole window), more ranks than
windows.  Every record against the counting definition on one stable sort."""
import numpy as np
import pytest
import torch

from paper_2309_06973_amd import shifter as S

pytestmark = pytest.mark.gpu

N = 600_011


def values(kind, n):
    rng = np.random.Generator(np.random.Philox(n + len(kind)))
    z = rng.standard_normal(n).astype(np.float32)
    if kind == "gauss":
        return z
    if kind == "equal":
        return np.where(z > 0, 0.5, -0.5).astype(np.float32)
    if kind == "half_zero":
        return np.where(rng.random(n) < 0.5, 0.0, z).astype(np.float32)
    if kind == "sorted":
        return np.sort(z)[::-1].copy()
    if kind == "half_precision":
        return z.astype(np.float16).astype(np.float32)
    if kind == "far_out":           # below, inside and above the 64 binades that are binned finely
        return (z * np.exp2(rng.integers(-140, 120, n).astype(np.float32))).astype(np.float32)
    raise ValueError(kind)


# a list has room for 2^19 / K pairs, 524288 of one rank and 8192 of each of 64; beyond 65536 pairs it is
# taken only by the last stage
@pytest.mark.parametrize("kind", ["gauss", "equal", "half_zero", "sorted", "half_precision", "far_out"])
@pytest.mark.parametrize("n,k", [(1, 1), (4095, 3), (4097, 2), (8193, 64), (524_288, 1), (524_289, 1), (N, 1), (N, 7),
                                 (N, 64)])
def test_records_by_counting(kind, n, k):
    w = values(kind, n)
    a = np.abs(w)
    order = np.argsort(a, kind="stable")
    ps = [0, 1, n, n // 2, (n + 1) // 2] + [(i * 7919 * 131) % (n + 1) for i in range(k)]
    ps = ps[:k] if k > 1 else [n // 2 + 1]
    ctx = S.shifter_create(0, torch.cuda.current_stream().cuda_stream)
    try:
        d_w = torch.from_numpy(w).cuda()
        d_thr = torch.zeros(len(ps) * S.THRESHOLD_BYTES, dtype=torch.uint8, device="cuda")
        for _ in range(2):                       # the second call finds what the first one left
            S.shifter_global_threshold_static(ctx, d_w, n, ps, d_thr)
        raw = d_thr.cpu().numpy().tobytes()
        sorted_a = a[order]
        for i, p in enumerate(ps):
            rec = S.Threshold.from_buffer_copy(raw, i * S.THRESHOLD_BYTES)
            assert rec.n_prune == p
            if p == 0:
                assert rec.cut == 0
                continue
            g = int(order[p - 1])
            key = int(a[g:g + 1].view(np.uint32)[0])
            assert (rec.t_key, rec.g_cut, rec.cut) == (key, g, ((key << 32) | g) + 1), (p, rec.t_key, rec.g_cut)
            lo, hi = np.searchsorted(sorted_a, a[g], "left"), np.searchsorted(sorted_a, a[g], "right")
            assert (rec.n_less, rec.n_equal) == (lo, hi - lo)
    finally:
        S.shifter_destroy(ctx)
