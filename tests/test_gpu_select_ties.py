"""The multi-pass select on weights that are equal in masses and on weights whose bin holds more
than a list: zeros of both signs beside values below the binned range, few distinct values (one
key to a bin), two keys to a bin, all weights in eight bins.  Every record against the
counting definition on one stable sort."""
import numpy as np
import pytest
import torch

from paper_2309_06973_amd import shifter as S

pytestmark = pytest.mark.gpu


def values(kind, n):
    rng = np.random.Generator(np.random.Philox(n + len(kind)))
    z = rng.standard_normal(n).astype(np.float32)
    if kind == "zeros":             # 95 % zeros, every other one negative; tiny values behind them
        z = np.where(rng.random(n) < 0.3, z * np.float32(2.0 ** -70), z).astype(np.float32)
        return np.where(rng.random(n) < 0.95, np.where(z > 0, 0.0, -0.0), z).astype(np.float32)
    if kind == "levels":
        return (np.round(z * 30) / 30).astype(np.float32)
    if kind == "two_keys":          # one bin, two keys, three quarters of the weights
        two = np.float32([0.75, np.nextafter(np.float32(0.75), np.float32(1))])[rng.integers(0, 2, n)]
        return np.where(rng.random(n) < 0.75, two, z).astype(np.float32)
    if kind == "eight_bins":        # no ties to speak of: 2^18 keys
        key = np.float32(0.75).view(np.uint32) + rng.integers(0, 1 << 18, n).astype(np.uint32)
        return np.where(z > 0, key.view(np.float32), -key.view(np.float32)).astype(np.float32)
    raise ValueError(kind)


# a list of up to 65536 pairs is ranked as it is; beyond, a window is split while a stage is left
@pytest.mark.parametrize("kind", ["zeros", "levels", "two_keys", "eight_bins"])
@pytest.mark.parametrize("n,k", [(257, 5), (65_536, 1), (65_537, 1), (262_144, 2), (400_003, 1), (1_000_003, 3), (1_000_003, 64),
                                 (2_500_000, 10)])
def test_records_by_counting(kind, n, k):
    w = values(kind, n)
    a = np.abs(w)
    order = np.argsort(a, kind="stable")
    zeros = int((a == 0).sum())
    # both sides of where the zeros end, the middle of the mass, then spread out
    ps = [n // 2, max(zeros, 1), min(zeros + 1, n), 1, n] + [(i * 7919 * 131) % n + 1 for i in range(k)]
    ps = ps[:k]
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
            g = int(order[p - 1])
            key = int(a[g:g + 1].view(np.uint32)[0])
            assert (rec.t_key, rec.g_cut, rec.cut) == (key, g, ((key << 32) | g) + 1), (p, rec.t_key, rec.g_cut)
            lo, hi = np.searchsorted(sorted_a, a[g], "left"), np.searchsorted(sorted_a, a[g], "right")
            assert (rec.n_less, rec.n_equal) == (lo, hi - lo)
    finally:
        S.shifter_destroy(ctx)
