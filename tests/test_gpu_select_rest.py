"""The multi-pass select's later stages, which share a launch: parts handed out to more and to fewer blocks than there
are, and the second stage in a launch of its own where a bin of spread-out weights is expected to outgrow a list
(n / 1536 beyond 2^19 / 32 pairs).  Every record by the counting definition."""
import pytest
import torch

from paper_2309_06973_amd import shifter as S

pytestmark = pytest.mark.gpu

EDGE = 1536 * (16384 + 1)


@pytest.mark.parametrize("kind,n,k,grid", [("normal", EDGE - 1, 32, 256), ("normal", EDGE, 32, 256), ("levels", EDGE, 32, 256),
                                           ("levels", 400_003, 3, 1), ("levels", 400_003, 3, 2), ("equal", 400_003, 1, 2),
                                           ("equal", 400_003, 20, 300), ("equal", 2_000_001, 40, 5)])
def test_later_stages(kind, n, k, grid):
    g = torch.Generator(device="cuda").manual_seed(n + k)
    w = torch.randn(n, generator=g, device="cuda")
    if kind == "levels":
        w = torch.round(w * 30) / 30
    elif kind == "equal":
        w = torch.where(w > 0, 0.5, -0.5)
    a = w.abs()
    ps = [1 + (i * 7919 * 131071) % n for i in range(k)]
    ctx = S.shifter_create(0, torch.cuda.current_stream().cuda_stream)
    try:
        S.shifter_set_select_grid(ctx, grid)
        thr = torch.zeros(k * S.THRESHOLD_BYTES, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            S.shifter_global_threshold_static(ctx, w, n, ps, thr)
        raw = thr.cpu().numpy().tobytes()
        for i, p in enumerate(ps):
            rec = S.Threshold.from_buffer_copy(raw, i * S.THRESHOLD_BYTES)
            key = torch.tensor([rec.t_key], dtype=torch.int32, device="cuda").view(torch.float32)
            at = torch.nonzero(a == key).flatten()
            assert (rec.n_prune, rec.n_less, rec.n_equal) == (p, int((a < key).sum()), at.numel())
            assert 0 < p - rec.n_less <= rec.n_equal and rec.g_cut == int(at[p - rec.n_less - 1])
            assert rec.cut == ((rec.t_key << 32) | rec.g_cut) + 1
    finally:
        S.shifter_destroy(ctx)
