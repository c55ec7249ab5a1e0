"""The wait in the multi-pass select's last launch has a bound.  With a bound of a look or a few, set by the host, blocks
leave while others still read: every call ends, a record is the right one or removes nothing, a call that reads records back
says so, and the next call with the usual bound is right everywhere."""
import numpy as np
import pytest
import torch

from paper_2309_06973_amd import shifter as S
from paper_2309_06973_amd import synth

pytestmark = pytest.mark.gpu

N = 3_000_001                                   # all equal: three stages, the later two in the last launch


def fields(raw, k):
    return [tuple(getattr(S.Threshold.from_buffer_copy(raw, i * S.THRESHOLD_BYTES), f)
                  for f in ("cut", "t_key", "g_cut", "n_prune", "n_less", "n_equal")) for i in range(k)]


@pytest.mark.parametrize("k", [1, 20, 64])
def test_flat_run(k):
    half = int(np.float32(0.5).view(np.uint32))
    w = torch.where(torch.arange(N, device="cuda") % 3 == 0, -0.5, 0.5)
    ps = [0 if i == 3 else 1 + (i * 7919 * 131071) % N for i in range(k)]
    right = [(0, 0, 2 ** 64 - 1, 0, 0, 0) if p == 0 else ((half << 32 | p - 1) + 1, half, p - 1, p, 0, N) for p in ps]
    none = [(0, 0, 2 ** 64 - 1, p, 0, 0) for p in ps]
    ctx = S.shifter_create(0, torch.cuda.current_stream().cuda_stream)
    try:
        gave_up = 0
        for polls in (1, 1, 2, 5, 20, 100, 0):
            S.shifter_set_select_polls(ctx, polls)
            thr = torch.full((k * S.THRESHOLD_BYTES,), 0xAB, dtype=torch.uint8, device="cuda")
            S.shifter_global_threshold_static(ctx, w, N, ps, thr)
            got = fields(thr.cpu().numpy().tobytes(), k)
            assert all(g in (r, e) for g, r, e in zip(got, right, none))
            gave_up += got != right
        assert got == right and gave_up > 0
    finally:
        S.shifter_destroy(ctx)


def test_calls_that_read_back():
    n = N
    model = S.shifter_model_create([synth.TensorDesc(0, 1, n, 1, 1, 1, 1, 0, 1)], [], [synth.GroupDesc(n, 1), synth.GroupDesc(1, 1)])
    w = torch.full((n + 16,), 0.25, device="cuda")
    ps = [n // 3, n // 2, 5]
    ctx = S.shifter_create(0, torch.cuda.current_stream().cuda_stream)
    try:
        S.shifter_set_select_path(ctx, 1)
        thr = torch.zeros(3 * S.THRESHOLD_BYTES, dtype=torch.uint8, device="cuda")
        codes = set()
        for polls in (1, 1, 1, 0):
            S.shifter_set_select_polls(ctx, polls)
            try:
                recs = S.shifter_global_threshold(ctx, model, w, ps, thr, sync=True)
                assert [r.g_cut for r in recs] == [p - 1 for p in ps]
                codes.add(0)
            except S.ShifterError as e:
                assert polls == 1
                codes.add(e.code)
            S.shifter_global_threshold_begin(ctx, model, w, ps, thr)
            try:
                recs, _ = S.shifter_global_threshold_end(ctx)
                assert [r.g_cut for r in recs] == [p - 1 for p in ps]
            except S.ShifterError as e:
                assert polls == 1
                codes.add(e.code)
        assert codes == {0, S.SHIFTER_ERR_INTERNAL}
    finally:
        S.shifter_model_destroy(model)
        S.shifter_destroy(ctx)
