"""The ranking of a step on a cache-sized arena where it changes kind: as many equal weights as a
step ranks itself and one more, a single count among ties, a window that no list holds (the step
is redone), network sizes around the tiles and blocks of the histogram kernels, NaN."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import shifter as S
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


def network(widths, seed, in_ch=3):
    spec = synth.chain_spec(widths, in_ch=in_ch)
    rng = np.random.Generator(np.random.Philox(seed))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    return spec, w, v, rng


def check_step(spec, w, v, ps, path=None, calls=2):
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    a = np.abs(O.gather_prunable(w, spec.tensors))
    pl = Pipeline(spec, w, v)
    try:
        k = len(ps)
        if k > 1:
            pl.enable_batch(k)
        for _ in range(calls):                   # the second call finds what the first one left
            recs, (rc, ot, ov, ew, ev) = pl.step(ps)
            torch.cuda.synchronize()
            if path:
                assert S.shifter_get_select_stats(pl.ctx)["path"] == path
            for i, (p, rec, ref) in enumerate(zip(ps, recs, refs)):
                assert rec.n_prune == p
                if p == 0:
                    assert rec.cut == 0
                    continue
                t = a[ref.sel.thr_index]
                assert (rec.g_cut, rec.n_less, rec.n_equal) == (ref.sel.thr_index, int((a < t).sum()), int((a == t).sum()))
                if k > 1:
                    mask = pl.b_mask[i * pl.m_stride:i * pl.m_stride + a.size]
                    out = pl.b_w_out[i * pl.cap_w:i * pl.cap_w + ew[i]]
                else:
                    mask, out = pl.d_mask[:a.size], pl.d_w_out[:ew[0]]
                assert np.array_equal(mask.cpu().numpy(), ref.mask)
                assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.compacted.w.view(np.uint32))
    finally:
        pl.close()


# path 1: the step ranks by itself; 2: it is redone
@pytest.mark.parametrize("n_tied,k,path", [(1000, 3, 1), (1024, 3, 1), (1025, 3, 2), (1025, 1, 1), (30000, 1, 1)])
def test_ties(n_tied, k, path):
    spec, w, v, rng = network([19, 101, 103], n_tied)
    w[w == 0.75] = 0.76
    at = rng.choice(w.size, n_tied, replace=False)
    w[at] = np.where(rng.random(n_tied) < 0.5, 0.75, -0.75).astype(np.float32)
    less = int((np.abs(w) < 0.75).sum())
    check_step(spec, w, v, [less + n_tied // 2] + [less // 2, 0][:k - 1], path)


def test_a_window_that_no_list_holds_is_redone():
    spec, w, v, _ = network([64, 512, 256], 7)           # 1.47 M weights
    w[:] = np.where(w > 0, 0.25, -0.25)
    check_step(spec, w, v, [w.size // 3], path=2)


# 1, a few and many tiles; ragged and whole ones; fewer weights than a block has threads
@pytest.mark.parametrize("widths,in_ch", [([2], 1), ([5, 3], 3), ([64, 64], 64), ([16, 256, 16], 16), ([91, 187], 7)])
@pytest.mark.parametrize("k", [1, 5])
def test_sizes(widths, in_ch, k):
    spec, w, v, _ = network(widths, sum(widths), in_ch)
    n = spec.n_prunable
    check_step(spec, w, v, [n // 2, n, 1, 0, (9 * n) // 10][:k])


def test_nan_is_reported_once():
    spec, w, v, _ = network([16, 32], 3)
    pl = Pipeline(spec, w, v)
    try:
        pl.d_w[7] = float("nan")
        with pytest.raises(S.ShifterError) as e:
            pl.step([spec.n_prunable // 2])
        assert e.value.code == S.SHIFTER_ERR_NONFINITE
        pl.step([0])                                     # nothing is ranked
        pl.d_w[7] = 1.0
        pl.step([spec.n_prunable // 2])
    finally:
        pl.close()
