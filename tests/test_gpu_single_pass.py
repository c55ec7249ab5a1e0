"""The sampled single pass where its launches change form: sampled by one block or by several, a
candidate list that fits the LDS of the block that ends last or not, ties around what it ranks."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import shifter as S
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


def network(widths, seed):
    spec = synth.chain_spec(widths, in_ch=3)
    rng = np.random.Generator(np.random.Philox(seed))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    return spec, w, v, rng


def check_step(spec, w, v, ps, path=1):
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    a = np.abs(O.gather_prunable(w, spec.tensors))
    pl = Pipeline(spec, w, v)
    try:
        k = len(ps)
        if k > 1:
            pl.enable_batch(k)
        for _ in range(2):                       # the second call finds what the first one left
            recs, (rc, ot, ov, ew, ev) = pl.step(ps)
            torch.cuda.synchronize()
            assert S.shifter_get_select_stats(pl.ctx)["path"] == path
            for i, (rec, ref) in enumerate(zip(recs, refs)):
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


# 0.2, 2.05 (one block samples up to 512 tiles of 4096 weights) and 2.2 M weights
@pytest.mark.parametrize("widths", [[64, 128, 96], [64, 410, 480], [64, 420, 500]])
@pytest.mark.parametrize("k", [1, 4])
def test_sampled_by_one_block_and_by_several(widths, k):
    spec, w, v, _ = network(widths, sum(widths))
    n = spec.n_prunable
    check_step(spec, w, v, [n // 2, n // 5, (9 * n) // 10, n // 3][:k])


# all 1.47 M weights on the 2^15 keys of one sample bin: 5700 of them in the bin of the candidates'
# histogram that holds the threshold, 45 to a key
@pytest.mark.parametrize("k", [1, 3])
def test_a_list_beyond_the_lds(k):
    spec, w, v, rng = network([64, 512, 256], 11)
    keys = np.float32(0.75).view(np.uint32) + rng.integers(0, 1 << 15, w.size).astype(np.uint32)
    w = np.where(w < 0, -keys.view(np.float32), keys.view(np.float32)).astype(np.float32)
    n = spec.n_prunable
    check_step(spec, w, v, [n // 2, n // 3, (4 * n) // 5][:k])


# a threshold that 1024 weights share is ranked by the pass, one that 1025 share is not
@pytest.mark.parametrize("n_tied,path", [(1024, 1), (1025, 2)])
@pytest.mark.parametrize("k", [1, 3])
def test_ties(n_tied, path, k):
    spec, w, v, rng = network([19, 101, 103], n_tied)
    w[w == 0.75] = 0.76
    w[w == -0.75] = 0.76
    near = (np.abs(w) > 0.7) & (np.abs(w) < 0.8)
    w[near] *= 2.0
    at = rng.choice(w.size, n_tied, replace=False)
    w[at] = np.where(rng.random(n_tied) < 0.5, 0.75, -0.75).astype(np.float32)
    less = int((np.abs(O.gather_prunable(w, spec.tensors)) < 0.75).sum())
    tied = int((np.abs(O.gather_prunable(w, spec.tensors)) == 0.75).sum())
    assert tied == n_tied
    check_step(spec, w, v, [less + n_tied // 2, less // 2, less // 3][:k], path)
