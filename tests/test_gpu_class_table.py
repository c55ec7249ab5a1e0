"""The K-rank pass classifies a weight by a table of 4096 bins (16 binades) from the first rank's interval on,
or of all bins where the intervals span more: weights spread evenly over so many binades, on networks whose
tensors end in ragged tiles."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import shifter as S
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


# the first and the last of the ranks lie at 10 % and 97 % of the weights, so 0.87 of the binades apart; the
# bins end at 2^14, and the last one holds all that lies above
@pytest.mark.parametrize("low,high", [(-3, -2), (-20, -4), (-20, -2), (-20, -1.5), (-20, -1), (-20, 0), (-48, 12), (-75, -30), (10, 16),
                                      (-1, 15), (6, 15), (12, 15)])
@pytest.mark.parametrize("widths,k", [([37, 91, 64], 2), ([37, 91, 64], 20), ([32, 96, 128, 64], 32)])
def test_classes(low, high, widths, k):
    spec = synth.chain_spec(widths, in_ch=3)
    rng = np.random.Generator(np.random.Philox(k + int(10 * (high - low))))
    w = np.exp2(rng.uniform(low, high, spec.w_elems)) * rng.choice([-1.0, 1.0], spec.w_elems)
    w = w.astype(np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    n = spec.n_prunable
    ps = [int(n * (0.1 + 0.87 * i / (k - 1))) for i in range(k)]
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    a = np.abs(O.gather_prunable(w, spec.tensors))
    pl = Pipeline(spec, w, v)
    try:
        pl.enable_batch(k)
        recs, (rc, ot, ov, ew, ev) = pl.step(ps)
        torch.cuda.synchronize()
        # The pass decides, whatever the table's form.  But twenty ranks of 84 k weights in one binade share one interval, open
        # to infinity for the last of them (97 % lie within the margin of 1300 samples' end): its 256 bins are a binade
        # each, and one of them holds more than the list's 65536 pairs.
        alone = k == 20 and high - low == 1
        assert S.shifter_get_select_stats(pl.ctx)["path"] == (2 if alone else 1)
        for i, (rec, ref) in enumerate(zip(recs, refs)):
            t = a[ref.sel.thr_index]
            assert (rec.g_cut, rec.n_less, rec.n_equal) == (ref.sel.thr_index, int((a < t).sum()), int((a == t).sum()))
            mask = pl.b_mask[i * pl.m_stride:i * pl.m_stride + a.size]
            assert np.array_equal(mask.cpu().numpy(), ref.mask)
            out = pl.b_w_out[i * pl.cap_w:i * pl.cap_w + ew[i]]
            assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.compacted.w.view(np.uint32))
    finally:
        pl.close()
