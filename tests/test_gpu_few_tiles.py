"""A portfolio of twenty on networks of a few tiles of 4096 weights, fewer, as many as and more than a
candidate region has parts: the blocks that finish the ranking follow the number of tiles."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import shifter as S
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


# the last layer (10 classes) is a tile of its own
@pytest.mark.parametrize("widths", [[4], [16, 28], [32, 64, 96], [64, 96, 75], [64, 96, 79], [64, 96, 84], [64, 128, 96]])
@pytest.mark.parametrize("levels", [0, 40])
def test_portfolio_of_twenty(widths, levels):
    spec = synth.chain_spec(widths, in_ch=3)
    rng = np.random.Generator(np.random.Philox(sum(widths) + levels))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    if levels:
        w = (np.round(w * levels) / levels).astype(np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    ps = [int(spec.n_prunable * (1 - 0.88 ** (i + 1))) for i in range(20)]
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    pl = Pipeline(spec, w, v)
    try:
        pl.enable_batch(len(ps))
        for _ in range(2):
            recs, (rc, ot, ov, ew, ev) = pl.step(ps)
            torch.cuda.synchronize()
            for i, (rec, ref) in enumerate(zip(recs, refs)):
                assert rec.g_cut == ref.sel.thr_index
                out = pl.b_w_out[i * pl.cap_w:i * pl.cap_w + ew[i]].cpu().numpy()
                assert np.array_equal(out.view(np.uint32), ref.compacted.w.view(np.uint32))
    finally:
        pl.close()
