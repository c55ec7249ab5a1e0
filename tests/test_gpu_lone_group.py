"""Groups that no tensor writes or reads, with and without vectors, pinned and not: one count's step and portfolios
plan them like the oracle (a pinned one stays whole, the other keeps nothing)."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pinned", [1, 0])
@pytest.mark.parametrize("vecs", [0, 2])
@pytest.mark.parametrize("k", [1, 2, 20])
def test_step(pinned, vecs, k):
    spec = synth.chain_spec([24, 40], in_ch=3)
    spec.groups.append(synth.GroupDesc(70, pinned))
    for _ in range(vecs):
        spec.vecs.append(synth.VecDesc(spec.v_elems, 70, len(spec.groups) - 1))
        spec.v_elems += 70
    rng = np.random.Generator(np.random.Philox(k + vecs))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    v = rng.standard_normal(spec.v_elems).astype(np.float32)
    n = spec.n_prunable
    ps = [n // 2] if k == 1 else [n // 3 + (n // 2) * i // (k - 1) for i in range(k)]
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    pl = Pipeline(spec, w, v)
    try:
        if k > 1:
            pl.enable_batch(k)
        for _ in range(2):
            recs, (rc, ot, ov, ew, ev) = pl.step(ps)
            torch.cuda.synchronize()
            g = len(spec.groups)
            widths = (pl.b_new_width if k > 1 else pl.d_new_width).cpu().numpy().reshape(k, g)
            w_out, v_out = (pl.b_w_out, pl.b_vecs_out) if k > 1 else (pl.d_w_out, pl.d_vecs_out)
            cap_w, cap_v = (pl.cap_w, pl.cap_v) if k > 1 else (0, 0)
            ew, ev = np.atleast_1d(ew), np.atleast_1d(ev)
            for i, ref in enumerate(refs):
                assert np.array_equal(widths[i], ref.plan.new_width)
                assert widths[i][-1] == (70 if pinned else 0)
                assert (ew[i], ev[i]) == (ref.compacted.w.size, ref.compacted.v.size)
                out = w_out[i * cap_w:i * cap_w + ref.compacted.w.size].cpu().numpy()
                assert np.array_equal(out.view(np.uint32), ref.compacted.w.view(np.uint32))
                out = v_out[i * cap_v:i * cap_v + ref.compacted.v.size].cpu().numpy()
                assert np.array_equal(out.view(np.uint32), ref.compacted.v.view(np.uint32))
    finally:
        pl.close()
