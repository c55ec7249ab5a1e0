"""A portfolio step that the sampled ranking cannot decide, because most magnitudes are one, and that is made again: its records and
rebuilt variants, to the ends that the call reports, against the oracle.  Kernels of 1 to 25 weights, ragged tiles, tensors
within one tile and over many, one of them not ranked, filters that no variant has and such of a weight or two."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import shifter as S
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,widths,ranked", [(3, [37, 91, 211, 131], True), (1, [130, 515, 700], True), (5, [33, 71, 129, 63], True),
                                                  (3, [60, 250, 301], False), (1, [1, 4100, 31, 700], True), (3, [260, 270, 300], True)])
@pytest.mark.parametrize("by_sampling", [0.2, 0.0])
def test_made_again(kernel, widths, ranked, by_sampling):
    spec = synth.chain_spec(widths, k=kernel, in_ch=3)
    if not ranked:
        spec.tensors[1].prunable = 0
    n = spec.n_prunable
    rng = np.random.Generator(np.random.Philox(spec.w_elems))
    w = np.where(rng.random(spec.w_elems) < 0.5, np.float32(-1), np.float32(1)).astype(np.float32)
    small = rng.random(spec.w_elems) < 2 * by_sampling        # what the first two ranks are found among
    w[small] = rng.uniform(0.01, 0.9, int(small.sum())).astype(np.float32)
    for t in spec.tensors:
        rows = w[t.offset:t.offset + t.numel].reshape(t.out_ch, -1)
        rows[rng.random(t.out_ch) < 0.1] = 0.0                # filters that no variant has
        few = np.flatnonzero(rng.random(t.out_ch) < 0.3)
        rows[few] *= rng.random((few.size, rows.shape[1])) < 2.0 / rows.shape[1]       # and such of a weight or two
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    zeros = sum(int((w[t.offset:t.offset + t.numel] == 0).sum()) for t in spec.tensors if t.prunable)
    small_n = sum(int(((np.abs(x) > 0) & (np.abs(x) < 1)).sum()) for x in (w[t.offset:t.offset + t.numel] for t in spec.tensors if t.prunable))
    tied = n - zeros - small_n
    ps = [zeros + small_n + int(tied * f) for f in (0.9, 0.3, 0.6)]
    if by_sampling:
        ps += [zeros + int(small_n * f) for f in (0.7, 0.4)]
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    pl = Pipeline(spec, w, v)
    try:
        pl.enable_batch(len(ps))
        for x in (pl.b_w_out, pl.b_vecs_out, pl.b_w_sparse):
            x.fill_(7.0)
        for x in (pl.b_mask, pl.b_out_alive, pl.b_in_alive):
            x.fill_(7)
        recs, (rc, ot, ov, ew, ev) = pl.step(ps)
        torch.cuda.synchronize()
        assert S.shifter_get_select_stats(pl.ctx)["path"] == 2
        bits = lambda x: np.ascontiguousarray(x).view(np.uint32)
        out_alive, in_alive = pl.b_out_alive.cpu().numpy(), pl.b_in_alive.cpu().numpy()
        so, si = out_alive.size // len(ps), in_alive.size // len(ps)
        a = np.abs(O.gather_prunable(w, spec.tensors))
        for k, ref in enumerate(refs):
            t = a[ref.sel.thr_index]
            assert (recs[k].g_cut, recs[k].n_less, recs[k].n_equal) == (ref.sel.thr_index, int((a < t).sum()), int((a == t).sum()))
            assert np.array_equal(pl.b_mask[k * pl.m_stride:k * pl.m_stride + n].cpu().numpy(), ref.mask)
            assert (ew[k], ev[k]) == (ref.compacted.w.size, ref.compacted.v.size)
            assert np.array_equal(bits(pl.b_w_out[k * pl.cap_w:k * pl.cap_w + ew[k]].cpu().numpy()), bits(ref.compacted.w))
            assert np.array_equal(bits(pl.b_vecs_out[k * pl.cap_v:k * pl.cap_v + ev[k]].cpu().numpy()), bits(ref.compacted.v))
            assert np.array_equal(bits(pl.b_w_sparse[k * pl.w_stride:k * pl.w_stride + spec.w_elems].cpu().numpy()), bits(ref.w_sparse))
            assert np.array_equal(out_alive[k * so:(k + 1) * so], np.concatenate(ref.out_alive))
            assert np.array_equal(in_alive[k * si:(k + 1) * si], np.concatenate(ref.in_alive))
    finally:
        pl.close()
