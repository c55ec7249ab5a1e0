"""A portfolio step that the sampled ranking cannot decide, because most magnitudes are one: the pass that is made on the records as they
are leaves levels alone, and what its rebuild wrote stays behind the ends of the variants made again.  That is compared with the
oracle's rebuild by such levels: kernels of 1 to 25 weights, ragged tiles, tensors within one tile and over many, one of them not ranked."""
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
def test_first_attempt(kernel, widths, ranked, by_sampling):
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
    K = len(ps)
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    found = [k >= 3 for k in range(K)]
    kept = [refs[k].w_sparse if found[k] else w for k in range(K)]
    count = sum((x != 0).astype(np.int32) for x in kept)      # variants that keep a weight; none keeps a zero
    level = [count[t.offset:t.offset + t.numel].reshape(t.out_ch, -1).max(axis=1) for t in spec.tensors]
    first = []
    for k in range(K):
        pos = sum(p < ps[k] for p in ps)
        plan = O.propagate_groups(spec.tensors, spec.groups, [(x > pos).astype(np.uint8) for x in level])
        first.append(O.compact(kept[k], v, spec.tensors, spec.vecs, plan).w)
    pl = Pipeline(spec, w, v)
    try:
        pl.enable_batch(K)
        pl.b_w_out.fill_(7.0)
        _, (rc, ot, ov, ew, ev) = pl.step(ps)
        torch.cuda.synchronize()
        assert S.shifter_get_select_stats(pl.ctx)["path"] == 2
        compared = 0
        for k, ref in enumerate(refs):
            assert ew[k] == ref.compacted.w.size
            got = pl.b_w_out[k * pl.cap_w:k * pl.cap_w + max(ew[k], first[k].size)].cpu().numpy().view(np.uint32)
            assert np.array_equal(got[:ew[k]], ref.compacted.w.view(np.uint32))
            assert np.array_equal(got[ew[k]:], first[k][ew[k]:].view(np.uint32))
            compared += got.size - ew[k]
        assert compared > 0
    finally:
        pl.close()
