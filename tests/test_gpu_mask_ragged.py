"""The batched mask pass on tensors that end one to three weights past a group of four, at, before and
behind the edge of a tile of 4096, with kernels of 1, 4 and 9 weights: masks, sparse arenas and flags."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


# second layer: 5, 6, 7, 4095, 4096, 4097, 4098 and 8191 weights with 1x1 kernels, more with larger ones
@pytest.mark.parametrize("widths", [[1, 5], [2, 3], [1, 7], [13, 315], [64, 64], [17, 241], [6, 683], [1, 8191]])
@pytest.mark.parametrize("kernel", [1, 2, 3])
@pytest.mark.parametrize("arenas", [True, False])
def test_mask_and_flags(widths, kernel, arenas):
    spec = synth.chain_spec(widths, k=kernel, in_ch=3)
    rng = np.random.Generator(np.random.Philox(sum(widths) + kernel))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    w[rng.random(w.size) < 0.2] = 0.0
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    n = spec.n_prunable
    ps = [0, n // 5, n // 2, (9 * n) // 10, n]
    refs = O.prune_and_compact(w, v, spec.tensors, spec.vecs, spec.groups, ps)
    pl = Pipeline(spec, w, v)
    try:
        pl.enable_batch(len(ps))
        pl.step(ps, sparse_arenas=arenas)
        torch.cuda.synchronize()
        outs, ins = sum(t.out_ch for t in spec.tensors), sum(t.in_ch for t in spec.tensors)
        for i, ref in enumerate(refs):
            assert np.array_equal(pl.b_mask[i * pl.m_stride:i * pl.m_stride + n].cpu().numpy(), ref.mask)
            if arenas:
                got = pl.b_w_sparse[i * pl.w_stride:i * pl.w_stride + w.size].cpu().numpy()
                assert np.array_equal(got.view(np.uint32), ref.w_sparse.view(np.uint32))
            assert np.array_equal(pl.b_out_alive[i * outs:(i + 1) * outs].cpu().numpy(), np.concatenate(ref.out_alive))
            assert np.array_equal(pl.b_in_alive[i * ins:(i + 1) * ins].cpu().numpy(), np.concatenate(ref.in_alive))
    finally:
        pl.close()
