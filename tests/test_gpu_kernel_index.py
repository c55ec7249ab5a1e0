"""The kernel-level zero index where kernels and tiles of 4096 weights do not line up: every byte is
written, into a buffer that holds anything, also for kernels that span tiles."""
import numpy as np
import pytest
import torch

from oracle import shifter_oracle as O
from paper_2309_06973_amd import synth
from paper_2309_06973_amd.pipeline import Pipeline

pytestmark = pytest.mark.gpu


# 1 x 1; ragged and whole tiles of 3 x 3 and 7 x 7; 64 x 64 = one tile; 65 x 65 and 95 x 95, more than one
# and more than two tiles
@pytest.mark.parametrize("k,widths", [(1, [64, 64, 130]), (3, [1, 2]), (3, [64, 64, 77]), (7, [16, 64, 33]), (64, [2, 3]),
                                      (65, [2, 3, 1]), (95, [2, 2])])
@pytest.mark.parametrize("kept", [0.002, 0.3])
def test_every_byte(k, widths, kept):
    spec = synth.chain_spec(widths, k=k)
    rng = np.random.Generator(np.random.Philox(k))
    w = np.where(rng.random(spec.w_elems) < kept, rng.standard_normal(spec.w_elems), 0.0).astype(np.float32)
    for t in spec.tensors:                        # a kernel whose only non-zero is its first or its last weight
        kk = t.kh * t.kw
        flat = w[t.offset:t.offset + t.numel].reshape(-1, kk)
        flat[::3] = 0.0
        flat[::6, 0] = -0.5
        flat[3::6, -1] = 0.5
    pl = Pipeline(spec, w, np.zeros(max(spec.v_elems, 4), dtype=np.float32))
    try:
        src = torch.from_numpy(w).cuda()
        pl.d_kernel_nz = torch.full((max(pl.model.sum_kernels, 16) + 64,), 0xAA, dtype=torch.uint8, device="cuda")
        pl.kernel_scan(src=src)
        got = pl.d_kernel_nz.cpu().numpy()
        want = np.concatenate([x.reshape(-1) for x in O.kernel_scan(w, spec.tensors)])
        assert want.size == pl.model.sum_kernels
        assert np.array_equal(got[:want.size], want)
        assert (got[want.size:] == 0xAA).all()
    finally:
        pl.close()
