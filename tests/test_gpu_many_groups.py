"""Networks with as many groups as the planning launch still makes the rebuild plans for, one more (they get a launch of
their own) and many more: one count's step and portfolios."""
import numpy as np
import pytest

from paper_2309_06973_amd import synth
from test_gpu_single_pass import check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", [640, 641, 1500])
@pytest.mark.parametrize("k", [1, 2, 5])
def test_step(groups, k):
    spec = synth.chain_spec([6] * (groups - 2), k=1, in_ch=3)
    assert len(spec.groups) == groups
    rng = np.random.Generator(np.random.Philox(groups + k))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    n = spec.n_prunable
    check_step(spec, w, v, [n // 3, n // 2, n // 5, (3 * n) // 5, n // 4][:k])
