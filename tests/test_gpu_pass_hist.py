"""One count's sampled pass around 256 tiles, up to which it counts the candidates' first histogram itself, on
continuous weights and on few distinct ones, with ragged tiles; and the finish whose blocks take up to four parts
of the candidates each."""
import numpy as np
import pytest

from paper_2309_06973_amd import synth
from test_gpu_single_pass import check_step

pytestmark = pytest.mark.gpu


# 1x1 kernels: tiles of the three layers (tiles of up to 512 weights go one weight a thread); 3 and 63 to 65 tiles: fewer blocks than the finish may have, and as many
@pytest.mark.parametrize("widths,tiles", [([8, 40], 3), ([256, 976], 63), ([256, 992], 64), ([256, 1008], 65), ([1024, 1012], 255),
                                          ([1024, 1016], 256), ([1024, 1017], 257), ([1024, 1020], 257)])
@pytest.mark.parametrize("levels", [0, 2000])
def test_step(widths, tiles, levels):
    spec = synth.chain_spec(widths, k=1, in_ch=3)
    assert sum((t.numel + 4095) // 4096 for t in spec.tensors) == tiles
    rng = np.random.Generator(np.random.Philox(sum(widths) + levels))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    if levels:                      # up to 210 of the million share a value: ties inside the second histogram
        w = (np.round(w * levels) / levels).astype(np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    check_step(spec, w, v, [(9 * spec.n_prunable) // 10], path=1)


# short tiles around 512 weights, up to which they go one weight a thread, in networks of up to 256 tiles and of more
@pytest.mark.parametrize("widths", [[16, 32], [27, 19], [16, 32] * 60, [27, 19] * 60, [16, 32] * 140, [27, 19] * 140, [7, 13] * 140])
@pytest.mark.parametrize("levels", [0, 2000])
def test_short_tiles(widths, levels):
    spec = synth.chain_spec(widths, k=1, in_ch=3)
    rng = np.random.Generator(np.random.Philox(sum(widths) + levels))
    w = rng.standard_normal(spec.w_elems, dtype=np.float32)
    if levels:
        w = (np.round(w * levels) / levels).astype(np.float32)
    v = rng.standard_normal(max(spec.v_elems, 4)).astype(np.float32)
    check_step(spec, w, v, [spec.n_prunable // 3], path=1)
