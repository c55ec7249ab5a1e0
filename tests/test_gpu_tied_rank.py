"""Ranks among many weights of one magnitude that the sampled pass still ranks itself: on both sides of the number from which it
goes by the upper bits of the indices first, the first and the last of them, ties all over the arena and side by side."""
import numpy as np
import pytest

from oracle import shifter_oracle as O
from tests.test_gpu_single_pass import check_step, network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tied", [256, 257, 700, 1024])
@pytest.mark.parametrize("where", ["spread", "start", "end"])
@pytest.mark.parametrize("k", [1, 3])
def test_rank(n_tied, where, k):
    spec, w, v, rng = network([19, 101, 103], n_tied)
    near = (np.abs(w) > 0.7) & (np.abs(w) < 0.8)
    w[near] *= 2.0
    ranked = np.concatenate([np.arange(t.offset, t.offset + t.numel) for t in spec.tensors if t.prunable])
    at = {"spread": rng.choice(ranked, n_tied, replace=False), "start": ranked[:n_tied], "end": ranked[-n_tied:]}[where]
    w[at] = np.where(rng.random(n_tied) < 0.5, 0.75, -0.75).astype(np.float32)
    less = int((np.abs(O.gather_prunable(w, spec.tensors)) < 0.75).sum())
    for nth in (1, n_tied // 2, n_tied):
        check_step(spec, w, v, [less + nth, less // 2, less // 3][:k])
