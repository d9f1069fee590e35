"""One sample's inter-bin MI on both sides of the size up to which the gradient
kernel finalizes the sample itself (chunk partials of 4096 doubles: chunks of 32
tokens x (2 E + 2)), against the oracle; without a gradient the finalize kernel
runs at every size and must give the same bits.

Bars: 1e-5 relative, as for the other MI cases (float32 results of float64 sums)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_23996_amd import smoes as S
from paper_2604_23996_amd import workloads as W
from tests.gpu_util import host, rel_err, say, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,B", [
    (992, 64, 8), (993, 64, 8),  # 31 and 32 chunks of 130 doubles
    (224, 256, 64), (225, 256, 64),  # 7 and 8 chunks of 514: one bin per 4 experts, 64 bins
    (7264, 8, 2), (7265, 8, 2),  # 227 and 228 chunks of 18: more tokens than 256 blocks of four waves
    (5, 12, 12), (33, 100, 10),  # fewer tokens than waves per block; experts past a wave
])
@pytest.mark.parametrize("offsets", [False, True])
def test_one_sample_mi(T, E, B, offsets):
    rng = np.random.default_rng(T + E)
    probs = W.random_probs(rng, T, E, 0.5)
    M = W.random_soft_scores(rng, T)
    e2b = W.random_bin_map(rng, E, B)
    off = np.array([0, T], np.int32)
    say("one sample MI", T, E, B, offsets)
    dev = (t(probs), t(M), t(off) if offsets else None, t(e2b), B)
    mi, loss, dl = S.mi_loss(*dev, grad_scale=0.37)
    mi2, loss2, _ = S.mi_loss(*dev, want_grad=False)
    torch.cuda.synchronize()
    assert torch.equal(mi, mi2) and torch.equal(loss, loss2)
    I_ref = O.mi_per_sample(probs, M, off, e2b, B)
    G_ref = O.mi_loss_grad_logits(probs, M, off, e2b, B, grad_scale=0.37)
    assert np.all(np.abs(host(mi) - I_ref) <= 1e-5 * np.abs(I_ref) + 1e-14)
    assert abs(host(loss)[0] + I_ref[0]) <= 1e-5 * abs(I_ref[0]) + 1e-14
    assert rel_err(host(dl), G_ref) <= 1e-5
