"""The mixture score of a token far from every mean, where the float64 sums are
large against their differences: a call of 4097 tokens (four per wave) and
shorter ones (one per wave) add in the same order, so a token's score and
responsibilities have the same bits in both."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2604_23996_amd import smoes as S
from paper_2604_23996_amd import workloads as W
from tests.gpu_util import say, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3, 4])
@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("d", [72, 4104])
def test_far_tokens_have_the_same_bits_at_any_count(d, dtype, K):
    say("gmm far", d, dtype, K)
    T = 4097
    rng = np.random.default_rng(d + K)
    # squared distances of 1e8 in some groups of eight columns and of 1 in the others, so that a
    # lane's float64 sum rounds in every step; sums of 1e11 at 4104 columns (held to 3e-5). The
    # components' means differ by 1e-3, which moves a sum by about 10 sqrt(d): the size of tau
    far = np.repeat(rng.random(d // 8) < 0.5, 8)
    x = np.where(far, 1e4, 1.0) * (1 + 0.01 * rng.standard_normal((T, d)))
    x = x.astype(np.float32)
    x = W.f32_to_bf16_bits(x) if dtype == W.BF16 else x
    mid = (rng.random(T) < 0.4).astype(np.uint8)
    n = (100 * (1 + rng.random((2, K)))).astype(np.float32)
    mean = 0.1 * rng.standard_normal(d) + 1e-3 * rng.standard_normal((2, K, d))
    smu = (n[..., None] * mean).astype(np.float32)
    ssig = np.repeat(2 * n[..., None], d, axis=2)  # variance 2 exactly, so log sigma^2 is not 0
    dev = [t(a) for a in (n, smu, ssig)]
    tau = 10.0 * d ** 0.5
    M, resp = S.gmm_modality_score(t(x), *dev, t(mid), tau=tau, want_resp=True)
    for cut in (1, 2048, 4095, 4096):
        a, r = S.gmm_modality_score(t(x[:cut]), *dev, t(mid[:cut]), tau=tau, want_resp=True)
        assert torch.equal(a, M[:cut]) and torch.equal(r, resp[:cut]), (cut, int((a != M[:cut]).sum()))
