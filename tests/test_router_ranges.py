"""The bf16 router sums each logit over ranges of the hidden dimension, about
one workgroup of 128 tokens x one range per CU. How many ranges a call takes is
part of its logits' bits, and so of the choice between near-tied experts."""
from __future__ import annotations

import os

import pytest

from paper_2604_23996_amd import smoes as S

SIZES = [(1, 2048, 64), (32, 2048, 64), (4096, 2048, 64), (8000, 2048, 64), (8113, 2048, 128), (16384, 2048, 64),
         (16384, 2048, 60), (16384, 4096, 160), (12000, 1024, 8), (40000, 4096, 32), (300, 256, 16)]


def _ranges(T, d):
    """(number of ranges, 32-column steps in each) for 256 CUs."""
    steps = -(-d // 32)
    ks = max(1, min(-(-256 // -(-T // 128)), max(1, steps // 8)))
    per = -(-steps // ks)
    return -(-steps // per), per


@pytest.mark.skipif(not os.path.exists(S.LIB_PATH), reason="libsmoes.so not built")
@pytest.mark.parametrize("T,d,E", SIZES)
def test_partial_planes_of_the_workspace(T, d, E):
    # split weights (three bf16 parts) + one float32 plane of padded logits per range + two alignments of 256
    up = lambda n: -(-n // 256) * 256
    ep = -(-E // 16) * 16
    ks, _ = _ranges(T, d)
    want = up(2 * 3 * ep * (-(-d // 32) * 32)) + up(4 * ks * T * ep) + 512
    assert S.lib().smoes_route_workspace_size(T, d, E, S.SMOES_BF16) == want


@pytest.mark.gpu
@pytest.mark.parametrize("T,d,E", [(32, 2048, 64), (8000, 2048, 64), (16384, 2048, 60), (8113, 1032, 17)])
def test_logits_are_the_ranges_summed_in_order(T, d, E):
    # with the columns outside one range zero, the other ranges add exact zeros
    import torch
    from tests.gpu_util import DEV, say

    say("router ranges", T, d, E)
    g = torch.Generator(device=DEV).manual_seed(T + d + E)
    x = torch.randn((T, d), generator=g, device=DEV).to(torch.bfloat16)
    w = torch.randn((E, d), generator=g, device=DEV) / d ** 0.5
    ks, per = _ranges(T, d)
    total = None
    for r in range(ks):
        part = torch.zeros_like(x)
        cols = slice(32 * per * r, 32 * per * (r + 1))
        part[:, cols] = x[:, cols]
        z = S.route(part, w, 2)["logits"]
        total = z if total is None else total + z
    assert torch.equal(S.route(x, w, 2)["logits"], total)
