"""Float32 routing at the sizes where its tiles change: tokens around the 16-
and 32-token workgroups and the line between them, experts around the 16- and
64-expert tiles, hidden sizes that end inside a 16-column slice or leave some
of the eight waves without one, rows that start at any element, and ties."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_23996_amd import smoes as S
from tests.gpu_util import check_topk, gate_rtol, host, say, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [8, 24, 136, 1000])
@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (15, 16, 16), (16, 17, 2), (17, 63, 6), (33, 65, 4), (8191, 8, 2),
                                   (8192, 64, 6), (8193, 129, 3), (40, 256, 16)])
def test_route_f32_tiles(T, E, k, d):
    # float64 products and sums rounded once: the logits are the float32 nearest
    # to the exact ones, up to one unit where the bias is added in float32
    say("route f32", T, E, k, d)
    rng = np.random.default_rng(T + 7 * E + d)
    x = rng.standard_normal((T, d)).astype(np.float32)
    w = (rng.standard_normal((E, d)) / np.sqrt(d)).astype(np.float32)
    b = rng.standard_normal(E).astype(np.float32)
    for bias, renorm in ((None, False), (b, True)):
        out = S.route(t(x), t(w), k, None if bias is None else t(bias), renorm_topk=renorm)
        z, g, idx, tw = O.route(x, w, k, bias, renorm)
        got = host(out["logits"])
        assert np.abs(got - z).max() <= 1.3e-7 * (np.abs(z).max() + 1.0)
        rt = gate_rtol(x, w, bias)
        assert np.all(np.abs(host(out["probs"]) - g) <= rt * g)
        clear = check_topk(host(out["topk_idx"]), idx, z, k)
        assert np.all(np.abs(host(out["topk_w"]) - tw)[clear] <= 2 * rt[clear] * tw[clear] + 1e-4 * (k > 1) * tw[clear])


def test_route_f32_any_element_and_ties():
    rng = np.random.default_rng(3)
    T, d, E = 37, 40, 24
    x = rng.standard_normal((T, d)).astype(np.float32)
    w = rng.standard_normal((E, d)).astype(np.float32)
    w[7] = w[3]  # equal logits: the lower index first
    a = S.route(t(x), t(w), 5)
    moved = []
    for v in (x, w):
        buf = torch.empty(v.size + 1, dtype=torch.float32, device="cuda:0")
        buf[1:] = t(v).reshape(-1)
        moved.append(buf[1:].view(v.shape))
    b = S.route(moved[0], moved[1], 5)
    for n in a:
        assert torch.equal(a[n], b[n]), n
    idx = host(a["topk_idx"])
    for row in idx:
        if 7 in row:
            assert list(row).index(3) == list(row).index(7) - 1
