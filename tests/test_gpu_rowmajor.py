"""Row-major matrix tiles (float32 layers; the backward of bf16 layers with
row-major weights) at the sizes where a tile can go wrong: rows one below, at
and one above the 64-row tiles, inner sizes of 16, 64 +- 16 and 128 +- 16,
hidden sizes one chunk past a K step, one token, tensors that start one
element off a 16-byte boundary, and an infinite upstream gradient.

Bars as in test_gpu_backward.py: float32 layers are float32 sums of at most a
few thousand exact-width products (1e-5 normwise, 6e-8 unit roundoff); the
bf16 layers' forward stores H and Y in bf16."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_23996_amd import smoes as S
from paper_2604_23996_amd import workloads as W
from tests.gpu_util import DEV, host, rel_err, say, t
from tests.test_gpu_backward import BARS, BARS_F32, ELEM, ELEM_F32, _compare, _inputs, _ref, run_gpu_backward

pytestmark = pytest.mark.gpu

# one expert, so that its rows are the tokens; then several with ragged rows
SIZES = [dict(d=72, E=1, k=1, inter=16, n_shared=1, n_bins=1, samples=((T - T // 3, T // 3),)) for T in (1, 63, 64, 65)]
SIZES += [dict(d=d, E=6, k=2, inter=i, n_shared=s, n_bins=2, samples=((100, 61),))
          for d, i, s in ((64, 48, 0), (136, 80, 1), (8, 112, 1), (264, 144, 2))]


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("size", range(len(SIZES)))
def test_rowmajor_tile_edges(size, dtype):
    cfg, inp, dout, aux = _inputs(SIZES[size], 700 + size, dtype=dtype)
    say("row-major tiles", size, dtype, "T", cfg.T)
    _, outs, g = run_gpu_backward(inp, dout, aux, False, packed=False)
    f32 = dtype == W.F32
    _compare(g, _ref(inp, cfg, dout, aux, False), inp, outs, cfg, bars=BARS_F32 if f32 else BARS,
             elem=ELEM_F32 if f32 else ELEM)
    if f32:
        z, _, idx, w = O.route(inp.x, inp.w_gate, cfg.k, None)
        ref, _, _ = O.experts_grouped(inp.x, idx, w, inp.w13, inp.w2, inp.ws13, inp.ws2, cfg.E)
        assert rel_err(host(outs["out"]), ref) <= 1e-5


def _shift(a):
    """The same tensor one element past the start of its allocation."""
    b = torch.empty(a.numel() + 1, dtype=a.dtype, device=a.device)
    b[1:] = a.reshape(-1)
    return b[1:].view(a.shape)


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_rowmajor_weights_at_any_element(dtype):
    # the weights may start at any element: same bits as at an aligned start
    cfg, inp, dout, _ = _inputs(SIZES[5], 711, dtype=dtype)
    from tests.gpu_util import run_gpu_layer
    spec, dev_in, outs, ws = run_gpu_layer(inp, keep_workspace=True, packed=False)
    a = S.moe_backward(spec, dev_in, outs, ws, None, t(dout), None)
    moved = dict(dev_in)
    for n in ("w13", "w2", "ws13", "ws2"):
        moved[n] = _shift(dev_in[n])
    if dtype == W.F32:
        out0 = outs["out"].clone()
        S.moe_forward(spec, moved, outs, ws)
        assert torch.equal(out0, outs["out"])
    b = S.moe_backward(spec, moved, outs, ws, None, t(dout), None)
    for n in a:
        assert torch.equal(a[n], b[n]), n


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_rowmajor_infinite_gradient_stays_in_its_rows(dtype):
    # an infinity in one token's upstream gradient leaves the other tokens' input
    # gradients and the weight gradients of the experts it did not choose as they were
    cfg, inp, dout, _ = _inputs(SIZES[4], 712, dtype=dtype)
    _, o, a = run_gpu_backward(inp, dout, None, False, packed=False)
    bad = dout.copy()
    bad[7, 3] = 0x7F80 if dtype == W.BF16 else np.inf
    _, _, b = run_gpu_backward(inp, bad, None, False, packed=False)
    keep = np.arange(cfg.T) != 7
    assert np.array_equal(host(a["dx"])[keep], host(b["dx"])[keep])
    used = set(host(o["topk_idx"])[7].tolist())
    for e in range(cfg.E):
        same = np.array_equal(host(a["dw2"][e]), host(b["dw2"][e]))
        assert same == (e not in used)
