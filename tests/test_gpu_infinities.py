"""Infinities and NaN where a kernel's padding, its split of an operand or its
order of work could turn them into something else: the row-major backward of
bf16 layers (float32 operands in three bf16 terms) against the float32 layer of
the same values, the k-packed padding of the packed backward, the MI of a
sample with an infinite probability, and routing past NaN logits."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

from paper_2604_23996_amd import smoes as S
from paper_2604_23996_amd import workloads as W
from tests.gpu_util import DEV, host, run_gpu_layer, say, t
from tests.test_gpu_backward import _inputs

pytestmark = pytest.mark.gpu

CASE = dict(d=72, E=4, k=2, inter=256, n_shared=1, n_bins=2, samples=((100, 61),))
INF = 0x7F80  # bf16 bits


def _kinds(a):
    """0 where finite, +-1 at infinities, 2 at NaN."""
    a = host(a)
    return np.where(np.isnan(a), 2, np.where(np.isinf(a), np.sign(a), 0)).astype(np.int8)


def _rowmajor_grads(inp, dout, moved):
    """Backward of the row-major layer; `moved` replaces tensors after the forward."""
    spec, dev_in, outs, ws = run_gpu_layer(inp, keep_workspace=True, packed=False)
    return S.moe_backward(spec, {**dev_in, **{n: t(v) for n, v in moved.items()}}, outs, ws, None, t(dout), None)


@pytest.mark.parametrize("where", ["dout", "w13", "ws13"])
@pytest.mark.parametrize("sign", [0, 0x8000])
def test_rowmajor_infinities_as_in_float32(where, sign):
    # a float32 value whose lower terms are zero times an infinity stays that infinity
    cfg, inp, dout, _ = _inputs(CASE, 731)
    say("row-major infinity", where, sign)
    moved = {}
    if where == "dout":
        dout = dout.copy()
        dout[7, 3] = INF | sign
    else:  # an up projection: its pre-activations become infinite, the gate's do not
        w = getattr(inp, where).copy()
        if where == "w13":
            w[:, cfg.inter + 5, 11] = INF | sign
        else:
            w[cfg.inter + 5, 11] = INF | sign
        moved[where] = w
    bf = _rowmajor_grads(inp, dout, moved)
    wide = lambda v: W.bf16_bits_to_f32(v) if v is not None and v.dtype == np.uint16 else v
    inp32 = dataclasses.replace(inp, cfg=dataclasses.replace(cfg, dtype=W.F32),
                                **{n: wide(getattr(inp, n)) for n in ("x", "w13", "w2", "ws13", "ws2")})
    f32 = _rowmajor_grads(inp32, wide(dout), {n: wide(v) for n, v in moved.items()})
    seen = 0
    for n in ("dx", "dw13", "dw2", "dws13", "dws2"):
        a, b = _kinds(bf[n]), _kinds(f32[n])
        seen += int((np.abs(b) == 1).sum())
        assert np.array_equal(a, b), (n, int((a != b).sum()))
    assert seen > 0


@pytest.mark.parametrize("streams", [False, True])
def test_packed_padding_rows_stay_zero_beside_an_infinite_weight(streams):
    # one token: 15 of the 16 rows of a k-packed slice are padding. With W2[3][5]
    # infinite dH, dA and dB of column 5 are; their weight gradients are that
    # infinity times x, and every other row's stay finite
    cfg, inp, dout, _ = _inputs(dict(d=72, E=1, k=1, inter=48, n_shared=1, n_bins=1, samples=((1, 0),)), 741)
    dout = dout.copy()
    dout[0, 3] = 0x3F80  # 1.0
    say("packed padding", streams)
    w2, ws2 = inp.w2.copy(), inp.ws2.copy()
    w2[0, 3, 5] = INF
    ws2[3, 5] = INF
    spec, dev_in, outs, ws = run_gpu_layer(inp, keep_workspace=True)
    packed_t = S.pack_transposed_weights(spec, {"w13": t(inp.w13), "w2": t(w2), "ws13": t(inp.ws13), "ws2": t(ws2)})
    st = S.Streams() if streams else None
    g = S.moe_backward(spec, dev_in, outs, ws, packed_t, t(dout), None, streams=st)
    torch.cuda.synchronize()
    if st is not None:
        st.close()
    for n, inter in (("dw13", cfg.inter), ("dws13", cfg.shared_inter)):
        k = _kinds(g[n]).reshape(2 * inter, cfg.d)
        x = W.bf16_bits_to_f32(inp.x)[0]
        assert np.all(x != 0)
        for row in (5, inter + 5):
            assert np.array_equal(np.abs(k[row]), np.ones(cfg.d)), (n, row)
            assert len(set((k[row] * np.sign(x)).tolist())) == 1  # the sign of dA or dB times that of x
        assert not np.delete(k, (5, inter + 5), axis=0).any(), n


@pytest.mark.parametrize("samples", [1, 3])
def test_mi_with_an_infinite_probability(samples):
    # the sample's joint has no finite normaliser: no cell counts, I = 0, as for an
    # empty joint; the other samples are untouched
    rng = np.random.default_rng(9)
    T, E, B = 90, 16, 4
    probs = W.random_probs(rng, T, E, 0.5)
    M, e2b = W.random_soft_scores(rng, T), W.random_bin_map(rng, E, B)
    off = np.linspace(0, T, samples + 1).astype(np.int32)
    clean = host(S.mi_loss(t(probs), t(M), t(off), t(e2b), B)[0])
    probs[2, 5] = np.inf
    say("MI infinite probability", samples)
    for grad in (True, False):
        mi, loss, _ = S.mi_loss(t(probs), t(M), t(off), t(e2b), B, want_grad=grad)
        torch.cuda.synchronize()
        assert host(mi)[0] == 0.0 and np.array_equal(host(mi)[1:], clean[1:])
        assert abs(host(loss)[0] + host(mi).mean()) <= 1e-6


@pytest.mark.parametrize("E,k", [(32, 16), (64, 6), (100, 16), (256, 16)])
def test_route_f32_past_nan_logits(E, k):
    # experts 0 .. 15 have NaN logits: the choice falls on the best of the others
    rng = np.random.default_rng(E)
    T, d = 33, 40
    x = rng.standard_normal((T, d)).astype(np.float32)
    w = rng.standard_normal((E, d)).astype(np.float32)
    best = 16 + np.argsort(-(x.astype(np.float64) @ w[16:].T.astype(np.float64)), axis=1)[:, :k]
    w[:16] = np.nan
    say("route f32 NaN", E, k)
    idx = host(S.route(t(x), t(w), k)["topk_idx"])
    assert np.array_equal(idx, best)


@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("E,k", [(4, 4), (20, 6), (100, 16), (256, 16)])
def test_route_with_too_few_logits_that_are_numbers(E, k, dtype):
    # three experts have a number and the others, by their bias, NaN; three tokens are NaN
    # altogether: numbers by value first, then the lowest of the rest, each expert once
    rng = np.random.default_rng(E + k)
    T, d = 37, 40
    x = rng.standard_normal((T, d)).astype(np.float32)
    w = rng.standard_normal((E, d)).astype(np.float32)
    bad = [0, 17, 36]
    x[bad, 3] = np.nan
    xd = W.f32_to_bf16_bits(x) if dtype == W.BF16 else x
    good = np.sort(rng.permutation(E)[:3])
    bias = np.full(E, np.nan, np.float32)
    bias[good] = 0
    say("route too few numbers", E, k, dtype)
    idx = host(S.route(t(xd), t(w), k, t(bias))["topk_idx"])
    xf = W.bf16_bits_to_f32(xd) if dtype == W.BF16 else x
    z = xf.astype(np.float64) @ w[good].T.astype(np.float64)
    rest = np.setdiff1d(np.arange(E), good)
    for j in range(T):
        want = np.arange(k) if j in bad else np.concatenate([good[np.argsort(-z[j])], rest])[:k]
        assert np.array_equal(idx[j], want), j


def test_layer_with_a_nan_token():
    # the token's rows go to the first experts; every other token's output keeps its bits
    cfg, inp, _, _ = _inputs(CASE, 751)
    say("layer NaN token")
    clean = run_gpu_layer(inp)[2]
    x = inp.x.copy()
    x[9, 5] = 0x7FC0
    o = run_gpu_layer(dataclasses.replace(inp, x=x))[2]
    assert np.array_equal(host(o["topk_idx"])[9], np.arange(cfg.k))
    keep = np.arange(cfg.T) != 9
    for n in ("topk_idx", "topk_w", "probs", "out"):
        assert np.array_equal(host(o[n])[keep], host(clean[n])[keep]), n
    assert np.isnan(host(o["out"])[9]).all()
