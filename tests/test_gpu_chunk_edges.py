"""Entry points whose kernels work in chunks of tokens, stripes of columns or
groups of chunks, at the sizes where one more token, column or chunk changes
the path: permutation (one 256-token chunk is one launch), binning and the
statistics of both estimators (64-token chunks, eight or four chunk groups,
64- and 512-column blocks); and the layer forward on both sides of the line
from which the combine runs inside the shared down GEMM."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_23996_amd import smoes as S
from paper_2604_23996_amd import workloads as W
from tests.gpu_util import host, rel_err, run_gpu_layer, say, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k", [(1, 1), (64, 6), (65, 2), (256, 16)])
@pytest.mark.parametrize("T", [1, 64, 255, 256, 257, 8449])
def test_permute_chunks(T, E, k):
    say("permute chunks", T, E, k)
    idx = W.random_topk(np.random.default_rng(T + E), T, E, k, skew=2.0)
    off, perm, inv, _ = S.permute(t(idx), E)
    _, ro, rp, ri = O.permutation(idx, E)
    assert np.array_equal(host(off), ro) and np.array_equal(host(perm), rp) and np.array_equal(host(inv), ri)


@pytest.mark.parametrize("E,k,bins", [(8, 2, 2), (64, 6, 8), (128, 4, 64), (256, 16, 4)])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 4 * 64 * 8 + 1])
def test_binning_chunks(T, E, k, bins):
    # counts and maps exact; the loss and its gradient are float64 sums rounded once
    say("binning chunks", T, E, k, bins)
    rng = np.random.default_rng(T * 7 + E)
    g, idx = W.random_probs(rng, T, E), W.random_topk(rng, T, E, k)
    mid = (rng.random(T) < 0.3).astype(np.uint8)
    e2b = W.random_bin_map(rng, E, bins, contiguous=False)
    out = S.binning(t(g), t(idx), t(mid), t(e2b), bins)
    C = O.modality_expert_counts(idx, mid, E)
    assert np.array_equal(host(out["counts"]), C)
    assert np.array_equal(host(out["f_spec"]), O.f_spec(C))
    assert np.array_equal(host(out["expert_to_bin_next"]), O.adaptive_bins(O.f_spec(C), bins))
    assert abs(float(out["bal_loss"]) - O.bin_balance_loss(g, idx, e2b, bins)) <= 1e-6 * O.bin_balance_loss(g, idx, e2b, bins)
    assert rel_err(host(out["dlogits"]), O.bin_balance_grad_logits(g, idx, e2b, bins)) <= 1e-6
    assert abs(float(out["msi"]) - O.msi(C[1], C[0])) <= 1e-6


SHAPES = [(1, 8), (63, 504), (64, 512), (65, 520), (129, 2056), (8 * 64 + 1, 64), (8 * 64 * 16 + 64, 72), (7, 4104)]


def _tokens(T, d, dtype, seed):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((T, d)) + 0.5).astype(np.float32)
    return (W.f32_to_bf16_bits(x) if dtype == W.BF16 else x), (rng.random(T) < 0.4).astype(np.uint8), rng


@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("T,d", SHAPES)
def test_gauss_chunks(T, d, dtype):
    # float32 state of float64 sums: 1e-6 normwise (one rounding is 6e-8); scores 1e-5
    say("gauss chunks", T, d, dtype)
    x, mid, rng = _tokens(T, d, dtype, T + d)
    n, smu, ssig = (t(a) for a in W.random_gauss_state(rng, d))
    st = O.GaussState.of(host(n), host(smu), host(ssig))
    M = S.modality_score(t(x), n, smu, ssig, t(mid), update=True)
    ref = O.gauss_update(st, x, mid, float(np.float32(0.99)))
    for got, r in ((n, ref.n), (smu, ref.s_mu), (ssig, ref.s_sig)):
        assert rel_err(host(got), r) <= 1e-6
    mu, var = O.gauss_params(ref, 1e-6)
    assert rel_err(host(M), O.modality_score(x, mu, var, 0.5 * d)) <= 1e-5


@pytest.mark.parametrize("K", [1, 2, 3, 4])
@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("T,d", SHAPES)
def test_gmm_chunks(T, d, dtype, K):
    say("gmm chunks", T, d, dtype, K)
    x, mid, rng = _tokens(T, d, dtype, T + d + K)
    n, smu, ssig = (t(a) for a in W.random_gmm_state(rng, d, K, spread=0.05))
    st = O.GmmState.of(host(n), host(smu), host(ssig))
    M, resp = S.gmm_modality_score(t(x), n, smu, ssig, t(mid), update=True, want_resp=True)
    pi, mu, var = O.gmm_params(st, 1e-6)
    # the responsibilities follow log-likelihoods of size d held to ~1e-7 relative
    assert np.abs(host(resp) - O.gmm_responsibilities(x, mid, pi, mu, var)).max() <= 2e-5 + 2e-7 * d
    ref = O.gmm_update(st, x, mid, float(np.float32(0.99)), 1e-6)
    for got, r in ((n, ref.n), (smu, ref.s_mu), (ssig, ref.s_sig)):
        assert rel_err(host(got), r) <= 1e-5
    pi, mu, var = O.gmm_params(ref, 1e-6)
    assert rel_err(host(M), O.gmm_modality_score(x, pi, mu, var, 0.5 * d)) <= 1e-5
    # score alone, with and without the responsibilities: the same scores
    a, _ = S.gmm_modality_score(t(x), n, smu, ssig, t(mid), want_resp=True)
    b, _ = S.gmm_modality_score(t(x), n, smu, ssig)
    assert torch.equal(a, b)


@pytest.mark.parametrize("K", [1, 4])
@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
def test_gmm_score_tokens_per_wave(dtype, K):
    # from 4096 tokens on a wave takes four tokens, below one: a token's score has the same bits
    T, d = 4097, 72
    say("gmm tokens per wave", dtype, K)
    x, mid, rng = _tokens(T, d, dtype, 3 + K)
    n, smu, ssig = (t(a) for a in W.random_gmm_state(rng, d, K, spread=0.05))
    M, resp = S.gmm_modality_score(t(x), n, smu, ssig, t(mid), want_resp=True)
    for cut in (1, 4095, 4096):
        a, r = S.gmm_modality_score(t(x[:cut]), n, smu, ssig, t(mid[:cut]), want_resp=True)
        assert torch.equal(a, M[:cut]) and torch.equal(r, resp[:cut]), cut


@pytest.mark.parametrize("T", [32640, 32641, 32700])
def test_combine_in_the_shared_down_gemm_from_512_tiles(T):
    # d = 264: two column tiles, so 32641 tokens are the first with 512 tiles; the
    # side-stream schedule has the bits of the single-stream one on both sides of
    # the line, with a short last row tile and a short last column tile
    say("fused combine", T)
    cfg = W.small_config(d=264, E=8, k=3, inter=16, n_shared=1, n_bins=2, samples=((T - T // 3, T // 3),), dtype=W.BF16,
                         seed=9)
    inp = W.make_layer_inputs(cfg)
    _, _, a = run_gpu_layer(inp)
    streams = S.Streams()
    _, _, b = run_gpu_layer(inp, streams=streams)
    for n in a:
        assert torch.equal(a[n], b[n]), n
    streams.close()
