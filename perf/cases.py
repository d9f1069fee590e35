"""The work whose speed this framework is judged by, as a user's program calls it.

A case is a dict of plain values; "kind" says which path it takes:

  forward    one SMoES MoE layer forward (moe_forward): routing, modality score,
             MI loss and its logit gradient, permutation, experts, combine. Prefill,
             scoring and evaluation; with few tokens a decode step.
  train      one training step of the layer: the forward, then moe_backward with the
             MI gradient folded in. Packed bf16 weights are packed again in the step
             (all forms the two calls read), because the optimiser has changed them.
  route      the router alone (route), for a program with its own expert engine.
  gauss      the Gaussian statistics update and modality score (modality_score).
  dispatch   what such a program does with its routing: the MI loss (mi_loss), the
             bin balance on top of its gradient and the next bins (binning), and the
             expert-contiguous order with the gathered rows (permute).
  gmm        the mixture estimator's EM step and score (gmm_modality_score).
  attention  the attention-accumulated score of one decoder layer (attention_scores,
             attn_score_update).

Sizes are those of the workloads, tests and benchmark of this repository (hidden
sizes 256 to 4096, 8 to 256 experts, top-1 to top-16, one token to 16384).
Inputs are drawn on the GPU from the seed alone: two modality means half a standard
deviation apart per column, samples of vision tokens followed by text tokens, a router
that leans to one modality per bin as a trained one does, weights N(0, 0.02^2).
"""
import math

import torch

from paper_2604_23996_amd import smoes as S

DEV = "cuda:0"
BETA = 0.99
VAR_FLOOR = 1e-6
FLOPS_MOST = 6.5e12   # of a drawn case on the matrix cores; the listed training step has 7e12
FLOPS_F32 = 6.0e10    # of a drawn case whose products are float32
BYTES_MOST = 6.2e9    # of a drawn layer's expert weights


def listed():
    return [
        # the smallest layer call: a float32 layer of 512 tokens, as in a parity check or a debugging run
        dict(name="layer-fp32-512", kind="forward", dtype="f32", packed=False, streams=False, T=512, batch=1, d=256,
             E=8, k=2, inter=512, shared=0, bins=2, bias=False, update=False, vision=True),
        # one decode step of 32 sequences: a token each, text only, nearly every expert's weights read
        dict(name="layer-decode-32", kind="forward", dtype="bf16", packed=True, streams=True, T=32, batch=1, d=2048,
             E=64, k=6, inter=1408, shared=2, bins=8, bias=False, update=False, vision=False),
        # prefill of four image-text prompts
        dict(name="layer-prefill-4096", kind="forward", dtype="bf16", packed=True, streams=True, T=4096, batch=4,
             d=2048, E=64, k=6, inter=1408, shared=2, bins=8, bias=False, update=False, vision=True),
        # fine-grained experts, no shared one, a ragged number of tokens
        dict(name="layer-finegrained-8113", kind="forward", dtype="bf16", packed=True, streams=True, T=8113, batch=8,
             d=2048, E=128, k=8, inter=768, shared=0, bins=16, bias=False, update=False, vision=True),
        # the largest layer that the benchmark runs, with unequal expert loads
        dict(name="layer-large-16384", kind="forward", dtype="bf16", packed=True, streams=True, T=16384, batch=16,
             d=4096, E=160, k=6, inter=1536, shared=2, bins=8, bias=True, update=False, vision=True),
        # a training step at training batch size, statistics re-estimated from the batch
        dict(name="train-packed-16384", kind="train", dtype="bf16", packed=True, streams=True, T=16384, batch=16,
             d=2048, E=64, k=6, inter=1408, shared=2, bins=8, bias=False, update=True, vision=True),
        # a small training step on row-major weights, as an optimiser holds them
        dict(name="train-rowmajor-1000", kind="train", dtype="bf16", packed=False, streams=False, T=1000, batch=2,
             d=1024, E=16, k=4, inter=512, shared=1, bins=4, bias=False, update=True, vision=True),
        # the router on its own, a ragged batch
        dict(name="route-8000", kind="route", dtype="bf16", T=8000, d=2048, E=64, k=6, bins=8, bias=False, renorm=True),
        # the Gaussian estimator of a training batch: statistics, then scores
        dict(name="gauss-update-16384", kind="gauss", dtype="bf16", T=16384, batch=16, d=2048, update=True),
        # losses and dispatch of a routed prefill batch
        dict(name="dispatch-4096", kind="dispatch", dtype="bf16", T=4096, batch=4, d=2048, E=64, k=6, bins=8),
        # the mixture estimator: EM step and score
        dict(name="gmm-8192", kind="gmm", dtype="bf16", T=8192, batch=8, d=2048, K=2, update=True),
        # grouped-query attention that carries the scores, ragged samples
        dict(name="attention-7000", kind="attention", T=7000, batch=5, d=4096, heads=32, kv_heads=8, head_dim=128),
    ]


# ---------------------------------------------------------------- drawn cases

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tokens(rng, lo=1, hi=16384):
    """lo to hi tokens, evenly over the logarithm; every other one a round number."""
    T = min(hi, max(lo, _log_int(rng, lo, hi)))
    return T if T < 16 or rng.random() < 0.5 else T // 16 * 16


def _batch(rng, T):
    return min(max(1, T // 16), rng.choice([1, 2, 3, 4, 7, 8, 16]))


def _hidden(rng, hi=4096):
    return 8 * _log_int(rng, 32, hi // 8) if rng.random() < 0.4 else rng.choice([d for d in (256, 512, 1024, 2048, 4096) if d <= hi])


def _experts(rng):
    E = rng.choice([8, 16, 24, 32, 60, 64, 96, 128, 160, 256])
    bins = rng.choice([b for b in (2, 4, 8, 12, 16, 32) if E % b == 0])
    k = rng.choice([k for k in (1, 2, 4, 6, 8, 16) if k <= E // 2])
    return E, k, bins


def _layer(rng, kind):
    while True:
        mode = rng.choice(["packed", "packed", "packed", "rowmajor", "f32"])
        E, k, bins = _experts(rng)
        T, d, inter = _tokens(rng), _hidden(rng), 16 * _log_int(rng, 4, 128)
        c = dict(kind=kind, dtype="f32" if mode == "f32" else "bf16", packed=mode == "packed",
                 streams=rng.random() < 0.7, T=T, batch=_batch(rng, T), d=d, E=E, k=k, inter=inter,
                 shared=rng.choice([0, 1, 2]), bins=bins, bias=rng.random() < 0.3,
                 update=kind == "train" or rng.random() < 0.3, vision=T >= 64)
        w = work(c)
        wbytes = 3 * (E + c["shared"]) * inter * d * (2 if mode != "f32" else 4)
        slow = mode == "f32" or (mode == "rowmajor" and kind == "train")
        if w["flops"] <= (FLOPS_F32 if slow else FLOPS_MOST) and wbytes <= (BYTES_MOST if kind == "forward" else 2.0e9):
            return c


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "train", "train", "route", "gauss", "dispatch", "gmm", "attention"])
    if kind in ("forward", "train"):
        return _layer(rng, kind)
    if kind == "attention":
        T = _tokens(rng)
        heads = rng.choice([8, 16, 32])
        return dict(kind=kind, T=T, batch=min(T, max(rng.choice([1, 2, 5, 8, 16]), T // 4096)), d=_hidden(rng), heads=heads,
                    kv_heads=heads // rng.choice([1, 2, 4, 8]), head_dim=rng.choice([64, 128]))
    dtype = rng.choice(["bf16", "bf16", "f32"])
    T, d = _tokens(rng, 16 if kind == "dispatch" else 1), _hidden(rng)
    if kind == "gauss":
        return dict(kind=kind, dtype=dtype, T=T, batch=_batch(rng, T), d=d, update=rng.random() < 0.7)
    if kind == "gmm":
        return dict(kind=kind, dtype=dtype, T=T, batch=_batch(rng, T), d=d, K=rng.choice([1, 2, 3, 4]), update=rng.random() < 0.7)
    E, k, bins = _experts(rng)
    if kind == "route":
        return dict(kind=kind, dtype=dtype, T=T, d=d, E=E, k=k, bins=bins, bias=rng.random() < 0.5, renorm=rng.random() < 0.5)
    return dict(kind="dispatch", dtype=dtype, T=T, batch=_batch(rng, T), d=d, E=E, k=k, bins=bins)


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _act(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _lengths(T, batch):
    """Unequal sample lengths, the same for every seed."""
    share = [3 + (5 * i) % 4 for i in range(batch)]
    cuts = [T * sum(share[:i]) // sum(share) for i in range(batch + 1)]
    return [b - a for a, b in zip(cuts, cuts[1:])]


def _offsets(T, batch):
    off = [0]
    for n in _lengths(T, batch):
        off.append(off[-1] + n)
    return off


def _modality(T, batch, vision=True):
    """0 for the vision tokens that open each sample (65 to 86 % of it), 1 for its text."""
    if not vision:
        return torch.ones(T, dtype=torch.uint8, device=DEV)
    mid = []
    for i, n in enumerate(_lengths(T, batch)):
        v = n * (65 + 7 * (i % 4)) // 100
        mid += [0] * v + [1] * (n - v)
    return torch.tensor(mid, dtype=torch.uint8, device=DEV)


def _means(g, d):
    return 0.5 * torch.randn((2, d), generator=g, device=DEV)


def _tokens_of(g, mu, mid, dtype):
    """Own mean + N(0, I), mixed towards the other modality's mean by U(0, 0.5)."""
    T, d = mid.numel(), mu.shape[1]
    own = mid.long()
    u = 0.5 * torch.rand((T, 1), generator=g, device=DEV)
    x = mu[own] + torch.randn((T, d), generator=g, device=DEV)
    return ((1 - u) * x + u * mu[1 - own]).to(dtype)


def _router(g, mu, E, bins):
    """Router weights whose lower half of the bins leans to vision and the upper half to text."""
    diff = mu[0] - mu[1]
    sign = torch.where(_bin_map(E, bins) < (bins + 1) // 2, 1.0, -1.0)
    noise = 0.02 * math.sqrt(2048 / mu.shape[1]) * torch.randn((E, mu.shape[1]), generator=g, device=DEV)
    return (noise + sign[:, None] * diff / diff.square().sum()).contiguous()


def _bin_map(E, bins):
    return (torch.arange(E, device=DEV) // (E // bins)).to(torch.int32)


def _gauss_state(g, mu):
    """The state after earlier batches: counts, sums of means and of squares."""
    n = torch.tensor([8000.0, 3000.0], device=DEV)
    near = mu + 0.05 * torch.randn(mu.shape, generator=g, device=DEV)
    var = 0.7 + 0.6 * torch.rand(mu.shape, generator=g, device=DEV)
    return n, (n[:, None] * near).contiguous(), (n[:, None] * var).contiguous()


def _gmm_state(g, mu, K):
    n = 2000.0 * (0.5 + torch.rand((2, K), generator=g, device=DEV))
    near = mu[:, None, :] + 0.1 * torch.randn((2, K, mu.shape[1]), generator=g, device=DEV)
    var = 0.7 + 0.6 * torch.rand(near.shape, generator=g, device=DEV)
    return n, (n[:, :, None] * near).contiguous(), (n[:, :, None] * var).contiguous()


def _weights(g, shape, dtype):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype).mul_(0.02)


def _layer_inputs(case, seed):
    g = _gen(seed)
    T, d, E, I, dt = case["T"], case["d"], case["E"], case["inter"], _act(case)
    SI = case["shared"] * I
    mid = _modality(T, case["batch"], case["vision"])
    mu = _means(g, d)
    inp = dict(x=_tokens_of(g, mu, mid, dt), modality_id=mid,
               sample_offsets=torch.tensor(_offsets(T, case["batch"]), dtype=torch.int32, device=DEV),
               w_gate=_router(g, mu, E, case["bins"]),
               logit_bias=torch.randn(E, generator=g, device=DEV) if case["bias"] else None,
               expert_to_bin=_bin_map(E, case["bins"]))
    inp["gauss_n"], inp["gauss_smu"], inp["gauss_ssig"] = _gauss_state(g, mu)
    inp["w13"], inp["w2"] = _weights(g, (E, 2 * I, d), dt), _weights(g, (E, d, I), dt)
    inp["ws13"], inp["ws2"] = (_weights(g, (2 * SI, d), dt), _weights(g, (d, SI), dt)) if SI else (None, None)
    if case["kind"] == "train":
        inp["dout"] = torch.randn((T, d), generator=g, device=DEV).to(dt)
    return inp


def _router_inputs(case, seed):
    g = _gen(seed)
    mu = _means(g, case["d"])
    mid = _modality(case["T"], 1)
    return dict(x=_tokens_of(g, mu, mid, _act(case)), w_gate=_router(g, mu, case["E"], case["bins"]),
                logit_bias=torch.randn(case["E"], generator=g, device=DEV) if case["bias"] else None)


def _score_inputs(case, seed):
    g = _gen(seed)
    mid = _modality(case["T"], case["batch"])
    mu = _means(g, case["d"])
    state = _gmm_state(g, mu, case["K"]) if case["kind"] == "gmm" else _gauss_state(g, mu)
    return dict(x=_tokens_of(g, mu, mid, _act(case)), modality_id=mid, state=state)


def _dispatch_inputs(case, seed):
    g = _gen(seed)
    T, E = case["T"], case["E"]
    mid = _modality(T, case["batch"])
    lean = torch.where(_bin_map(E, case["bins"]) < (case["bins"] + 1) // 2, 1.0, -1.0)
    z = torch.randn((T, E), generator=g, device=DEV) + torch.randn(E, generator=g, device=DEV) * 0.5
    z = z + torch.where(mid == 0, 0.5, -0.5)[:, None] * lean
    a = torch.sigmoid(torch.where(mid == 0, 0.6, -0.6) + 0.3 * torch.randn(T, generator=g, device=DEV))
    return dict(x=torch.randn((T, case["d"]), generator=g, device=DEV).to(_act(case)), modality_id=mid,
                probs=torch.softmax(z, 1), topk_idx=torch.topk(z, case["k"], dim=1).indices.to(torch.int32).contiguous(),
                M=torch.stack([a, 1 - a], 1).contiguous(),
                sample_offsets=torch.tensor(_offsets(T, case["batch"]), dtype=torch.int32, device=DEV),
                expert_to_bin=_bin_map(E, case["bins"]),
                load_ema=200.0 * torch.rand((2, E), generator=g, device=DEV, dtype=torch.float64))


def _attention_inputs(case, seed):
    g = _gen(seed)
    T, d, H, G, D = case["T"], case["d"], case["heads"], case["kv_heads"], case["head_dim"]

    def draw_(shape, scale):
        return (scale * torch.randn(shape, generator=g, device=DEV)).to(torch.bfloat16)
    a = torch.rand(T, generator=g, device=DEV)
    return dict(q=draw_((T, H, D), math.sqrt(2.0)), k=draw_((T, G, D), math.sqrt(2.0)), v=draw_((T, G, D), 1.0),
                x=draw_((T, d), 1.0), x_attn=draw_((T, d), 0.5), m_in=torch.stack([a, 1 - a], 1).contiguous(),
                sample_offsets=torch.tensor(_offsets(T, case["batch"]), dtype=torch.int32, device=DEV))


def _inputs(case, seed):
    return {"forward": _layer_inputs, "train": _layer_inputs, "route": _router_inputs, "gauss": _score_inputs,
            "gmm": _score_inputs, "dispatch": _dispatch_inputs, "attention": _attention_inputs}[case["kind"]](case, seed)


def prepare(case, seed):
    """Inputs on the GPU and what a program keeps between calls: descriptor, packed
    weights (forward), output buffers, workspaces and side streams."""
    st = dict(case=case, inp=_inputs(case, seed))
    if case["kind"] not in ("forward", "train"):
        return st
    train = case["kind"] == "train"
    spec = S.LayerSpec(T=case["T"], d=case["d"], E=case["E"], k=case["k"], inter=case["inter"],
                       shared_inter=case["shared"] * case["inter"], n_bins=case["bins"], n_batch=case["batch"],
                       act_dtype=S.SMOES_F32 if case["dtype"] == "f32" else S.SMOES_BF16, beta=BETA,
                       var_floor=VAR_FLOOR, update_stats=case["update"], weights_packed=case["packed"],
                       save_preact=train and case["packed"])
    if case["packed"] and not train:
        S.pack_layer_inputs(spec, st["inp"])
    st.update(spec=spec, outs=S.alloc_outputs(spec, DEV, _act(case), want_perm=False, want_dlogits=case["vision"]),
              ws=torch.empty(S.workspace_bytes(spec), dtype=torch.uint8, device=DEV),
              streams=S.Streams() if case["streams"] else None, grads=None, bws=None)
    if train:
        st["bws"] = torch.empty(S.backward_workspace_bytes(spec), dtype=torch.uint8, device=DEV)
        T, d, E, I, SI = case["T"], case["d"], case["E"], case["inter"], spec.shared_inter
        f = dict(dtype=torch.float32, device=DEV)
        w = dict(dtype=_act(case), device=DEV)
        st["grads"] = dict(dx=torch.empty((T, d), **f), dw_gate=torch.empty((E, d), **f), dbias=torch.empty(E, **f),
                           dz=torch.empty((T, E), **f), dw=torch.empty((T, case["k"]), **f),
                           dw13=torch.empty((E, 2 * I, d), **w), dw2=torch.empty((E, d, I), **w),
                           dws13=torch.empty((2 * SI, d), **w) if SI else None,
                           dws2=torch.empty((d, SI), **w) if SI else None)
    return st


# ---------------------------------------------------------------- one pass

_LAYER_OUTS = ("logits", "probs", "topk_idx", "topk_w", "M", "out")
_LOSS_OUTS = ("mi_per_sample", "loss", "dlogits")  # a decode step (text alone, a few tokens) has no use for the loss
_STATE = ("gauss_n", "gauss_smu", "gauss_ssig")


def run(state):
    case, inp = state["case"], state["inp"]
    kind = case["kind"]
    if kind == "route":
        return S.route(inp["x"], inp["w_gate"], case["k"], inp["logit_bias"], renorm_topk=case["renorm"])
    if kind == "gauss":
        M = S.modality_score(inp["x"], *inp["state"], inp["modality_id"], update=case["update"], beta=BETA,
                             var_floor=VAR_FLOOR)
        return dict(M=M, state=inp["state"])
    if kind == "gmm":
        M, resp = S.gmm_modality_score(inp["x"], *inp["state"], inp["modality_id"], update=case["update"], beta=BETA,
                                       var_floor=VAR_FLOOR, want_resp=True)
        return dict(M=M, resp=resp, state=inp["state"])
    if kind == "dispatch":
        mi, loss, dl = S.mi_loss(inp["probs"], inp["M"], inp["sample_offsets"], inp["expert_to_bin"], case["bins"])
        b = S.binning(inp["probs"], inp["topk_idx"], inp["modality_id"], inp["expert_to_bin"], case["bins"], beta=BETA,
                      load_ema=inp["load_ema"], dlogits=dl, accumulate=True)
        off, perm, inv, xp = S.permute(inp["topk_idx"], case["E"], inp["x"])
        return dict(b, mi=mi, mi_loss=loss, load_ema=inp["load_ema"], offsets=off, perm_token=perm, perm_inv=inv, x_perm=xp)
    if kind == "attention":
        o, mh = S.attention_scores(inp["q"], inp["k"], inp["v"], inp["sample_offsets"], inp["m_in"])
        return dict(o=o, m_heads=mh, m_out=S.attn_score_update(inp["x"], inp["x_attn"], mh, inp["m_in"]))
    spec, outs = state["spec"], state["outs"]
    names = _LAYER_OUTS + (_LOSS_OUTS if case["vision"] else ())
    if kind == "forward":
        S.moe_forward(spec, inp, outs, state["ws"], streams=state["streams"])
        out = {n: outs[n] for n in names}
    else:
        now, packed_t = inp, None
        if spec.weights_packed:
            now = dict(inp)
            packed_t = S.pack_transposed_weights(spec, inp)
            S.pack_layer_inputs(spec, now)
        S.moe_forward(spec, now, outs, state["ws"], streams=state["streams"])
        out = {n: outs[n] for n in names}
        out.update(S.moe_backward(spec, now, outs, state["ws"], packed_t, inp["dout"], outs["dlogits"],
                                  grads=state["grads"], workspace=state["bws"], streams=state["streams"]))
    if spec.update_stats:
        out.update({n: inp[n] for n in _STATE})
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    kind, T, d = case["kind"], case["T"], case["d"]
    s = 4 if case.get("dtype") == "f32" else 2
    if kind == "gauss":
        return dict(bytes=T * d * s + T * 8 + (T + 32 * d if case["update"] else 16 * d), flops=(12 if case["update"] else 6) * T * d)
    if kind == "gmm":
        K = case["K"]
        return dict(bytes=T * d * s + T * (9 + 4 * K) + (32 if case["update"] else 16) * K * d, flops=(14 if case["update"] else 8) * K * T * d)
    if kind == "attention":
        H, G, D = case["heads"], case["kv_heads"], case["head_dim"]
        pairs = sum(n * (n + 1) // 2 for n in _lengths(T, case["batch"]))
        return dict(bytes=2 * T * D * (2 * H + 2 * G) + 8 * T * H * 2 + 4 * T * d + 24 * T, flops=4 * pairs * H * (D + 2))
    E, k = case["E"], case["k"]
    if kind == "route":
        return dict(bytes=T * d * s + E * d * 4 + T * E * 8 + T * k * 8, flops=2 * T * d * E)
    if kind == "dispatch":
        return dict(bytes=T * E * 4 + T * E * 4 + T * (9 + 4 * k) + 8 * T * k + T * d * s + T * k * d * s + 40 * E, flops=20 * T * E)
    I, SI = case["inter"], case["shared"] * case["inter"]
    hit = min(E, T * k)
    rows = T * k * I + T * SI
    wb = 3 * d * s
    flops = 2 * T * d * E + 6 * rows * d
    size = 2 * T * d * s + E * d * 4 + T * (E * (12 if case["vision"] else 8) + k * 8 + 8) + (hit * I + SI) * wb
    if case["update"]:
        size += 32 * d
    if kind == "train":
        flops += 4 * T * d * E + 12 * rows * d
        size += T * d * s + T * d * 4 + E * d * 4 + T * E * 8 + (E * I + SI) * wb
    return dict(bytes=size, flops=flops)


def tolerance(case):
    """About four times what the path shows against `exact`, and for a choice of experts
    that a rounding can turn, a share of whole values."""
    kind = case["kind"]
    if kind in ("forward", "train"):
        if case["dtype"] == "f32":
            return dict(rel=1e-5, max=0.01, differ=1e-3)
        return dict(rel=0.014, max=0.5, differ=1e-3)
    if kind == "attention":
        return dict(rel=0.009, max=0.1)
    if kind == "dispatch":
        return dict(rel=1e-5, max=1e-3)
    return dict(rel=5e-6, max=1e-3, differ=1e-3 if kind == "route" else 0.0)


# ---------------------------------------------------------------- the same in 64 bits

def _beta():
    return float(torch.tensor(BETA, dtype=torch.float32))


def _floor():
    return float(torch.tensor(VAR_FLOOR, dtype=torch.float32))


def _x_routing(x, w_gate, bias, k, renorm=False):
    z = x @ w_gate.double().t()
    if bias is not None:
        z = z + bias.double()
    g = torch.softmax(z, 1)
    idx = torch.topk(z, k, dim=1).indices
    w = g.gather(1, idx)
    return z, g, idx, w / w.sum(1, keepdim=True) if renorm else w


def _x_merge(n0, mu0, sg0, n, mean, sq):
    """The decayed state with one batch's count, mean and centred squares folded in."""
    b = _beta() * n0
    tot = b + n
    both = (n0 > 0) & (n > 0)
    prev = mu0 / torch.where(n0 > 0, n0, 1.0)[..., None]
    cross = torch.where(both, b * n / torch.where(tot > 0, tot, 1.0), 0.0)[..., None] * (mean - prev).square()
    return tot, _beta() * mu0 + n[..., None] * mean, _beta() * sg0 + sq + cross


def _x_gauss(x, mid, state, update):
    n, smu, ssig = (v.double() for v in state)
    if update:
        sel = [x[mid == m] for m in (0, 1)]
        cnt = torch.tensor([float(v.shape[0]) for v in sel], device=DEV, dtype=torch.float64)
        mean = torch.stack([v.mean(0) if v.shape[0] else torch.zeros_like(x[0]) for v in sel])
        sq = torch.stack([(v - m).square().sum(0) for v, m in zip(sel, mean)])
        n, smu, ssig = _x_merge(n, smu, ssig, cnt, mean, sq)
    mu = smu / n[:, None]
    var = (ssig / n[:, None]).clamp_min(_floor())
    ll = torch.stack([-0.5 * (var[m].log().sum() + ((x - mu[m]).square() / var[m]).sum(1)) for m in (0, 1)], 1)
    return torch.softmax(ll / (0.5 * x.shape[1]), 1), (n, smu, ssig)


def _x_gmm(x, mid, state, K, update):
    n, smu, ssig = (v.double() for v in state)

    def logs():
        mu, var = smu / n[..., None], (ssig / n[..., None]).clamp_min(_floor())
        lp = (n / n.sum(1, keepdim=True)).log()
        return torch.stack([torch.stack([lp[m, c] - 0.5 * (var[m, c].log().sum() + ((x - mu[m, c]).square() / var[m, c]).sum(1))
                                         for c in range(K)], 1) for m in (0, 1)], 1)
    resp = torch.softmax(logs()[torch.arange(x.shape[0], device=DEV), mid.long()], 1)
    if update:
        r = torch.stack([torch.where((mid == m)[:, None], resp, 0.0) for m in (0, 1)])
        cnt = r.sum(1)
        safe = torch.where(cnt > 0, cnt, 1.0)
        mean = torch.stack([(r[m].t() @ x) / safe[m][:, None] for m in (0, 1)])
        sq = torch.stack([torch.stack([(r[m, :, c, None] * (x - mean[m, c]).square()).sum(0) for c in range(K)]) for m in (0, 1)])
        n, smu, ssig = _x_merge(n, smu, ssig, cnt, mean, sq)
    return torch.softmax(torch.logsumexp(logs(), 2) / (0.5 * x.shape[1]), 1), resp, (n, smu, ssig)


def _x_mi(g, M, off, e2b, bins):
    """MI of every sample, the loss and its logit gradient."""
    E = g.shape[1]
    hot = torch.zeros((E, bins), dtype=torch.float64, device=DEV)
    hot[torch.arange(E, device=DEV), e2b.long()] = 1.0
    G = g @ hot
    mis, dz, n = [], torch.zeros_like(g), len(off) - 1
    for a, b in zip(off, off[1:]):
        if b == a:
            mis.append(torch.zeros((), dtype=torch.float64, device=DEV))
            continue
        m, gs = M[a:b].double(), G[a:b]
        W = m.sum(0)
        Sb = (m.t() @ gs) / (E // bins * W[:, None])
        Z = Sb.sum()
        P = Sb / Z
        r = (P / (P.sum(1, keepdim=True) * P.sum(0, keepdim=True))).log()
        I = (P * r).sum()
        h = m @ ((r - I) / (E // bins * W[:, None] * Z))
        dz[a:b] = -g[a:b] * (h[:, e2b.long()] - (h * gs).sum(1, keepdim=True)) / n
        mis.append(I)
    mis = torch.stack(mis)
    return mis, -mis.mean().reshape(1), dz


def _x_swiglu(x, w13, w2):
    a, b = (x @ w13.t()).chunk(2, 1)
    return (a * torch.sigmoid(a) * b) @ w2.t()


def _x_swiglu_grad(x, w13, w2, dy, wrow):
    """dx, dw13, dw2 and <dy, y> per row of rows weighted by wrow."""
    a, b = (x @ w13.t()).chunk(2, 1)
    sg = torch.sigmoid(a)
    h = a * sg * b
    dot = (dy * (h @ w2.t())).sum(1)
    dyw = dy * wrow[:, None]
    dh = dyw @ w2
    dab = torch.cat([dh * b * sg * (1 + a * (1 - sg)), dh * a * sg], 1)
    return dab @ w13, dab.t() @ x, dyw.t() @ h, dot


def _x_layer(case, inp):
    x, mid, k, E, dt = inp["x"].double(), inp["modality_id"], case["k"], case["E"], _act(case)
    z, g, idx, w = _x_routing(x, inp["w_gate"], inp["logit_bias"], k)
    M, st = _x_gauss(x, mid, [inp[n] for n in _STATE], case["update"])
    train = case["kind"] == "train"
    out = torch.zeros_like(x)
    grads = {}
    if train:
        dy = inp["dout"].double()
        dx, dw, ones = torch.zeros_like(x), torch.zeros_like(w), torch.ones_like(x[:, 0])
        dw13 = torch.zeros(inp["w13"].shape, dtype=torch.float64, device=DEV)
        dw2 = torch.zeros(inp["w2"].shape, dtype=torch.float64, device=DEV)
    for e in range(E):
        t, slot = (idx == e).nonzero(as_tuple=True)
        if t.numel() == 0:
            continue
        w13, w2, xe = inp["w13"][e].double(), inp["w2"][e].double(), x[t]
        out.index_add_(0, t, _x_swiglu(xe, w13, w2) * w[t, slot][:, None])
        if train:
            dxe, dw13[e], dw2[e], dot = _x_swiglu_grad(xe, w13, w2, dy[t], w[t, slot])
            dx.index_add_(0, t, dxe)
            dw[t, slot] = dot
    if case["shared"]:
        ws13, ws2 = inp["ws13"].double(), inp["ws2"].double()
        out += _x_swiglu(x, ws13, ws2)
        if train:
            dxs, grads["dws13"], grads["dws2"], _ = _x_swiglu_grad(x, ws13, ws2, dy, ones)
            dx += dxs
    res = dict(logits=z, probs=g, topk_idx=None, topk_w=w, M=M, out=out)
    if case["vision"]:
        mi, loss, dl = _x_mi(g, M, _offsets(case["T"], case["batch"]), inp["expert_to_bin"], case["bins"])
        res.update(mi_per_sample=mi, loss=loss, dlogits=dl)
    if train:
        dg = torch.zeros_like(g).scatter_(1, idx, dw)
        dz = g * (dg - (g * dg).sum(1, keepdim=True)) + res.get("dlogits", 0.0)
        res.update(grads, dx=dx + dz @ inp["w_gate"].double(), dw_gate=dz.t() @ x, dbias=dz.sum(0), dz=dz, dw=dw,
                   dw13=dw13, dw2=dw2)
    if case["update"]:
        res.update(zip(_STATE, st))
    return res


def _x_dispatch(case, inp):
    g, idx, mid, E, bins = inp["probs"].double(), inp["topk_idx"].long(), inp["modality_id"].long(), case["E"], case["bins"]
    e2b = inp["expert_to_bin"].long()
    mi, loss, dl = _x_mi(g, inp["M"], _offsets(case["T"], case["batch"]), e2b, bins)
    T, NB = case["T"], E // bins
    chosen = torch.zeros((T, E), dtype=torch.float64, device=DEV).scatter_(1, idx, 1.0)
    C = torch.stack([chosen[mid == m].sum(0) for m in (0, 1)])
    ema = _beta() * inp["load_ema"] + (1.0 - _beta()) * C
    tot = ema.sum(0)
    f_spec = torch.where(tot > 0, ema[1] / torch.where(tot > 0, tot, 1.0), 0.5)
    in_bin = torch.zeros((T, bins), dtype=torch.float64, device=DEV).scatter_(1, e2b[idx], 1.0)
    Tk = in_bin.sum(0)[e2b]
    safe = torch.where(Tk > 0, Tk, 1.0)
    f = chosen.sum(0) / safe
    P = (g * in_bin[:, e2b]).sum(0) / safe
    dg = in_bin[:, e2b] * (NB * f / safe)
    share = C / C.sum(1, keepdim=True).clamp_min(1.0)
    den = share.sum(0)
    msi = (2 * (torch.where(den > 0, share[1] / torch.where(den > 0, den, 1.0), 0.5) - 0.5).abs()).mean()
    order = torch.sort(inp["topk_idx"].reshape(-1).long(), stable=True).indices
    return dict(counts=None, f_spec=f_spec, expert_to_bin_next=None, bal_loss=(NB * (f * P).sum()).reshape(1), msi=msi.reshape(1),
                dlogits=dl + g * (dg - (g * dg).sum(1, keepdim=True)), mi=mi, mi_loss=loss, load_ema=ema, offsets=None,
                perm_token=None, perm_inv=None, x_perm=inp["x"][order // case["k"]].double())


def _x_attention(case, inp):
    q, k, v, m = (inp[n].double() for n in ("q", "k", "v", "m_in"))
    H, rep = case["heads"], case["heads"] // case["kv_heads"]
    o, mh = torch.zeros_like(q), torch.zeros((case["T"], H, 2), dtype=torch.float64, device=DEV)
    off = _offsets(case["T"], case["batch"])
    for a, b in zip(off, off[1:]):
        hide = torch.triu(torch.ones((b - a, b - a), dtype=torch.bool, device=DEV), 1)
        for h in range(H if b > a else 0):
            z = (q[a:b, h] @ k[a:b, h // rep].t()) / math.sqrt(case["head_dim"])
            p = torch.softmax(z.masked_fill_(hide, float("-inf")), 1)
            o[a:b, h], mh[a:b, h] = p @ v[a:b, h // rep], p @ m[a:b]
    na, nx = (inp[n].double().norm(dim=1, keepdim=True) for n in ("x_attn", "x"))
    return dict(o=o, m_heads=mh, m_out=(na * mh.mean(1) + nx * m) / (na + nx))


def exact(case, seed):
    inp, kind = _inputs(case, seed), case["kind"]
    if kind in ("forward", "train"):
        return _x_layer(case, inp)
    if kind == "dispatch":
        return _x_dispatch(case, inp)
    if kind == "attention":
        return _x_attention(case, inp)
    x = inp["x"].double()
    if kind == "route":
        z, g, _, w = _x_routing(x, inp["w_gate"], inp["logit_bias"], case["k"], case["renorm"])
        return dict(logits=z, probs=g, topk_idx=None, topk_w=w)
    if kind == "gauss":
        M, st = _x_gauss(x, inp["modality_id"], inp["state"], case["update"])
        return dict(M=M, state=st)
    M, resp, st = _x_gmm(x, inp["modality_id"], inp["state"], case["K"], case["update"])
    return dict(M=M, resp=resp, state=st)
