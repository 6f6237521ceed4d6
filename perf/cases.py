"""Timed cases of the framework's public entry points.

Four kinds of call, each as a user's program makes it:

* ``layer``: new tokens arrive in the state's buffer, the state is reset and
  one MoE layer runs (``trimmoe_layer_step``): route, decide, grouped expert
  FFN, combine, exit head, gate and compaction;
* ``stack``: the same for every layer of a model (``trimmoe_stack_forward``,
  or ``trimmoe_stack_forward_static``, which needs no workspace);
* ``labels``: the output head's prediction of cached hidden states of one
  layer and the consistency labels against the full-depth prediction;
* ``train``: the sigmoid exit head of one layer trained on such labels.

``listed`` holds the sizes the framework's configurations name (Switch-Base,
Qwen-MoE and Mixtral MoE layers, decode and prefill batches) and ragged ones
between them; ``draw`` spreads over the same ranges.  Inputs are made on the
GPU from the seed alone, with the recipe of ``synthgen`` in short: remote
experts are noisy copies of local ones (so that substitutions fall on both
sides of the budget) and tokens carry a planted output direction (so that
some exit early).
"""
from __future__ import annotations

import math

import torch

from paper_2608_00573_amd import abi

DEV = "cuda"
SIGMA = 0.02

# MoE layer shapes (d_model, experts, top_k, d_ff, shared d_ff, vocabulary)
SHAPES = {
    "tiny": dict(d_model=64, n_experts=8, top_k=1, d_ff=256, d_ff_shared=0, vocab_exit=512,
                 act="relu", normalize_topk=0, n_local=4, zipf=0.0),
    "switch": dict(d_model=768, n_experts=8, top_k=1, d_ff=3072, d_ff_shared=0, vocab_exit=32128,
                   act="relu", normalize_topk=0, n_local=3, zipf=0.0),
    "qwen": dict(d_model=2048, n_experts=60, top_k=4, d_ff=1408, d_ff_shared=5632,
                 vocab_exit=151936, act="swiglu", normalize_topk=0, n_local=20, zipf=0.0),
    "mixtral": dict(d_model=4096, n_experts=8, top_k=2, d_ff=14336, d_ff_shared=0,
                    vocab_exit=32000, act="swiglu", normalize_topk=1, n_local=4, zipf=1.1),
}

POLICY = dict(p_exit=0.9, budget=0.02, omega_t=0.5, t_local=1.0, t_remote=100.0, phi_scale=1.0,
              sim_min=-1.0)

TRANS_B = 4  # entries of an expert transition row (look-ahead)


def _layer(name, shape, tokens, dtype="bf16", horizon=1, per_token=False, conf="softmax"):
    c = dict(kind="layer", shape=shape, tokens=tokens, layers=1, dtype=dtype, horizon=horizon,
             per_token=per_token, conf=conf)
    return dict(c, name=name) if name else c


def _stack(name, shape, tokens, layers, dtype, static, per_token=False, conf="softmax"):
    c = dict(kind="stack", shape=shape, tokens=tokens, layers=layers, dtype=dtype, horizon=1,
             per_token=per_token, conf=conf, static=static)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest model: one request of 64 tokens through both layers;
        # launches and latency are what it costs
        _stack("stack_tiny_f32_64", "tiny", 64, 2, "f32", True),
        # the Switch-Base batch through its whole MoE stack (throughput inference)
        _stack("stack_switch_4096", "switch", 4096, 6, "bf16", False),
        # one user's decode step
        _layer("mixtral_decode_1", "mixtral", 1),
        # the decode batch of the Mixtral configuration
        _layer("mixtral_decode_32", "mixtral", 32),
        # the same decode batch with the look-ahead decision (horizon 3)
        _layer("mixtral_decode_32_h3", "mixtral", 32, horizon=3),
        # a chunk of a prefill scheduled between decode steps, ragged
        _layer("mixtral_chunk_333", "mixtral", 333),
        # the Mixtral prefill batch
        _layer("mixtral_prefill_8192", "mixtral", 8192),
        # a small decode batch over many small experts and a large vocabulary,
        # every request with its own budget and confidence requirement
        _layer("qwen_decode_16", "qwen", 16, per_token=True),
        # an odd prefill batch with a shared expert
        _layer("qwen_prefill_4099", "qwen", 4099),
        # fp32 storage at the Switch-Base shape (validation of a bf16 deployment)
        _layer("switch_f32_777", "switch", 777, dtype="f32"),
        # offline: consistency labels of one layer over a calibration chunk
        dict(kind="labels", name="labels_qwen_2048", vocab=151936, d=2048, rows=2048, dtype="bf16"),
        # offline: one layer's sigmoid exit head, full-batch descent
        dict(kind="train", name="train_head_4096", d=2048, rows=4096, epochs=8, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "chunk", "chunk", "prefill", "stack", "tiny", "f32",
                       "labels", "train"])
    if kind == "decode":
        shape = rng.choice(["mixtral", "qwen", "switch"])
        lookahead = shape == "mixtral" and rng.random() < 0.25
        return _layer(None, shape, _log_int(rng, 1, 64), horizon=rng.choice([2, 3]) if lookahead
                      else 1, per_token=rng.random() < 0.3)
    if kind == "chunk":
        return _layer(None, rng.choice(["mixtral", "qwen", "switch"]), _log_int(rng, 65, 2047),
                      per_token=rng.random() < 0.3,
                      conf="sigmoid" if rng.random() < 0.15 else "softmax")
    if kind == "prefill":
        shape = rng.choice(["mixtral", "qwen", "switch"])
        return _layer(None, shape, _log_int(rng, 2048, 6000 if shape == "qwen" else 8192))
    if kind == "stack":
        return _stack(None, "switch", _log_int(rng, 64, 4096), rng.choice([2, 4, 6]), "bf16", False,
                      per_token=rng.random() < 0.3)
    if kind == "tiny":
        return _stack(None, "tiny", _log_int(rng, 1, 512), 2, rng.choice(["f32", "bf16"]), True)
    if kind == "f32":
        return _layer(None, "switch", _log_int(rng, 8, 777), dtype="f32",
                      per_token=rng.random() < 0.3)
    if kind == "labels":
        d, vocab = rng.choice([(768, 32128), (2048, 151936), (4096, 32000)])
        return dict(kind="labels", vocab=vocab, d=d, rows=_log_int(rng, 64, 2048), dtype="bf16")
    return dict(kind="train", d=64 * _log_int(rng, 1, 64), rows=_log_int(rng, 64, 4096),
                epochs=rng.randint(4, 8), dtype=rng.choice(["bf16", "f32"]))


# ----------------------------------------------------------------- inputs --
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, shape, sigma=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).mul_(sigma)


def _rand(g, shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float32)


def _dt(case):
    return {"bf16": torch.bfloat16, "f32": torch.float32}[case["dtype"]]


def _experts(g, E, shape, sigma, twin, alpha, dt):
    """[E, *shape]: remote experts (twin >= 0) are noisy copies of their twin."""
    out = torch.empty((E,) + shape, dtype=dt, device=DEV)
    order = [e for e in range(E) if twin[e] < 0] + [e for e in range(E) if twin[e] >= 0]
    for e in order:
        w = _randn(g, shape, sigma)
        if twin[e] >= 0:
            w.mul_(math.sqrt(1.0 - alpha[e] ** 2)).add_(out[twin[e]].float(), alpha=alpha[e])
        out[e] = w.to(dt)
    return out


def _make_layer(g, case, S, w_lm, l, n_model_layers):
    E, d, F, Fs = S["n_experts"], S["d_model"], S["d_ff"], S["d_ff_shared"]
    dt = _dt(case)
    perm = torch.randperm(E, generator=g, device=DEV).tolist()
    local = sorted(perm[: S["n_local"]])
    mask = [1 if e in local else 0 for e in range(E)]
    u = _rand(g, (E,)).tolist()
    twin, alpha, n = [-1] * E, [1.0] * E, 0
    for e in range(E):
        if not mask[e]:
            twin[e] = local[n % len(local)]
            alpha[e] = 1.0 - 10.0 ** (-4.0 + 3.0 * u[e])
            n += 1
    # cosines of such experts: unrelated ones near 0, a copy and its twin
    # alpha, two copies of one twin the product
    sim = _randn(g, (E, E), 1e-4)
    sim = (sim + sim.T) / 2
    root = [twin[e] if twin[e] >= 0 else e for e in range(E)]
    for a in range(E):
        for b in range(E):
            if a == b:
                sim[a, b] = 1.0
            elif root[a] == root[b]:
                sim[a, b] = alpha[a] * alpha[b]
    down_sigma = SIGMA / math.sqrt(64.0) if S["act"] == "swiglu" else SIGMA
    b_router = None
    if S["zipf"] > 0:
        rank = torch.randperm(E, generator=g, device=DEV).float()
        b_router = -S["zipf"] * torch.log(rank + 1.0)
        b_router -= b_router.mean()
    gated = S["act"] == "swiglu"
    theta = 0.25 + 0.2 * (l + float(_rand(g, (1,)))) / n_model_layers
    if S["top_k"] > 1:
        theta += 0.3
    # confidences step up with depth
    gamma = 1.0 + 0.5 * ((2 * l) // max(1, n_model_layers - 1)) if n_model_layers > 2 else 1.0
    sigmoid = case["conf"] == "sigmoid"
    L = dict(
        w_router=_randn(g, (E, d), SIGMA).to(dt), b_router=b_router,
        w_up=_experts(g, E, (F, d), SIGMA, twin, alpha, dt),
        w_gate=_experts(g, E, (F, d), SIGMA, twin, alpha, dt) if gated else None,
        w_down=_experts(g, E, (d, F), down_sigma, twin, alpha, dt),
        ws_up=_randn(g, (Fs, d), SIGMA).to(dt) if Fs else None,
        ws_gate=_randn(g, (Fs, d), SIGMA).to(dt) if Fs else None,
        ws_down=_randn(g, (d, Fs), down_sigma).to(dt) if Fs else None,
        w_exit=(w_lm * gamma).to(dt),
        b_exit=_randn(g, (1,), 0.5) if sigmoid else None,
        local_mask=torch.tensor(mask, dtype=torch.uint8, device=DEV), sim=sim.contiguous(),
        theta=theta, skip_slope=0.01 / max(theta, 0.05))
    if case["horizon"] > 1:
        to = torch.stack([torch.randperm(E, generator=g, device=DEV)[:TRANS_B] for _ in range(E)])
        pr = _rand(g, (E, TRANS_B)) ** 3 + 1e-3
        L["trans_to"] = to.to(torch.int16).contiguous()
        L["trans_p"] = (pr / pr.sum(1, keepdim=True)).contiguous()
    return L


# planted strengths: hard tokens, and groups whose confidence passes the
# requirement after the first, a middle or a late exit head
_PLANTS = (7.6, 10.5, 18.0)


def _make_tokens(g, case, S, w_lm, seed_share):
    T, d = case["tokens"], S["d_model"]
    h = _randn(g, (T, d))
    u = _rand(g, (T,))
    if case["conf"] == "sigmoid":
        # the head's own direction, either sign
        v = torch.zeros(T, dtype=torch.int64, device=DEV)
        c = torch.where(u < seed_share, 4.0 + 0.0 * u, -4.0 + 0.0 * u)
    else:
        v = torch.randint(0, w_lm.shape[0], (T,), generator=g, device=DEV)
        c = 3.0 * _rand(g, (T,))
        for i, p in enumerate(_PLANTS):
            lo = seed_share * i / len(_PLANTS)
            c = torch.where((u >= lo) & (u < lo + seed_share / len(_PLANTS)), torch.full_like(c, p), c)
    rows = w_lm[v]
    h += rows * (c / (rows * rows).sum(1))[:, None]
    return h.to(_dt(case))


class _Step:
    """A model, its state and workspace, and the tokens of the next call."""


def _prepare_step(case, seed):
    S = SHAPES[case["shape"]]
    if case["conf"] == "sigmoid":
        S = dict(S, vocab_exit=1)
    g = _gen(seed)
    s = _Step()
    # a layer case is layer 0 of a model deep enough for its exit head and its
    # look-ahead; the later layers of that model stand on the same tensors
    n_model = case["layers"] if case["kind"] == "stack" else max(2, case["horizon"])
    w_lm = _randn(g, (S["vocab_exit"], S["d_model"]), SIGMA)
    s.layers = [_make_layer(g, case, S, w_lm, l, n_model) for l in range(case["layers"])]
    s.layers += [s.layers[0]] * (n_model - case["layers"])
    s.tokens = _make_tokens(g, case, S, w_lm, 0.4)
    del w_lm
    s.dims = dict(S, n_layers=n_model, dtype=case["dtype"], conf_mode=case["conf"])
    s.handle = abi.model_handle(s.dims, s.layers)
    T = case["tokens"]
    s.pol = dict(POLICY, p_exit_tok=None, budget_tok=None, horizon=case["horizon"], la_subs=4)
    if case["per_token"]:
        s.pol["p_exit_tok"] = 0.5 + 0.4 * _rand(g, (T,))
        s.pol["budget_tok"] = 0.04 * _rand(g, (T,))
    s.policy = abi.make_policy(**s.pol)
    s.state = abi.StateBuffers(torch.empty_like(s.tokens))
    s.static = case.get("static", False)
    s.kind = case["kind"]
    s.ws = None if s.static else abi.alloc_workspace(s.handle.model, T, DEV)
    return s


def _prepare_labels(case, seed):
    g = _gen(seed)
    dt = _dt(case)
    s = _Step()
    s.kind = "labels"
    w = _randn(g, (case["vocab"], case["d"]), SIGMA)
    v = torch.randint(0, case["vocab"], (case["rows"],), generator=g, device=DEV)
    rows = w[v]
    c = 12.0 * _rand(g, (case["rows"],))
    s.h = (_randn(g, (case["rows"], case["d"])) + rows * (c / (rows * rows).sum(1))[:, None]).to(dt)
    s.w_head = w.to(dt)
    s.final = v.to(torch.int32)  # the full-depth prediction
    return s


def _prepare_train(case, seed):
    g = _gen(seed)
    s = _Step()
    s.kind = "train"
    s.epochs, s.lr = case["epochs"], 0.5
    h = _randn(g, (case["rows"], case["d"]))
    u = _randn(g, (case["d"],), 1.0 / math.sqrt(case["d"]))
    s.h = h.to(_dt(case))
    s.labels = (h @ u + 0.3 * _randn(g, (case["rows"],)) + 0.5 > 0).to(torch.uint8)
    return s


def prepare(case, seed):
    if case["kind"] == "labels":
        return _prepare_labels(case, seed)
    if case["kind"] == "train":
        return _prepare_train(case, seed)
    return _prepare_step(case, seed)


# ------------------------------------------------------------------- pass --
def run(s):
    if s.kind == "labels":
        pred = abi.trimmoe_head_argmax(s.w_head, s.h)
        return dict(pred=pred, labels=abi.trimmoe_consistency_labels(pred, s.final))
    if s.kind == "train":
        w = torch.zeros(s.h.shape[1], dtype=torch.float32, device=s.h.device)
        c = torch.zeros(1, dtype=torch.float32, device=s.h.device)
        loss = torch.zeros(s.epochs, dtype=torch.float32, device=s.h.device)
        abi.trimmoe_train_exit_head(s.h, s.labels, s.epochs, s.lr, w, c, loss)
        return dict(w=w, c=c, loss=loss)
    st = s.state
    st.h.copy_(s.tokens)  # the call's tokens arrive in the state's buffer
    if s.kind == "layer":
        abi.trimmoe_state_reset(s.handle.model, st.state)
        abi.trimmoe_layer_step(s.handle.model, 0, s.policy, st.state, None, s.ws)
    elif s.static:
        abi.trimmoe_stack_forward_static(s.handle.model, s.policy, st.state, None)
    else:
        abi.trimmoe_stack_forward(s.handle.model, s.policy, st.state, None, s.ws)
    # active_idx holds its first n_active entries only (the tokens whose
    # exit_layer is still the layer count), so exit_layer stands for it
    return dict(h=st.h, d_acc=st.d_acc, xi=st.xi, exit_layer=st.exit_layer, n_active=st.n_active)


# ------------------------------------------------------ work and accuracy --
def _expected_experts(S, draws):
    """Distinct experts that `draws` uniform picks run on average: the local
    ones, and about one remote in seven, whose substitutes exceed the budget."""
    n = S["n_local"] + (S["n_experts"] - S["n_local"]) / 7.0
    return n * (1.0 - (1.0 - 1.0 / n) ** draws)


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "labels":
        V, d, Q = case["vocab"], case["d"], case["rows"]
        return dict(bytes=(V * d + Q * d) * es + 9 * Q, flops=2 * V * d * Q)
    if case["kind"] == "train":
        d, Q, n = case["d"], case["rows"], case["epochs"]
        # the hidden states fit the chip's last-level cache, so one read from
        # memory can serve every epoch
        return dict(bytes=Q * d * es + Q + 4 * d, flops=4 * d * Q * n)
    S = SHAPES[case["shape"]]
    V = 1 if case["conf"] == "sigmoid" else S["vocab_exit"]
    T, d, E, k, F, Fs = (case["tokens"], S["d_model"], S["n_experts"], S["top_k"], S["d_ff"],
                         S["d_ff_shared"])
    mats = 3 if S["act"] == "swiglu" else 2
    total = dict(bytes=2.0 * T * d * es, flops=0.0)
    n_active = float(T)
    for l in range(case["layers"]):
        rows = n_active * k
        total["flops"] += rows * mats * 2 * d * F + n_active * (3 * 2 * d * Fs + 2 * d * E)
        total["bytes"] += es * (_expected_experts(S, rows) * mats * d * F + 3 * d * Fs + E * d)
        if case["kind"] == "layer" or l < case["layers"] - 1:
            total["flops"] += n_active * 2 * d * V
            total["bytes"] += es * V * d
        n_active *= 0.87  # exits (planted share over the exit heads)
    return total


def tolerance(case):
    if case["kind"] == "labels":
        return dict(rel=0.0, differ=0.002)  # near ties of the output head
    if case["kind"] == "train":
        return dict(rel=1e-5, max=1e-4)
    if case["dtype"] == "f32":
        # a decision that falls the other way moves one token of a batch
        return dict(rel=1e-5, max=1e-3, differ=0.005) if case["kind"] == "layer" else \
            dict(rel=1e-4, max=1e-2, differ=0.005)
    if case["kind"] == "stack":
        return dict(rel=0.02, max=0.9, differ=0.005)
    return dict(rel=7e-3, max=0.1, differ=0.002)


# -------------------------------------------------- the same in 64 bits --
def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _substitutes(L, pol):
    """Per expert: its least-loss local substitute (-1: none) and the loss."""
    sim, mask = L["sim"].double(), L["local_mask"].bool()
    E = sim.shape[0]
    q = torch.clamp(_f32(pol["phi_scale"]) * (1.0 - sim) * 0.5, max=1.0)
    ok = mask[None, :] & (sim >= _f32(pol["sim_min"])) & ~torch.eye(E, dtype=torch.bool, device=DEV)
    q = torch.where(ok, q, torch.full_like(q, math.inf))
    best, idx = q.min(1)  # unrelated experts draw distinct losses: no ties matter
    return torch.where(torch.isinf(best), torch.full_like(idx, -1), idx), best


def _decide(L, S, pol, h, D, budget):
    """The H = 1 rule over the rows of h: experts run and weights [n, k], skip, new D."""
    k = S["top_k"]
    z = h @ L["w_router"].double().T
    if L["b_router"] is not None:
        z = z + L["b_router"].double()
    p = torch.softmax(z, 1)
    pv, tgt = torch.topk(p, k, dim=1)
    imp = pv.sum(1)
    w = pv / imp[:, None] if S["normalize_topk"] else pv
    sub, q = _substitutes(L, pol)
    local = L["local_mask"].bool()[tgt]
    can = (~local) & (sub[tgt] >= 0)
    wt = _f32(pol["omega_t"])
    wd = 1.0 - wt
    pos = budget > 0
    safe = torch.where(pos, budget, torch.ones_like(budget))
    n_rem = (~local).sum(1)
    best = torch.full_like(D, math.inf)
    best_sq, best_m, all_local = torch.zeros_like(D), torch.zeros_like(n_rem), torch.zeros_like(pos)
    for m in sorted(range(1 << k), key=lambda m: (bin(m).count("1"), m)):
        take = torch.tensor([(m >> s) & 1 for s in range(k)], dtype=torch.bool, device=DEV)[None, :]
        valid = (can | ~take).all(1)
        sq = torch.where(take & can, q[tgt], torch.zeros_like(pv)).sum(1)
        feas = valid & (D + sq <= budget)
        ns = bin(m).count("1")
        f = wt * ((k - n_rem + ns) * _f32(pol["t_local"]) + (n_rem - ns) * _f32(pol["t_remote"]))
        f = f + torch.where(pos, wd * sq / safe, torch.zeros_like(sq))
        all_local |= feas & (n_rem == ns)
        better = feas & (f < best)
        best = torch.where(better, f, best)
        best_sq = torch.where(better, sq, best_sq)
        best_m = torch.where(better, torch.full_like(best_m, m), best_m)
    lam = torch.clamp(_f32(L["skip_slope"]) * imp, max=1.0)
    fs = torch.where(pos, wd * lam / safe, torch.zeros_like(lam))
    skip = ~all_local & (imp <= _f32(L["theta"])) & (D + lam <= budget) & (fs < best)
    bits = (best_m[:, None] >> torch.arange(k, device=DEV)[None, :]) & 1
    run_e = torch.where(bits.bool(), sub[tgt], tgt)
    return run_e, w, skip, D + torch.where(skip, lam, best_sq)


def _ffn(x, up, gate, down, dt):
    u = x @ up.double().T
    if gate is None:
        a = torch.relu(u)
    else:
        g = x @ gate.double().T
        a = g / (1.0 + torch.exp(-g)) * u
    return a.to(dt).double() @ down.double().T  # activations are stored in dt


def _moe(L, S, x, run_e, w, dt):
    out = torch.zeros_like(x)
    for e in range(S["n_experts"]):
        we = torch.where(run_e == e, w, torch.zeros_like(w)).sum(1)
        rows = torch.nonzero((run_e == e).any(1)).reshape(-1)
        if rows.numel():
            y = _ffn(x[rows], L["w_up"][e], None if L["w_gate"] is None else L["w_gate"][e],
                     L["w_down"][e], dt)
            out[rows] += we[rows][:, None] * y
    if S["d_ff_shared"]:
        out += _ffn(x, L["ws_up"], L["ws_gate"], L["ws_down"], dt)
    return out


def _confidence(L, h, sigmoid):
    w, out = L["w_exit"], []
    for i in range(0, h.shape[0], 512):
        z = torch.cat([h[i:i + 512] @ w[j:j + 16384].double().T for j in range(0, w.shape[0], 16384)], 1)
        if L["b_exit"] is not None:
            z = z + L["b_exit"].double()
        out.append(torch.sigmoid(z[:, 0]) if sigmoid
                   else torch.exp(z.max(1).values - torch.logsumexp(z, 1)))
    return torch.cat(out) if out else h.new_zeros(0)


def _exact_step(case, seed):
    s = _prepare_step(case, seed)
    S, dt, T = s.dims, _dt(case), case["tokens"]
    h = s.tokens.double()  # the state, rounded to its storage type once per layer
    out_h = h.clone()      # ... and its last update before that rounding
    D = torch.zeros(T, dtype=torch.float64, device=DEV)
    xi = torch.full((T,), math.nan, dtype=torch.float64, device=DEV)
    active = torch.ones(T, dtype=torch.bool, device=DEV)

    def per_token(key, scalar):
        t = s.pol[key]
        return torch.full_like(D, _f32(scalar)) if t is None else t.double()

    budget, p_exit = per_token("budget_tok", s.pol["budget"]), per_token("p_exit_tok", s.pol["p_exit"])
    n_layers = len(s.layers)
    for l in range(case["layers"]):
        L = s.layers[l]
        idx = torch.nonzero(active).reshape(-1)
        if not idx.numel():
            break
        run_e, w, skip, D[idx] = _decide(L, S, s.pol, h[idx], D[idx], budget[idx])
        ex = idx[~skip]
        new = h[ex] + _moe(L, S, h[ex], run_e[~skip], w[~skip], dt)
        out_h[ex] = new
        h[ex] = new.to(dt).double()
        if l < n_layers - 1:
            conf = _confidence(L, new, case["conf"] == "sigmoid")
            xi[ex] = conf
            active[ex[conf >= p_exit[ex]]] = False
    return dict(h=out_h, d_acc=D, xi=xi, exit_layer=None, n_active=None)


def exact(case, seed):
    if case["kind"] == "labels":
        return None  # whole numbers only
    if case["kind"] == "train":
        s = _prepare_train(case, seed)
        h, y, lr = s.h.double(), s.labels.double(), _f32(s.lr)
        w = torch.zeros(h.shape[1], dtype=torch.float64, device=DEV)
        c, losses = torch.zeros(1, dtype=torch.float64, device=DEV), []
        for _ in range(s.epochs):
            z = h @ w + c
            losses.append((torch.clamp(z, min=0) - y * z + torch.log1p(torch.exp(-z.abs()))).mean())
            r = torch.sigmoid(z) - y
            w = w - lr * (r @ h) / h.shape[0]
            c = c - lr * r.mean()
        return dict(w=w, c=c, loss=torch.stack(losses))
    if case["horizon"] > 1:
        return None  # the recursion of the look-ahead is not a plain expression
    return _exact_step(case, seed)
