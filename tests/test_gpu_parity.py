"""GPU parity of the HIP path (through the C ABI) against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from synthgen import make_inputs, workload

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests.gpu_harness import (GpuRun, check_invariants_gpu, compare_stack, gpu_state_np,
                                   gpu_trace_np, log, oracle_run, policy32, teacher_forced)


def _run_and_compare(cfg, pol=None, edit=None, **kw):
    inp = make_inputs(cfg)
    if edit is not None:
        edit(inp)
    log(f"[parity] {cfg['name']} T={cfg['n_tokens']} N={cfg['n_layers']} {kw}")
    g = GpuRun(inp)
    st, tr = g.stack(pol=pol, **{k: v for k, v in kw.items() if k in ("p_exit_tok", "budget_tok")})
    gst, gtr = gpu_state_np(st), gpu_trace_np(tr)
    ref_state, ref_traces = oracle_run(inp, pol=pol, token_budget=kw.get("budget_tok"),
                                       token_p_exit=kw.get("p_exit_tok"))
    stats = compare_stack(cfg, ref_state, ref_traces, gst, gtr)
    check_invariants_gpu(cfg, policy32(inp["policy"] if pol is None else pol), gst, gtr,
                         kw.get("budget_tok"), kw.get("p_exit_tok"))
    log(f"[parity] ok {stats}")
    return inp, gst, gtr, ref_state, ref_traces, stats


def test_tiny_fp32_stack():
    cfg = workload("tiny_fp32")
    _, gst, gtr, ref, _, stats = _run_and_compare(cfg)
    assert stats["excluded_tokens"] <= 4
    # the recipe reaches every branch of the rule on this case
    assert (gtr["action"] == O.ACT_SKIP).any()
    assert (gtr["kind"] == O.KIND_SUB).any()
    assert (gst["exit_layer"] < cfg["n_layers"]).any()


def test_tiny_bf16_swiglu_top2_shared():
    cfg = workload("tiny_fp32", dtype="bf16", act="swiglu", top_k=2, d_ff_shared=128,
                   normalize_topk=1, n_layers=3)
    _run_and_compare(cfg)


@pytest.mark.parametrize("dtype,act", [("f32", "relu"), ("f32", "swiglu"), ("bf16", "relu")])
def test_shared_expert_with_every_routed_activation(dtype, act):
    # the shared expert (SwiGLU) beside ReLU or SwiGLU routed experts, on the
    # fp32 path and beside ReLU on the bf16 path (the bf16 SwiGLU case is
    # above); 200 tokens leave ragged route, row and token tiles
    cfg = workload("tiny_fp32", dtype=dtype, act=act, top_k=2, normalize_topk=1,
                   d_ff_shared=192, n_tokens=200, n_layers=3)
    _run_and_compare(cfg)


def test_large_batch_swiglu_top2_shared():
    # 6144 tokens: the 256-token exit-head tile; top-2 over 4 experts gives
    # long, ragged expert groups
    cfg = workload("tiny_fp32", dtype="bf16", act="swiglu", top_k=2, normalize_topk=1,
                   n_tokens=6144, d_model=128, d_ff=256, n_experts=4, n_local=2,
                   vocab_exit=2048, n_layers=3, d_ff_shared=256)
    _run_and_compare(cfg)


def test_large_batch_relu_top1():
    cfg = workload("switch_base_8e", n_tokens=6500, n_layers=3, d_model=128, d_ff=384,
                   n_experts=2, n_local=1, vocab_exit=1500)
    _run_and_compare(cfg)


def test_large_expert_groups_skewed_ragged():
    # Mixtral-like routing (top-2 of 8, Zipf-skewed router bias) at 4096
    # tokens: 1024 rows per expert on average, so the expert GEMMs take
    # 256-row tiles; d_ff = 576 and d_model = 320 leave partial column tiles
    # in the up/gate (128-column) and down (256-column) GEMMs
    cfg = workload("mixtral_8x7b_prefill", n_tokens=4096, n_layers=2, d_model=320, d_ff=576,
                   vocab_exit=1000)
    # the library picks 256-row tiles from the batch shape: T k >= 1024 E
    assert cfg["n_tokens"] * cfg["top_k"] >= 1024 * cfg["n_experts"]
    _run_and_compare(cfg)


def test_decode_sized_swiglu_split_down_ragged():
    # a decode-sized batch (29 tokens, a few rows per expert) at bf16:
    # d_model 576 leaves a partial 256-column down tile, d_ff 1152 gives the
    # down GEMM two K splits, and the exit head takes its decode tile
    # (vocabulary 1000: a partial 128-row tile)
    cfg = workload("mixtral_8x7b_decode", n_tokens=29, n_layers=3, d_model=576, d_ff=1152,
                   vocab_exit=1000)
    _run_and_compare(cfg)


def test_decode_sized_relu_top1_ragged_up():
    # ReLU up tiles (256 columns) over d_ff 704 leave a partial tile; 32
    # tokens over 8 experts
    cfg = workload("switch_base_8e", n_tokens=32, n_layers=3, d_model=512, d_ff=704,
                   vocab_exit=1000)
    _run_and_compare(cfg)


@pytest.mark.parametrize("dtype,E,k,d,T", [
    ("bf16", 16, 8, 64, 9),       # one column tile; K of one slice; every slot count
    ("bf16", 17, 2, 832, 300),    # two column tiles; a partial last slice
    ("bf16", 48, 5, 576, 40),     # three column tiles, two of the eight wavefronts idle
    ("bf16", 65, 4, 192, 700),    # five column tiles; 16-token blocks
    ("bf16", 129, 3, 128, 33),    # nine column tiles: a wavefront takes two
    ("bf16", 16, 2, 64, 8225),    # more blocks than CUs, one K slice; a block of one token
    ("bf16", 5, 2, 448, 8600),    # ... slices of the small ring with a remainder
    ("f32", 8, 2, 528, 5000),     # fp32 steps of 16 K; 32-token blocks
    ("f32", 33, 4, 72, 20),       # fp32 rows of a partial step: FMA logits
    ("f32", 256, 8, 64, 50),      # the most experts and slots
])
def test_route_blocks(dtype, E, k, d, T):
    # router logits through the LDS ring, top-k, and the register form of the
    # decision, at the edges of their tiles and loops
    cfg = workload("tiny_fp32", dtype=dtype, n_experts=E, n_local=max(1, E // 2), top_k=k,
                   d_model=d, d_ff=64, n_tokens=T, vocab_exit=200, n_layers=2,
                   normalize_topk=1, budget=0.05)
    _, _, gtr, _, _, _ = _run_and_compare(cfg)
    assert (gtr["kind"] == O.KIND_SUB).any()


@pytest.mark.parametrize("E,T,p_exit", [
    (64, 500, 0.5),    # the last expert count one wavefront scans (63 route blocks)
    (65, 500, 0.5),    # ... and the first of the block-wide scans
    (1, 1023, 0.5),    # one expert over every route block
    (33, 100, 0.0),    # later layers route no token
])
def test_bucket_scans(E, T, p_exit):
    cfg = workload("tiny_fp32", n_tokens=T, n_experts=E, n_local=max(1, E // 2), d_ff=32,
                   vocab_exit=50, n_layers=3, p_exit=p_exit)
    _run_and_compare(cfg)


@pytest.mark.parametrize("act,T,k,E,d,F,Fs,V", [
    ("swiglu", 1, 1, 1, 64, 64, 0, 1000),       # K of two k-steps: half the wavefronts idle
    ("relu", 16, 1, 2, 128, 192, 64, 17),       # one full 16-row tile; one row past a group
    ("swiglu", 17, 2, 2, 192, 320, 0, 128),     # every expert sees 17 rows: a second row tile
    ("relu", 33, 1, 1, 320, 704, 192, 130),     # a third row tile: the widest streams
    ("swiglu", 64, 1, 1, 1088, 576, 64, 515),   # the largest batch; clipped last sets
    ("swiglu", 64, 4, 16, 256, 1408, 128, 3000),
    ("swiglu", 65, 2, 4, 256, 128, 64, 1000),   # the first batch of the 128-row tiles
])
def test_weight_streaming_edges(act, T, k, E, d, F, Fs, V):
    # decode-sized batches: row tiles of 16, odd column groups per block, and
    # K quarters of whole, clipped and empty sets
    cfg = workload("tiny_fp32", dtype="bf16", act=act, n_tokens=T, top_k=k, n_experts=E,
                   n_local=max(1, E // 2), d_model=d, d_ff=F, d_ff_shared=Fs, vocab_exit=V,
                   normalize_topk=1, n_layers=3)
    _run_and_compare(cfg)


def _width_changes(rows, N):
    """Changes of the row-tile width (up to 16, 32 or more rows) inside one
    block's range of 16-column groups (row tiles of experts with rows, N
    columns each, dealt evenly to a block per CU)."""
    w = [1 if r <= 16 else 2 if r <= 32 else 4 for r in rows if r > 0]
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    npt, out = N // 16, set()
    total = npt * len(w)
    for v in range(n_cu):
        ts = sorted({g // npt for g in range(total * v // n_cu, total * (v + 1) // n_cu)})
        out |= {(w[a], w[b]) for a, b in zip(ts, ts[1:]) if w[a] != w[b]}
    return out


@pytest.mark.parametrize("skew", [(1.6, -1.0, 0.5, -1.0, 1.6, 0.5, -1.0),
                                  (-1.0, 0.5, 1.6, -1.0, 1.6, -1.0, 0.5)])
@pytest.mark.parametrize("act,d,F", [
    ("swiglu", 64, 2496),   # K of two k-steps: wavefronts without one join the sums at once
    ("relu", 128, 2496),
    ("relu", 192, 2496),
    ("swiglu", 2496, 64),   # ... in the down projection
    ("relu", 2496, 128),
    ("swiglu", 2496, 192),
    ("swiglu", 1088, 2496),  # long K, both projections
])
def test_weight_streaming_row_tiles_of_different_width(act, d, F, skew):
    # a block goes on from one expert's row tile to another's of a different
    # width: the sums' LDS area changes its layout
    cfg = workload("tiny_fp32", dtype="bf16", act=act, n_tokens=64, top_k=2, n_experts=len(skew),
                   n_local=3, d_model=d, d_ff=F, vocab_exit=130, normalize_topk=1, n_layers=2)

    def edit(inp):
        for L in inp["layers"]:
            L["b_router"] = torch.tensor(skew) * (0.02 * d ** 0.5)
    # no budget: every token runs its own experts
    pol = dict(make_inputs(cfg, with_layers=False)["policy"], budget=0.0)
    _, _, gtr, _, _, _ = _run_and_compare(cfg, pol=pol, edit=edit)
    rows = [int((gtr["exec"][0] == e).sum()) for e in range(len(skew))]
    assert _width_changes(rows, F) | _width_changes(rows, d), rows


@pytest.mark.parametrize("T,d,V", [
    (16, 64, 16),       # streaming: one group of rows, K of two k-steps
    (32, 128, 16),
    (33, 128, 16),      # ... and the first batch of its tiles
    (16, 1984, 515),    # tiles: the longest rows that are not streamed
    (1, 2048, 130),     # streaming: rows from here on,
    (16, 2112, 515),    # ... up to 16 tokens
    (17, 2112, 515),    # tiles
    (64, 2048, 24575),
    (64, 2048, 24576),  # streaming: and beyond 16 tokens with this many rows
    (20, 2112, 24601),
])
def test_decode_sized_exit_heads(T, d, V):
    # both exit kernels of a decode-sized batch at the borders of their rule
    cfg = workload("tiny_fp32", dtype="bf16", n_tokens=T, n_experts=2, n_local=1, d_model=d, d_ff=64,
                   vocab_exit=V, n_layers=2)
    _run_and_compare(cfg)


@pytest.mark.parametrize("T", [1, 16, 33, 64])
@pytest.mark.parametrize("d", [64, 704, 2048])
def test_decode_sized_sigmoid_heads(T, d):
    cfg = workload("tiny_fp32", dtype="bf16", n_tokens=T, n_experts=2, n_local=1, d_model=d, d_ff=64,
                   vocab_exit=1, n_layers=2, conf_mode="sigmoid")
    _run_and_compare(cfg)


@pytest.mark.parametrize("act,T,k,E,d,F,Fs,V", [
    ("relu", 64, 1, 8, 64, 256, 0, 130),        # two K slices; a partial vocabulary tile
    ("swiglu", 65, 2, 4, 96, 160, 64, 1),       # three slices; the 128-token exit tile
    ("relu", 300, 1, 2, 32, 2080, 0, 300),      # one slice; 64-column tiles, ragged rows
    ("swiglu", 300, 1, 2, 64, 4128, 96, 257),   # 64-column SwiGLU tiles with a remainder
    ("relu", 300, 1, 4, 64, 8224, 0, 100),      # 128-column tiles with a remainder
    ("swiglu", 130, 2, 4, 64, 100, 33, 70),     # F and Fs of partial slices: FMA down kernels
    ("relu", 40, 1, 4, 40, 64, 0, 70),          # d of a partial slice: FMA up and exit kernels
])
def test_fp32_tiles(act, T, k, E, d, F, Fs, V):
    # fp32 models: the fp32 MFMA tiles at their widths and remainders, and the
    # FMA kernels of rows that are not whole K slices
    cfg = workload("tiny_fp32", act=act, n_tokens=T, top_k=k, n_experts=E, n_local=max(1, E // 2),
                   d_model=d, d_ff=F, d_ff_shared=Fs, vocab_exit=V, normalize_topk=1, n_layers=3,
                   conf_mode="sigmoid" if V == 1 else "softmax")
    _run_and_compare(cfg)


@pytest.mark.parametrize("T,k,E,d,F", [
    (70, 1, 2, 64, 8192),     # few tiles, long K: eight splits fit the workspace or fewer
    (130, 2, 8, 320, 1024),   # two splits of eight slices; partial column tiles
    (400, 1, 3, 128, 1088),   # 17 K slices: no even split
])
def test_live_down_splits(T, k, E, d, F):
    # the down GEMM's K split follows the live tiles; the combine adds the slices
    cfg = workload("tiny_fp32", dtype="bf16", act="swiglu", n_tokens=T, top_k=k, n_experts=E,
                   n_local=max(1, E // 2), d_model=d, d_ff=F, vocab_exit=300, n_layers=3,
                   normalize_topk=1)
    _run_and_compare(cfg)


@pytest.mark.parametrize("act,T,k,E,d,F,Fs", [
    ("swiglu", 300, 2, 8, 64, 4224, 0),    # 33 column tiles: more than a round, short K
    ("swiglu", 500, 2, 2, 2048, 4224, 0),  # a full round, the rest in halves
    ("relu", 1000, 1, 2, 2112, 8448, 0),
    ("relu", 90, 1, 4, 128, 512, 0),       # less than a round: halves only
    ("swiglu", 90, 1, 2, 128, 192, 0),     # a column tile cut short: no halves
    ("swiglu", 101, 1, 2, 192, 64, 320),   # shared expert: a second pass over the weights
    ("relu", 128, 1, 2, 64, 64, 1152),     # ... of two whole row tiles
    ("swiglu", 129, 1, 2, 320, 64, 576),   # its down GEMM in 64-column tiles,
    ("swiglu", 1900, 1, 2, 1152, 64, 64),  # ... 128 (15 row tiles x 18 of 64 columns)
    ("swiglu", 2047, 1, 2, 2112, 64, 128),  # ... and 256 (16 x 17 of 128)
])
def test_last_round_halves_and_shared_expert_tiles(act, T, k, E, d, F, Fs):
    # no budget: every token runs its own experts, so the tile counts are these
    cfg = workload("tiny_fp32", dtype="bf16", act=act, n_tokens=T, top_k=k, n_experts=E,
                   n_local=max(1, E // 2), d_model=d, d_ff=F, d_ff_shared=Fs, vocab_exit=70,
                   normalize_topk=1, n_layers=2)
    inp = make_inputs(cfg)
    _run_and_compare(cfg, pol=dict(inp["policy"], budget=0.0))


def test_wide_model_exit_head_ragged():
    # d_model 2048 at 1100 tokens: the exit head takes 256 x 256 tiles with
    # 4 wavefronts; 1100 tokens and 1000 vocabulary rows leave partial token
    # and vocabulary tiles
    cfg = workload("tiny_fp32", dtype="bf16", n_tokens=1100, d_model=2048, d_ff=256,
                   n_experts=4, n_local=2, vocab_exit=1000, n_layers=2)
    _run_and_compare(cfg)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sigmoid_exit_head(dtype):
    # the paper's own exit head: one logit w . h + b through a sigmoid
    # (p_J = 0.99: the planted logits cross 4.6 at different depths)
    cfg = workload("tiny_fp32", dtype=dtype, vocab_exit=1, conf_mode="sigmoid", n_layers=4,
                   n_tokens=200, p_exit=0.99)
    _, gst, gtr, _, _, _ = _run_and_compare(cfg)
    exits = [(gst["exit_layer"] == l).sum() for l in range(cfg["n_layers"])]
    assert sum(e > 0 for e in exits) >= 2


def test_many_experts_bf16_top4_substitution():
    # 160 SwiGLU experts, top-4, 80 local, in bf16: each lane of the
    # substitute table's wavefront scans two or three candidates (160 =
    # 2 x 64 + 32) and the router's MFMA tiles span 10 expert column tiles
    cfg = workload("qwen_moe_a2_7b", n_tokens=512, n_layers=2, d_model=256, d_ff=128,
                   d_ff_shared=128, n_experts=160, n_local=80, vocab_exit=1000)
    _, _, gtr, _, _, _ = _run_and_compare(cfg)
    assert (gtr["kind"] == O.KIND_SUB).any()
    assert (gtr["action"] == O.ACT_SKIP).any()


def test_max_experts_and_top_k_bf16():
    # the library's maxima together: 256 SwiGLU experts, top-8, 128 of them
    # local, bf16 (a whole wavefront per token in top-k and softmax, every
    # token's Eq. (34) enumeration over 8 slots, up to 256 groups of a few
    # rows in the expert GEMMs), 300 tokens (a ragged route block)
    cfg = workload("qwen_moe_a2_7b", n_tokens=300, n_layers=2, d_model=128, d_ff=128,
                   d_ff_shared=128, n_experts=256, n_local=128, top_k=8, vocab_exit=512)
    _, _, gtr, _, _, _ = _run_and_compare(cfg)
    assert (gtr["kind"] == O.KIND_SUB).any()
    assert (gtr["action"] == O.ACT_SKIP).any()


@pytest.mark.parametrize("E,k", [(8, 2), (60, 4)])
def test_tied_router_logits_rank_lower_id_first(E, k):
    # router rows duplicated in pairs: experts 2j and 2j + 1 get bitwise equal
    # logits, so the rank order takes 2j first and its twin right after it
    # (8 experts: 8-lane groups per token; 60: a whole wavefront per token)
    cfg = workload("tiny_fp32", dtype="bf16", n_experts=E, n_local=E // 2, top_k=k,
                   normalize_topk=1, n_tokens=300, n_layers=2)

    def tie(inp):
        for L in inp["layers"]:
            L["w_router"][1::2] = L["w_router"][0::2]

    _, _, gtr, _, _, _ = _run_and_compare(cfg, edit=tie)
    tgt = gtr["target"].reshape(cfg["n_layers"], cfg["n_tokens"], k)
    live = tgt[..., 0] >= 0
    for r in range(0, k, 2):
        assert np.all(tgt[..., r][live] % 2 == 0)
        assert np.all(tgt[..., r + 1][live] == tgt[..., r][live] + 1)


def test_ragged_tokens_bf16_relu():
    # T not a multiple of any tile (route 32, GEMM 128)
    cfg = workload("switch_base_8e", n_tokens=333, n_layers=3, d_model=256, d_ff=512,
                   vocab_exit=1000)
    _run_and_compare(cfg)


def test_single_token():
    cfg = workload("tiny_fp32", n_tokens=1, n_layers=3)
    _run_and_compare(cfg)


def test_all_tokens_exit_after_first_layer():
    # p_J = 0: every token exits after layer 0, later layers see n_active = 0
    cfg = workload("tiny_fp32", n_layers=4)
    inp = make_inputs(cfg)
    pol = dict(inp["policy"], p_exit=0.0)
    _, gst, gtr, _, _, _ = _run_and_compare(cfg, pol=pol)
    # a token exits right after its first executed layer; a skipped layer
    # never triggers an exit (Eq. (9)), so skippers stay active until then
    act = gtr["action"]
    for t in range(cfg["n_tokens"]):
        first = int(np.argmax(act[:, t] == O.ACT_EXEC)) if (act[:, t] == O.ACT_EXEC).any() else None
        if first is not None and first < cfg["n_layers"] - 1:
            assert gst["exit_layer"][t] == first
            assert np.all(act[first + 1:, t] == O.ACT_INACTIVE)
            assert np.all(act[:first, t] == O.ACT_SKIP)
    assert (act[0] == O.ACT_EXEC).sum() > 0


def test_zero_budget_and_per_token_arrays():
    cfg = workload("tiny_fp32", n_layers=3)
    inp = make_inputs(cfg)
    T = cfg["n_tokens"]
    budget_tok = np.where(np.arange(T) % 2 == 0, 0.0, 0.05).astype(np.float32)
    pexit_tok = np.where(np.arange(T) % 3 == 0, 2.0, 0.5).astype(np.float32)
    _, gst, _, _, _, _ = _run_and_compare(cfg, budget_tok=budget_tok, p_exit_tok=pexit_tok)
    assert np.all(gst["d_acc"][budget_tok == 0] == 0)


def test_switch_base_full_size():
    # the benchmark workload: 6 layers, d=768, 8 experts top-1, 4096 tokens
    cfg = workload("switch_base_8e")
    _, gst, gtr, _, _, stats = _run_and_compare(cfg)
    # a token leaves the comparison at its first decision within 1e-3 of a
    # threshold; over 6 layers that is ~8% of tokens on this recipe
    assert stats["excluded_tokens"] < 0.10 * cfg["n_tokens"]
    c = gtr["counters"]
    log(f"[switch] counters per layer (active, exec, skip, exit, subst, remote, rows, experts):\n{c}")
    assert c[:, 2].sum() > 0 and c[:, 3].sum() > 0 and c[:, 4].sum() > 0


def test_determinism_bitwise():
    cfg = workload("switch_base_8e", n_tokens=1024, n_layers=3)
    inp = make_inputs(cfg)
    g = GpuRun(inp)
    st1, tr1 = g.stack()
    st2, tr2 = g.stack()
    assert torch.equal(st1.h, st2.h)
    for k in ("action", "exec", "gate", "xi", "d_acc", "counters"):
        assert torch.equal(getattr(tr1, k).nan_to_num(0) if getattr(tr1, k).is_floating_point()
                           else getattr(tr1, k),
                           getattr(tr2, k).nan_to_num(0) if getattr(tr2, k).is_floating_point()
                           else getattr(tr2, k)), k


@pytest.mark.parametrize("shape", ["large_groups", "wide_exit"])
def test_determinism_bitwise_large_tiles(shape):
    # the large-group expert GEMMs (256-row tiles, dense shared expert) and the
    # large-tile exit head: fixed K order and no atomics, so repeated passes
    # are bit-identical
    if shape == "large_groups":
        cfg = workload("tiny_fp32", dtype="bf16", act="swiglu", top_k=2, normalize_topk=1,
                       n_tokens=4096, d_model=192, d_ff=320, n_experts=4, n_local=2,
                       vocab_exit=700, n_layers=2, d_ff_shared=256)
    else:
        cfg = workload("tiny_fp32", dtype="bf16", n_tokens=1100, d_model=2048, d_ff=256,
                       n_experts=4, n_local=2, vocab_exit=1000, n_layers=2)
    g = GpuRun(make_inputs(cfg))
    st1, tr1 = g.stack()
    st2, tr2 = g.stack()
    assert torch.equal(st1.h, st2.h)
    for k in ("action", "exec", "gate", "xi", "d_acc", "counters"):
        a, b = getattr(tr1, k), getattr(tr2, k)
        if a.is_floating_point():
            a, b = a.nan_to_num(0), b.nan_to_num(0)
        assert torch.equal(a, b), k


def test_switch_base_teacher_forced_layers():
    # every layer of the benchmark workload on 1024 tokens, fed the oracle's
    # exact state: decisions bit-exact outside a 1e-5 band
    cfg = workload("switch_base_8e", n_tokens=1024)
    stats = teacher_forced(make_inputs(cfg))
    assert sum(s["excluded_tokens"] for s in stats) < 0.01 * 1024 * cfg["n_layers"]


def test_tiny_fp32_teacher_forced():
    teacher_forced(make_inputs(workload("tiny_fp32", n_layers=3)))
