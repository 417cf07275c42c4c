"""GPU parity: the HIP path behind the C ABI against the fp64 oracle, element by element, under
teacher forcing.  Tolerances (relative to the tensor's largest magnitude): 1e-4 for float32
models, 2e-2 for bfloat16 models; integer state, row sets and decisions are bit-exact (decisions
wherever the oracle's margins exceed the tolerance)."""
import math

import numpy as np
import pytest

import ec_inputs
import paper_2603_18489_amd as ec
from oracle import entropycache as eco
from tests.gpu_harness import run_teacher_forced, run_teacher_forced_batch, relerr

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2, "fp8w": 2e-2}


def small_cfg(dtype, hq=4, hkv=4, hd=64, d=256, f=768, vocab=4096, layers=2, scale=16.0):
    return ec_inputs.ModelCfg(n_layers=layers, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd,
                              d_ffn=f, vocab=vocab, mask_id=vocab - 1, rms_eps=1e-5,
                              rope_base=10000.0, logit_scale=scale, dtype=dtype)


def block_shape(cfg, product, T):
    """blocks of a product over the T rows of one sequence's full step (its list is padded to 256)"""
    return ec.block_shape(cfg, product, (T + 255) // 256 * 256, T)


def full_step_attn_tiles(cfg, lengths):
    """row tiles to a block of the attention in a full step of sequences of these lengths (those of up to 96 rows go elsewhere)"""
    many = [T for T in lengths if T > 96]
    return ec.attn_tiles(cfg, many, many)


def test_tiny_f32_whole_generation():
    wl = ec_inputs.WORKLOADS["tiny_f32"]
    cfg = wl.model.replace(logit_scale=16.0)      # both modes occur (about half the steps FULL)
    w = ec_inputs.make_weights(cfg, wl.seed, gain_jitter=0.1)
    prompt = ec_inputs.make_prompt(cfg.vocab, wl.prompt_len, wl.seed)
    s = run_teacher_forced(cfg, w, wl.decode, prompt, TOL["f32"])
    print(s)
    assert s["steps"] == 64 and s["modes"][eco.FULL] >= 2 and s["modes"][eco.PARTIAL] >= 10
    assert s["exact_checked"] >= 32


@pytest.mark.parametrize("dtype,hq,hkv,hd,P,N,block,k,n,tau", [
    ("f32", 4, 2, 64, 37, 45, 16, 3, 2, 2.5),       # GQA, ragged last block, T not / 16
    ("f32", 2, 1, 128, 5, 9, 32, 0, 1, 1e9),        # gen shorter than block, k = 0, head_dim 128
    ("bf16", 4, 4, 64, 64, 64, 32, 2, 1, 3.0),
    ("bf16", 4, 2, 128, 50, 70, 32, 4, 2, 2.5),     # GQA, head_dim 128, 70 = 2 blocks + 6
    ("bf16", 8, 2, 64, 100, 33, 32, 2, 3, 1e9),     # T = 133 > 128 rows: tiled GEMM in FULL
    ("bf16", 4, 2, 64, 40, 128, 32, 64, 1, 1e9),    # k = 64: partial steps of 65 .. 96 rows
])
def test_small_models_whole_generation(dtype, hq, hkv, hd, P, N, block, k, n, tau):
    cfg = small_cfg(dtype, hq, hkv, hd, d=hq * hd if hq * hd >= 256 else 256)
    w = ec_inputs.make_weights(cfg, 7, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=N, block=block, k_recent=k, tokens_per_step=n, tau=tau)
    prompt = ec_inputs.make_prompt(cfg.vocab, P, 3)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL[dtype])
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0 and s["modes_exact"] > 0


@pytest.mark.parametrize("dtype,thr,metric,tau,scale", [
    ("f32", 0.5, ec.EC_GATE_MAX_ENTROPY, 2.5, 13.0),
    ("f32", 0.35, ec.EC_GATE_ENTROPY_SUM, 4.0, 13.0),
    ("f32", 0.5, ec.EC_GATE_MAX_CONFIDENCE, 0.3, 13.0),
    ("bf16", 0.5, ec.EC_GATE_MAX_ENTROPY, 2.5, 13.0),
    ("bf16", 0.5, ec.EC_GATE_ENTROPY_SUM, 6.0, 13.0),
])
def test_confidence_threshold_decoding_and_gate_metrics(dtype, thr, metric, tau, scale):
    """Confidence-based parallel decoding (several tokens per step, the recent set grows by ties)
    and the alternative thresholding variables, against the oracle under teacher forcing."""
    cfg = small_cfg(dtype, 4, 2, 64, scale=scale)
    w = ec_inputs.make_weights(cfg, 17, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=80, block=32, k_recent=4, tokens_per_step=1, tau=tau,
                              conf_threshold=thr, gate_metric=metric)
    prompt = ec_inputs.make_prompt(cfg.vocab, 45, 9)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL[dtype])
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["modes"][eco.FULL] >= 1
    assert s["steps"] < 80, "no step decoded several tokens: the threshold path did not run"
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0 and s["modes_exact"] > 0


@pytest.mark.parametrize("dtype,block,k,n,thr,tau", [
    ("f32", 16, 3, 2, 0.0, 2.5),      # window slides by two slots a step
    ("bf16", 32, 4, 1, 0.5, 2.5),     # with confidence-based parallel decoding
])
def test_sliding_window_schedule(dtype, block, k, n, thr, tau):
    """Sliding-window decoding: M^t is the leftmost `block` masked slots, so the row sets differ
    from the blockwise ones at every step."""
    cfg = small_cfg(dtype, 4, 2, 64, scale=13.0)
    w = ec_inputs.make_weights(cfg, 17, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=70, block=block, k_recent=k, tokens_per_step=n, tau=tau,
                              conf_threshold=thr, schedule=ec.EC_SCHED_SLIDING)
    prompt = ec_inputs.make_prompt(cfg.vocab, 45, 9)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL[dtype])
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["modes"][eco.FULL] >= 1
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0 and s["modes_exact"] > 0


@pytest.mark.parametrize("hq,hkv,hd", [(4, 4, 64), (4, 2, 128)])
def test_long_context_partial_steps(hq, hkv, hd):
    """More than 2048 keys: the partial-step attention cuts the keys into slices that different
    blocks reduce and the last one to finish adds up."""
    cfg = small_cfg("bf16", hq, hkv, hd, d=hq * hd if hq * hd >= 256 else 256)
    w = ec_inputs.make_weights(cfg, 11, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=40, block=32, k_recent=3, tokens_per_step=2, tau=1e9)
    prompt = ec_inputs.make_prompt(cfg.vocab, 2100, 5)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL["bf16"], max_steps=8)
    print(s)
    assert s["modes"][eco.PARTIAL] >= 6
    assert s["tokens_exact"] > 0 and s["modes_exact"] > 0


@pytest.mark.parametrize("hq,hkv,hd,plens,N,block,k,n,tau,fast", [
    (4, 4, 64, [40, 100, 7], 40, 16, 2, 2, 3.0, None),      # ragged prompts, mixed modes
    (4, 2, 128, [70, 9, 33, 150], 36, 32, 3, 1, 2.5, 1),    # GQA; sequence 1 finishes early;
                                                             # 150 + 36 rows: a many-row sequence
])
def test_batched_sequences_match_their_own_oracle_runs(hq, hkv, hd, plens, N, block, k, n, tau, fast):
    """Sequences of a batch are independent: each must reproduce the oracle run on it alone,
    whatever modes the others are in and after some of them have finished."""
    cfg = small_cfg("bf16", hq, hkv, hd, d=hq * hd if hq * hd >= 256 else 256)
    w = ec_inputs.make_weights(cfg, 13, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=N, block=block, k_recent=k, tokens_per_step=n, tau=tau,
                              batch=len(plens))
    prompts = [ec_inputs.make_prompt(cfg.vocab, P, 20 + i) for i, P in enumerate(plens)]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL["bf16"], fast_seq=fast)
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["modes"][eco.FULL] >= len(plens)
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0 and s["modes_exact"] > 0
    if fast is not None:
        assert s["finished_early"] >= 1


def test_tile_counts_that_do_not_divide_the_block_widths():
    """Feature counts whose 16-row tiles are not a multiple of the tiles a GEMM block owns:
    772 gate/up tiles in groups of 3, 257 vocabulary tiles in groups of 4 (the last group of the
    packed layout is partly empty, the last block's surplus tiles must be dropped)."""
    cfg = small_cfg("bf16", 4, 2, 64, f=6176, vocab=4112)
    w = ec_inputs.make_weights(cfg, 37, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=40, block=32, k_recent=2, tokens_per_step=2, tau=3.0)
    prompt = ec_inputs.make_prompt(cfg.vocab, 150, 8)    # 190 rows in FULL steps: tiled GEMMs
    s = run_teacher_forced(cfg, w, dec, prompt, TOL["bf16"])
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["modes"][eco.FULL] >= 1
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0 and s["modes_exact"] > 0


def _random_case(seed):
    r = np.random.RandomState(seed)
    hkv, hd = int(r.choice([1, 2, 4])), int(r.choice([64, 128]))
    hq = hkv * int(r.choice([1, 2, 4])) if hd == 64 else hkv * int(r.choice([1, 2]))
    return dict(dtype=str(r.choice(["f32", "bf16"])), hq=hq, hkv=hkv, hd=hd,
                P=int(r.randint(0, 90)), N=int(r.randint(5, 70)), block=int(r.choice([4, 8, 16, 32])),
                k=int(r.randint(0, 12)), n=int(r.randint(1, 4)), tau=float(r.choice([1.5, 2.5, 3.5, 1e9])),
                thr=float(r.choice([0.0, 0.0, 0.4])), metric=int(r.choice([0, 0, 1, 2])),
                schedule=int(r.choice([0, 1])), scale=float(r.choice([10.0, 13.0, 16.0])))


@pytest.mark.parametrize("seed", list(range(100, 112)))
def test_random_configurations(seed):
    """Seeded sweep over head layouts, sizes, schedules and decoding rules (whole generations,
    teacher forced)."""
    c = _random_case(seed)
    d = max(256, c["hq"] * c["hd"])
    cfg = small_cfg(c["dtype"], c["hq"], c["hkv"], c["hd"], d=d, scale=c["scale"])
    w = ec_inputs.make_weights(cfg, seed, gain_jitter=0.1)
    tau = c["tau"] if c["metric"] != 2 else min(c["tau"], 0.5)
    dec = ec_inputs.DecodeCfg(gen_len=c["N"], block=c["block"], k_recent=c["k"],
                              tokens_per_step=c["n"], tau=tau, conf_threshold=c["thr"],
                              gate_metric=c["metric"], schedule=c["schedule"])
    prompt = ec_inputs.make_prompt(cfg.vocab, c["P"], seed + 1)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL[c["dtype"]], max_steps=40)
    print(c, s)
    assert s["tokens_exact"] > 0


def test_largest_batch():
    """EC_MAX_BATCH sequences with ragged prompts, every one against its own oracle run."""
    cfg = small_cfg("bf16", 4, 2, 64, scale=13.0)
    w = ec_inputs.make_weights(cfg, 41, gain_jitter=0.1)
    B = ec.EC_MAX_BATCH
    dec = ec_inputs.DecodeCfg(gen_len=12, block=8, k_recent=2, tokens_per_step=2, tau=2.5, batch=B)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 1 + (7 * b) % 23, 300 + b) for b in range(B)]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL["bf16"], check_cache_every=3)
    print(s)
    assert s["steps"] == 6 and s["modes"][eco.FULL] >= B
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0 and s["modes_exact"] > 0


def test_many_few_row_sequences_one_attention_block_per_sequence_and_head():
    """32 ragged sequences x 8 heads whose partial steps recompute up to 36 rows each: the row
    list packs them back to back (a 16-row tile holds rows of two or three sequences), and the
    batch is large enough that the attention serves all row tiles of a (sequence, head) from one
    block that reads the sequence's K/V once.  Every sequence against its own oracle run."""
    cfg = small_cfg("bf16", 8, 4, 64, scale=13.0)
    w = ec_inputs.make_weights(cfg, 59, gain_jitter=0.1)
    B = 32
    dec = ec_inputs.DecodeCfg(gen_len=40, block=32, k_recent=4, tokens_per_step=2, tau=1e9, batch=B)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 5 + (11 * b) % 57, 500 + b) for b in range(B)]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL["bf16"], max_steps=7, check_cache_every=3)
    print(s)
    assert s["modes"][eco.PARTIAL] == 6 * B and s["tokens_exact"] > 0


def test_batched_generate_runs_every_sequence_to_the_end():
    """ec_generate on a batch: free-running, sequences in different modes side by side; every
    generation slot ends up decoded, the counters add up, and a reset reproduces the run."""
    cfg = small_cfg("bf16", 4, 2, 64, scale=13.0)
    w = ec_inputs.make_weights(cfg, 31, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=48, block=16, k_recent=2, tokens_per_step=2, tau=2.5, batch=3)
    prompts = [ec_inputs.make_prompt(cfg.vocab, P, 50 + i) for i, P in enumerate((30, 5, 64))]
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompts)
    try:
        toks, stats = g.generate()
        assert toks.shape == (3, 48) and stats["tokens"] == 3 * 48 and stats["steps"] == 24
        assert stats["full_steps"] + stats["partial_steps"] == 3 * 24 and stats["full_steps"] >= 3
        for b in range(3):
            assert not g.debug_read(ec.EC_DBG_MASKED, seq=b).any()
            assert np.array_equal(g.debug_read(ec.EC_DBG_X, seq=b)[len(prompts[b]):], toks[b])
        g.reset(prompts)
        toks2, stats2 = g.generate()
        assert np.array_equal(toks, toks2) and stats2["full_steps"] == stats["full_steps"]
    finally:
        g.close()


def test_recompute_ratio_counter():
    """RR = rows recomputed / (steps x T), the fraction of KV states recomputed per step: 1 when
    the threshold lies below every entropy (all steps FULL); with a threshold nothing exceeds it
    is one FULL step plus |M u R| <= block + k rows per step, and equals the oracle's count."""
    cfg = small_cfg("f32", 4, 2, 64)
    w = ec_inputs.make_weights(cfg, 67, gain_jitter=0.1)
    prompt = ec_inputs.make_prompt(cfg.vocab, 40, 13)
    dw = ec.weights_to_device(cfg, w)
    T, N, block, k = 40 + 32, 32, 8, 2
    for tau in (-1.0, 1e9):
        dec = ec_inputs.DecodeCfg(gen_len=N, block=block, k_recent=k, tokens_per_step=1, tau=tau)
        g = ec.EntropyCache(cfg, dw, dec, prompt)
        try:
            _, stats = g.generate()
        finally:
            g.close()
        assert stats["steps"] == N
        rr = stats["rows_recomputed"] / (stats["steps"] * T)
        if tau < 0:
            assert stats["full_steps"] == N and rr == 1.0
        else:
            assert stats["full_steps"] == 1 and stats["partial_steps"] == N - 1
            rows_oracle = sum(len(r["S"]) for r in eco.eco_generate(
                eco.eco_init(eco.OracleModel(cfg, w), dec, prompt)))
            assert stats["rows_recomputed"] == rows_oracle
            assert T < stats["rows_recomputed"] <= T + (N - 1) * (block + k)
            assert rr < 0.25


@pytest.mark.parametrize("dtype,P,N,block,k,n,tau", [
    ("f32", 0, 20, 8, 2, 1, 2.5),          # no prompt at all
    ("bf16", 3, 40, 128, 100, 32, 1e9),    # largest block and tokens per step, k beyond the generation
    ("f32", 9, 12, 4, 1, 1, -1.0),         # threshold below any entropy: every step FULL
    ("bf16", 17, 33, 1, 0, 1, 1e9),        # block of one: strictly left to right, no recent rows
])
def test_degenerate_shapes(dtype, P, N, block, k, n, tau):
    cfg = small_cfg(dtype, 4, 2, 64)
    w = ec_inputs.make_weights(cfg, 23, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=N, block=block, k_recent=k, tokens_per_step=n, tau=tau)
    prompt = ec_inputs.make_prompt(cfg.vocab, P, 4)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL[dtype])
    print(s)
    assert s["tokens_exact"] > 0 and s["rows_decided"] > 0
    if tau < 0:
        assert s["modes"][eco.PARTIAL] == 0


def test_largest_context_properties():
    """15000 positions (the largest context the library accepts) on a small model, where the
    oracle is too slow: properties that hold at any size.  A second FULL step with nothing
    committed in between is idempotent (same logits, same cache); a PARTIAL step after it sees an
    exact cache and reproduces those logits on the block rows."""
    cfg = small_cfg("bf16", 4, 2, 64)
    w = ec_inputs.make_weights(cfg, 29, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=200, block=32, k_recent=2, tokens_per_step=1, tau=1.0)
    prompt = ec_inputs.make_prompt(cfg.vocab, 14800, 6)
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompt)
    g.keep_logits(True)
    try:
        r1 = g.step_forced(ec.EC_FULL, [], [])
        z1 = g.debug_read(ec.EC_DBG_LOGITS, count=32)
        k1 = g.debug_read(ec.EC_DBG_KCACHE, 1)
        r2 = g.step_forced(ec.EC_FULL, [], [])
        z2 = g.debug_read(ec.EC_DBG_LOGITS, count=32)
        k2 = g.debug_read(ec.EC_DBG_KCACHE, 1)
        assert r1["n_query_rows"] == r2["n_query_rows"] == 15000
        assert np.array_equal(z1, z2) and np.array_equal(k1, k2)      # same kernels, same inputs
        assert np.isfinite(z1).all() and float(np.abs(z1).max()) > 0
        r3 = g.step_forced(ec.EC_PARTIAL, [], [])
        z3 = g.debug_read(ec.EC_DBG_LOGITS, count=32)
        assert r3["n_query_rows"] == 32
        assert relerr(z3, z1) <= TOL["bf16"]
        # the partial step rewrote the block rows' K/V from the same inputs
        assert relerr(ec_bits(g.debug_read(ec.EC_DBG_KCACHE, 1)), ec_bits(k1)) <= TOL["bf16"]
    finally:
        g.close()


def ec_bits(a):
    return (a.astype(np.uint32) << np.uint32(16)).view(np.float32) if a.dtype == np.uint16 else a


def test_free_running_generation_matches_oracle_f32():
    """Without forcing: the GPU's own decisions reproduce the oracle's generation (float32 model,
    margins far above 1e-4 at every step of this seed)."""
    wl = ec_inputs.WORKLOADS["tiny_f32"]
    cfg = wl.model.replace(logit_scale=16.0)
    w = ec_inputs.make_weights(cfg, wl.seed)
    prompt = ec_inputs.make_prompt(cfg.vocab, wl.prompt_len, wl.seed)
    st = eco.eco_init(eco.OracleModel(cfg, w), wl.decode, prompt)
    trace = eco.eco_generate(st)
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), wl.decode, prompt)
    toks, stats = g.generate()
    assert stats["steps"] == len(trace) and stats["full_steps"] == st.n_full
    assert stats["rows_recomputed"] == st.rows_recomputed
    assert np.array_equal(toks, st.x[st.P:].astype(np.int32))
    # reset and step by step: same sequence of modes, positions, tokens, entropies
    g.reset(prompt)
    for r in trace:
        q = g.step(ec.EC_AUTO)
        assert q["mode_run"] == r["mode"] and q["positions"] == r["positions"]
        assert q["tokens"] == r["tokens"]
        assert abs(q["max_entropy"] - r["E"]) < 1e-3
    g.close()


def test_state_errors_and_forced_mode_schedule():
    cfg = small_cfg("f32")
    w = ec_inputs.make_weights(cfg, 5)
    dec = ec_inputs.DecodeCfg(gen_len=8, block=4, k_recent=2, tokens_per_step=1, tau=1e9)
    prompt = ec_inputs.make_prompt(cfg.vocab, 6, 1)
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompt)
    with pytest.raises(ec.EcError) as e:
        g.step(ec.EC_PARTIAL)
    assert e.value.code == ec.EC_ERR_STATE
    with pytest.raises(ec.EcError) as e:
        g.step_forced(ec.EC_FULL, [2], [1])            # a prompt position is not a masked slot
    assert e.value.code == ec.EC_ERR_ARG
    # forced all-FULL schedule vs oracle forced the same way
    st = eco.eco_init(eco.OracleModel(cfg, w), dec, prompt)
    for i in range(8):
        r = eco.eco_step(st, eco.FULL)
        q = g.step_forced(ec.EC_FULL, r["positions"], r["tokens"])
        assert q["n_query_rows"] == st.T
        assert relerr(g.debug_read(ec.EC_DBG_LOGITS, count=len(r["Mb"])), r["logits"]) < 1e-4
    assert q["done"]
    with pytest.raises(ec.EcError) as e:
        g.step(ec.EC_AUTO)
    assert e.value.code == ec.EC_ERR_STATE
    g.close()


def test_entropy_closed_forms_through_the_whole_path():
    """Zero LM head -> uniform logits: H = ln V, confidence 1/V, token 0 (lowest id on ties),
    most confident row = lowest position.  One dominant LM-head row -> H ~ 0, confidence ~ 1."""
    cfg = small_cfg("f32", scale=1.0)
    w = ec_inputs.make_weights(cfg, 9)
    dec = ec_inputs.DecodeCfg(gen_len=8, block=8, k_recent=2, tokens_per_step=2, tau=1.0)
    prompt = ec_inputs.make_prompt(cfg.vocab, 10, 2)
    w0 = dict(w); w0["lm_head"] = np.zeros_like(w["lm_head"])
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w0), dec, prompt)
    q = g.step(ec.EC_AUTO)
    assert q["positions"] == [10, 11] and q["tokens"] == [0, 0]
    assert q["max_entropy"] == pytest.approx(math.log(cfg.vocab), rel=1e-6)
    assert q["confidence"][0] == pytest.approx(1.0 / cfg.vocab, rel=1e-6)
    assert q["next_mode"] == ec.EC_FULL
    g.close()
    # dominant row: lm_head[77] = 1000 * (direction every final hidden state has a positive
    # component along): use the final norm's output sign trick by making all other rows zero and
    # row 77 and 78 equal -> exactly two equal maxima -> H = ln 2 when they dominate
    w1 = dict(w)
    lm = np.zeros_like(w["lm_head"])
    w1["lm_head"] = lm
    st = eco.eco_init(eco.OracleModel(cfg, w), dec, prompt)
    hfin = eco.forward_rows(st, np.arange(st.T), eco.current_block_masked(st))
    lm[77] = lm[78] = (200.0 * hfin[0] / np.linalg.norm(hfin[0]) ** 2).astype(np.float32)
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w1), dec, prompt)
    q = g.step(ec.EC_AUTO)
    stats = g.debug_read(ec.EC_DBG_ROW_STATS, count=8)
    assert int(stats[0, 0]) == 77                      # lowest id among the equal maxima
    assert stats[0, 2] == pytest.approx(math.log(2.0), rel=1e-4)
    assert stats[0, 1] == pytest.approx(0.5, rel=1e-4)
    g.close()


def test_large_magnitude_residual_stream():
    """Residual rows with sums of squares near 1e10 (embeddings of magnitude ~6000, as the
    massive activations of trained models): the fixed-point row sums behind the folded RMSNorm
    must neither wrap nor lose the row."""
    from tests.gpu_harness import bf16_bits_to_f32
    cfg = small_cfg("bf16", 4, 2, 64)
    w = ec_inputs.make_weights(cfg, 43, gain_jitter=0.1)
    w["tok_emb"] = ec_inputs.f32_to_bf16_bits(bf16_bits_to_f32(w["tok_emb"]) * np.float32(3e5))
    dec = ec_inputs.DecodeCfg(gen_len=40, block=32, k_recent=2, tokens_per_step=2, tau=1e9)
    prompt = ec_inputs.make_prompt(cfg.vocab, 150, 8)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL["bf16"])
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["rows_decided"] > 0 and s["modes_exact"] > 0


def test_long_context_ragged_batch_gqa():
    """Two sequences of more than 2048 positions with grouped-query heads of 128: the key slices
    of the partial-step attention (pieces summed by the last block to arrive) on a ragged batch."""
    cfg = small_cfg("bf16", 4, 2, 128, d=512)
    w = ec_inputs.make_weights(cfg, 47, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=24, block=16, k_recent=3, tokens_per_step=2, tau=1e9, batch=2)
    prompts = [ec_inputs.make_prompt(cfg.vocab, P, 60 + i) for i, P in enumerate((2100, 2333))]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL["bf16"], max_steps=6, check_cache_every=3)
    print(s)
    assert s["modes"][eco.PARTIAL] >= 8 and s["tokens_exact"] > 0


def test_logits_stay_out_of_memory_unless_asked_for():
    """The bfloat16 path reduces the vocabulary inside the LM-head kernel: by default a step
    leaves no logits behind (reading them is a state error), and switching the store on changes
    nothing else - same tokens, same statistics, bit for bit."""
    cfg = small_cfg("bf16", 4, 2, 64, scale=13.0)
    w = ec_inputs.make_weights(cfg, 53, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=48, block=16, k_recent=2, tokens_per_step=2, tau=2.5)
    prompt = ec_inputs.make_prompt(cfg.vocab, 30, 12)
    dw = ec.weights_to_device(cfg, w)
    runs = []
    for keep in (False, True):
        g = ec.EntropyCache(cfg, dw, dec, prompt)
        g.keep_logits(keep)
        trace = []
        while True:
            q = g.step(ec.EC_AUTO)
            stats = g.debug_read(ec.EC_DBG_ROW_STATS, count=q["n_block_rows"])
            trace.append((q, stats.copy()))
            if keep:
                z = g.debug_read(ec.EC_DBG_LOGITS, count=q["n_block_rows"])
                assert np.array_equal(z.max(axis=1), stats[:, 3])
            else:
                with pytest.raises(ec.EcError) as e:
                    g.debug_read(ec.EC_DBG_LOGITS, count=1)
                assert e.value.code == ec.EC_ERR_STATE
            if q["done"]:
                break
        runs.append(trace)
        g.close()
    assert len(runs[0]) == len(runs[1])
    for (qa, sa), (qb, sb) in zip(*runs):
        assert qa == qb and np.array_equal(sa, sb)


@pytest.mark.parametrize("hq,hkv,hd,P,N,block,k,n,tau,f", [
    (4, 4, 64, 64, 64, 32, 2, 1, 3.0, 768),
    (4, 2, 128, 50, 70, 32, 4, 2, 2.5, 1280),    # GQA, head_dim 128, ragged last block
    (8, 2, 64, 100, 33, 32, 2, 3, 1e9, 768),     # 133 rows in FULL steps: tiled kernels + scales
    (4, 2, 64, 40, 128, 32, 64, 1, 1e9, 6208),   # up to 96 rows; 776 gate/up tiles in groups of 3
])
def test_e4m3_weight_models_whole_generation(hq, hkv, hd, P, N, block, k, n, tau, f):
    """Matrices stored as e4m3 codes with per-row scales (EC_FP8W): partial steps stream the
    codes and widen them in registers, full steps run on their exact bf16 expansion; both apply
    the row scales to the sums.  The oracle decodes the same codes exactly."""
    cfg = small_cfg("fp8w", hq, hkv, hd, d=hq * hd if hq * hd >= 256 else 256, f=f)
    w = ec_inputs.make_weights(cfg, 7, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=N, block=block, k_recent=k, tokens_per_step=n, tau=tau)
    prompt = ec_inputs.make_prompt(cfg.vocab, P, 3)
    s = run_teacher_forced(cfg, w, dec, prompt, TOL["fp8w"])
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["tokens_exact"] > 0 and s["modes_exact"] > 0


def test_e4m3_weight_batch():
    cfg = small_cfg("fp8w", 4, 2, 128, d=512)
    w = ec_inputs.make_weights(cfg, 13, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=36, block=32, k_recent=3, tokens_per_step=1, tau=2.5, batch=4)
    prompts = [ec_inputs.make_prompt(cfg.vocab, P, 20 + i) for i, P in enumerate((70, 9, 33, 150))]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL["fp8w"], max_steps=12)
    print(s)
    assert s["modes"][eco.PARTIAL] >= 1 and s["tokens_exact"] > 0


@pytest.mark.parametrize("dtype,batch", [("bf16", 1), ("f32", 1), ("bf16", 3)])
def test_rows_of_nan_logits_are_reported_and_nothing_leaves_its_buffers(dtype, batch):
    """A model whose final norm gain is NaN: every logit is NaN, so no row has a maximum.  The
    step must say so (EC_ERR_NONFINITE), the rows take token 0 (a row's token indexes the
    embedding table at the next step), further steps and a generation run to their end the same
    way, and a healthy context next to it is unaffected."""
    cfg = small_cfg(dtype, 4, 2, 64)
    good = ec_inputs.make_weights(cfg, 61, gain_jitter=0.1)
    bad = dict(good)
    bad["final_norm"] = good["final_norm"].copy()
    if dtype == "f32":
        bad["final_norm"][:] = np.nan
    else:
        bad["final_norm"][:] = 0x7FC0          # a bfloat16 NaN
    dec = ec_inputs.DecodeCfg(gen_len=24, block=8, k_recent=2, tokens_per_step=2, tau=2.5, batch=batch)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 9 + 5 * b, 70 + b) for b in range(batch)]
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, bad), dec, prompts if batch > 1 else prompts[0])
    for mode in (ec.EC_AUTO, ec.EC_AUTO, ec.EC_PARTIAL, ec.EC_FULL):
        with pytest.raises(ec.EcError) as e:
            g.step(mode)
        assert e.value.code == ec.EC_ERR_NONFINITE
        x = g.debug_read(ec.EC_DBG_X)
        assert x.min() >= 0 and x.max() < cfg.vocab
    stats = g.debug_read(ec.EC_DBG_ROW_STATS, count=1)
    assert stats[0, 0] == 0 and stats[0, 1] == 0 and np.isinf(stats[0, 2])
    with pytest.raises(ec.EcError) as e:
        g.generate()
    assert e.value.code == ec.EC_ERR_NONFINITE
    g.close()
    # the same shapes with finite weights still match the oracle
    s = (run_teacher_forced(cfg, good, dec, prompts[0], TOL[dtype], max_steps=4) if batch == 1 else
         run_teacher_forced_batch(cfg, good, dec, prompts, TOL[dtype], max_steps=4))
    assert s["steps"] == 4


@pytest.mark.parametrize("dtype,batch,block", [
    ("bf16", 1, 24), ("f32", 1, 24), ("bf16", 2, 48),   # reduced in the LM head; over 64 rows, from stored logits
])
def test_rows_with_an_infinite_maximum_take_token_0(dtype, batch, block):
    """Two vocabulary rows with an infinite weight each, of either sign for the same feature: one of their logits is +inf.  Such
    rows have no finite maximum: they take token 0, confidence 0 and infinite entropy, and the step reports them."""
    cfg = small_cfg(dtype, 4, 2, 64)
    w = ec_inputs.make_weights(cfg, 61, gain_jitter=0.1)
    w["lm_head"] = w["lm_head"].copy()
    w["lm_head"][[1234, 2345], 7] = (np.inf, -np.inf) if dtype == "f32" else (0x7F80, 0xFF80)
    dec = ec_inputs.DecodeCfg(gen_len=block, block=block, k_recent=2, tokens_per_step=2, tau=2.5, batch=batch)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 9 + 5 * b, 70 + b) for b in range(batch)]
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompts if batch > 1 else prompts[0])
    with pytest.raises(ec.EcError) as e:
        g.step(ec.EC_FULL)
    assert e.value.code == ec.EC_ERR_NONFINITE
    s = np.concatenate([g.debug_read(ec.EC_DBG_ROW_STATS, seq=b) for b in range(batch)])
    g.close()
    assert (s[:, 3] == np.inf).all()
    assert not s[:, :2].any() and np.isinf(s[:, 2]).all()


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("dtype,batch,block", [
    ("bf16", 1, 24), ("f32", 1, 24), ("bf16", 2, 48),   # reduced in the LM head; over 64 rows, from stored logits
])
def test_logits_far_apart_are_a_distribution(dtype, batch, block, sign):
    """Half of the vocabulary at logits around 1e36, either sign, with the other half near 0: finite logits, of which the lower half counts
    nothing.  The decision's statistics are those of the step's own logits in 64 bits, but for the float32 sums, a fast exponential of
    4e-6 at most (arguments down to -87) and their rounding: under 1e-5."""
    cfg = small_cfg(dtype, 4, 2, 64, vocab=8192)
    w = ec_inputs.make_weights(cfg, 61, gain_jitter=0.1)
    w["lm_head"] = w["lm_head"].copy()
    w["lm_head"][2048:6144, 7] = sign * 1e36 if dtype == "f32" else (0x7B41 if sign > 0 else 0xFB41)   # 1.002e36
    dec = ec_inputs.DecodeCfg(gen_len=block, block=block, k_recent=2, tokens_per_step=2, tau=2.5, batch=batch)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 9 + 5 * b, 70 + b) for b in range(batch)]
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompts if batch > 1 else prompts[0])
    g.keep_logits(True)
    g.step(ec.EC_FULL)
    for b in range(batch):
        z = g.debug_read(ec.EC_DBG_LOGITS, seq=b, count=block).astype(np.float64)
        assert np.isfinite(z).all() and np.ptp(z, axis=1).min() > 1e34
        s = g.debug_read(ec.EC_DBG_ROW_STATS, seq=b, count=block)
        ref = np.array([eco.softmax_stats(r) for r in z])
        assert np.array_equal(s[:, 0], ref[:, 0])
        assert np.allclose(s[:, 1], ref[:, 1], rtol=1e-5) and np.allclose(s[:, 2], ref[:, 2], rtol=1e-5, atol=1e-5)
    g.close()


@pytest.mark.parametrize("batch,gen_len,n", [(1, 1024, 32), (16, 512, 32), (64, 96, 7)])
def test_every_result_is_whole_when_its_step_returns(batch, gen_len, n):
    """A step returns as soon as the host sees its serial number in pinned memory.  The lists that it hands over then are the step's
    own: the tokens that the device holds at their positions in the end, each position once, in order of confidence."""
    cfg = small_cfg("bf16", 4, 2, 64, d=64, f=64, vocab=512, layers=1, scale=24.0)
    w = ec_inputs.make_weights(cfg, 157, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(batch=batch, gen_len=gen_len, block=64, k_recent=0, tokens_per_step=n, tau=1e9)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 3 + b % 5, 80 + b) for b in range(batch)]
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompts if batch > 1 else prompts[0])
    x = [{} for _ in range(batch)]
    done = [False] * batch
    while not all(done):
        r = g.step(ec.EC_AUTO)
        for b, q in enumerate(r if batch > 1 else [r]):
            if done[b]:
                continue
            assert 0 < q["n_unmasked"] == len(q["positions"]) <= n
            assert not set(q["positions"]) & set(x[b])
            assert q["confidence"] == sorted(q["confidence"], reverse=True) and min(q["confidence"]) > 0
            x[b].update(zip(q["positions"], q["tokens"]))
            done[b] = q["done"]
    for b in range(batch):
        P = len(prompts[b])
        got = g.debug_read(ec.EC_DBG_X, seq=b)
        assert [x[b][p] for p in range(P, P + gen_len)] == got[P:].tolist()
    g.close()


@pytest.mark.parametrize("hq,hkv,hd,d,f,vocab,P,shift", [
    (2, 1, 64, 136, 200, 1003, 19, 0),     # K = 136 and 200: half-filled last k-chunks, odd tile counts
    (3, 3, 128, 264, 1032, 4099, 40, 0),   # K just above 256: eight waves to a block
    (8, 2, 64, 512, 1032, 515, 300, 0),    # many tiles: four to a block, both k-lengths
    (2, 2, 64, 72, 8, 2, 1, 0),            # one tile, the smallest vocabulary
    (4, 2, 64, 256, 520, 777, 30, 1),      # weights that start at any element
    (8, 2, 64, 264, 1032, 4115, 300, 3),   # ... and many tiles of them
])
def test_f32_gemm_edges(hq, hkv, hd, d, f, vocab, P, shift):
    """The float32 kernels at the edges of their tiles, k-chunks and dispatch rules."""
    cfg = small_cfg("f32", hq, hkv, hd, d=d, f=f, vocab=vocab, scale=8.0)
    w = ec_inputs.make_weights(cfg, 61, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=21, block=8, k_recent=3, tokens_per_step=2, tau=1e9)
    prompt = ec_inputs.make_prompt(max(vocab, 98), P, 4) % vocab
    st = eco.eco_init(eco.OracleModel(cfg, w), dec, prompt)
    dw = ec.weights_to_device(cfg, w)
    if shift:
        import torch

        def moved(t):
            buf = torch.empty(t.numel() + shift, dtype=t.dtype, device=t.device)
            return buf[shift:].view(t.shape).copy_(t)
        dw = {k: [moved(t) for t in v] if isinstance(v, list) else moved(v) for k, v in dw.items()}
    g = ec.EntropyCache(cfg, dw, dec, prompt)
    g.keep_logits(True)
    for i in range(4):
        r = eco.eco_step(st, eco.FULL if i in (0, 2) else eco.PARTIAL)
        g.step_forced(r["mode"], r["positions"], r["tokens"])
        z = g.debug_read(ec.EC_DBG_LOGITS, count=len(r["Mb"]))
        assert relerr(z, r["logits"]) < 1e-5, (i, relerr(z, r["logits"]))
        for l in range(cfg.n_layers):
            assert relerr(g.debug_read(ec.EC_DBG_KCACHE, l), st.Kc[l]) < 1e-5
            assert relerr(g.debug_read(ec.EC_DBG_VCACHE, l), st.Vc[l]) < 1e-5
    g.close()


@pytest.mark.parametrize("hq,hkv,hd,d,f,P,gate_up", [
    (4, 2, 64, 288, 12320, 760, None),    # 9 k-steps, an odd number; 1540 weight tiles
    (4, 4, 64, 32, 4128, 900, None),      # a single k-step; 129 k-steps for 2 weight tiles
    (8, 8, 128, 1056, 6176, 1400, None),  # 33 and 193 k-steps, uneven K ranges, ragged row and column tiles
    (4, 4, 64, 96, 9152, 520, (192, 320, 1)),   # the last row and column block ragged
    (4, 4, 64, 96, 8192, 760, (256, 256, 1)),   # the last of four row blocks 3 rows
])
def test_tiled_gemm_k_steps_and_ragged_tiles(hq, hkv, hd, d, f, P, gate_up):
    """The many-row GEMMs at odd and tiny numbers of k-steps, with tiles that the matrices do not
    fill."""
    cfg = small_cfg("bf16", hq, hkv, hd, d=d, f=f, vocab=512, scale=4.0)
    w = ec_inputs.make_weights(cfg, 67, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=11, block=4, k_recent=2, tokens_per_step=1, tau=1e9)
    if gate_up:
        assert block_shape(cfg, ec.EC_K_GATEUP, P + 11) == gate_up
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, P, 6), TOL["bf16"], max_steps=2)
    print(s)
    assert s["rows_stat"] > 0    # (d = 32 gives logits too flat for exact tokens)


@pytest.mark.parametrize("hq,hkv,hd,plens,tiles", [
    # eight tiles to a block: sequences of 7 to 17 row tiles, one of whole groups; one of few rows among them; ten of 24 to 37 tiles
    (4, 2, 64, [72, 88, 216, 217, 90], 8),
    (4, 4, 128, [231, 56, 200], 8),
    (16, 16, 64, [530, 537, 520, 471, 536, 529, 344, 535, 530, 533], 8),
    # twelve, from enough blocks on: groups that end in the next sequence or in padding, and whole ones
    (16, 16, 64, [530, 537, 520, 471, 536, 529, 504, 535, 530, 533], 12),
    (16, 4, 128, [530, 472, 537, 520, 535, 529, 536, 504, 530, 533], 12),
    # one sequence alone, without a table of groups: 81 and 67 tiles, the last blocks part empty
    (48, 16, 128, [1250], 12),
    (64, 64, 64, [1021], 12),
])
def test_many_row_attention_of_ragged_batches(hq, hkv, hd, plens, tiles):
    """Attention of full steps, whose blocks take eight or twelve row tiles of one sequence: the tiles of a sequence's last block
    that belong to the next one or hold padding rows only."""
    cfg = small_cfg("bf16", hq, hkv, hd, d=64, f=64, vocab=512, layers=2, scale=8.0)
    w = ec_inputs.make_weights(cfg, 139, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(batch=len(plens), gen_len=40, block=20, k_recent=2, tokens_per_step=1, tau=1e9)
    assert full_step_attn_tiles(cfg, [P + 40 for P in plens]) == tiles
    prompts = [ec_inputs.make_prompt(cfg.vocab, P, 20 + i) for i, P in enumerate(plens)]
    s = (run_teacher_forced(cfg, w, dec, prompts[0], TOL["bf16"], max_steps=2) if len(plens) == 1 else
         run_teacher_forced_batch(cfg, w, dec, prompts, TOL["bf16"], max_steps=2))
    print(s)
    assert s["modes"][eco.FULL] == len(plens) and s["rows_stat"] > 0


@pytest.mark.parametrize("dtype,tiles,block", [
    ("bf16", 33, 9), ("bf16", 1023, 20), ("fp8w", 1023, 40), ("bf16", 1023, 64),    # two weight tiles to a block
    ("bf16", 1025, 9), ("fp8w", 1026, 20), ("bf16", 2047, 40), ("bf16", 1027, 64),  # four
    ("bf16", 2049, 9), ("fp8w", 2051, 20), ("bf16", 2055, 40),                      # eight
])
def test_lm_head_tiles_to_a_block(dtype, tiles, block):
    """The few-row LM head at each number of weight tiles to a block, the last block part empty, with one to four row
    tiles: logits and the vocabulary reduction merged from the blocks' tiles."""
    cfg = small_cfg(dtype, 4, 2, 64, d=64, f=64, vocab=16 * tiles, layers=1, scale=24.0)
    w = ec_inputs.make_weights(cfg, 137, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=block + 3, block=block, k_recent=2, tokens_per_step=2, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, 12, 6), TOL[dtype], max_steps=3)
    print(s)
    assert s["rows_stat"] > 0


@pytest.mark.parametrize("d", [32, 64, 96, 128, 160, 192])
def test_tiled_gemm_ranges_around_the_operand_ring(d):
    """One to six k-steps through the 8-wave kernels, whose ring holds four and is filled three ahead."""
    cfg = small_cfg("bf16", 4, 4, 64, d=d, f=4128, vocab=512, layers=1, scale=4.0)
    assert block_shape(cfg, ec.EC_K_GATEUP, 911) == (192, 256, 1)
    w = ec_inputs.make_weights(cfg, 131, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=11, block=4, k_recent=2, tokens_per_step=1, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, 900, 6), TOL["bf16"], max_steps=2)
    print(s)
    assert s["rows_stat"] > 0


@pytest.mark.parametrize("dtype,hq,hkv,hd,d,f,P,blocks", [
    # q/k/v with rotation and cache stores, the last row and column block ragged
    ("bf16", 32, 32, 128, 96, 256, 760, {"QKV": (192, 320, 1)}),
    ("bf16", 32, 32, 128, 96, 256, 1089, {"QKV": (256, 256, 1)}),
    ("fp8w", 32, 32, 128, 128, 256, 760, {"QKV": (192, 320, 1)}),
    ("fp8w", 32, 32, 128, 128, 256, 1089, {"QKV": (256, 256, 1)}),
    # gate/up with row scales
    ("fp8w", 4, 4, 64, 128, 6016, 760, {"GATEUP": (192, 320, 1)}),
    ("fp8w", 4, 4, 64, 128, 8128, 760, {"GATEUP": (256, 256, 1)}),
    # residual products, K whole and split over blocks that meet
    ("bf16", 4, 4, 64, 4640, 64, 2538, {"OPROJ": (192, 320, 1), "DOWN": (192, 320, 1)}),
    ("fp8w", 4, 4, 64, 4672, 64, 2538, {"OPROJ": (192, 320, 1), "DOWN": (192, 320, 1)}),
    ("bf16", 4, 4, 64, 6176, 64, 2538, {"OPROJ": (256, 256, 1), "DOWN": (256, 256, 1)}),
    ("fp8w", 4, 4, 64, 6208, 64, 2538, {"OPROJ": (256, 256, 1), "DOWN": (256, 256, 1)}),
    ("bf16", 4, 4, 64, 4128, 4096, 520, {"DOWN": (192, 320, 4)}),
    ("fp8w", 4, 4, 64, 4160, 4096, 520, {"DOWN": (192, 320, 4)}),
    ("bf16", 4, 4, 64, 4128, 6176, 1089, {"DOWN": (256, 256, 3)}),
    ("fp8w", 4, 4, 64, 4160, 6208, 1089, {"DOWN": (256, 256, 3)}),
])
def test_widest_tiled_blocks(dtype, hq, hkv, hd, d, f, P, blocks):
    """Blocks of 192 x 320 and 256 x 256 under every epilogue, with and without row scales, at sizes that
    leave the last blocks ragged.  The sizes are those at which the kernels pick these blocks."""
    cfg = small_cfg(dtype, hq, hkv, hd, d=d, f=f, vocab=512, layers=1, scale=4.0)
    for product, shape in blocks.items():
        assert block_shape(cfg, getattr(ec, "EC_K_" + product), P + 11) == shape, product
    w = ec_inputs.make_weights(cfg, 83, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=11, block=4, k_recent=2, tokens_per_step=1, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, P, 6), TOL[dtype], max_steps=2)
    print(s)
    assert s["rows_stat"] > 0


@pytest.mark.parametrize("dtype,vocab,shape", [("bf16", 32752, (256, 256, 1)), ("fp8w", 32752, (256, 256, 1)),
                                               ("bf16", 26224, (192, 320, 1)), ("fp8w", 26224, (192, 320, 1))])
def test_widest_tiled_blocks_lm_head(dtype, vocab, shape):
    """The same for the LM head of four sequences with 128 masked positions each."""
    cfg = small_cfg(dtype, 4, 2, 64, d=128, f=256, vocab=vocab, layers=1, scale=8.0)
    dec = ec_inputs.DecodeCfg(batch=4, gen_len=128, block=128, k_recent=2, tokens_per_step=1, tau=1e9)
    assert ec.block_shape(cfg, ec.EC_K_LMHEAD, 512, 512) == shape
    w = ec_inputs.make_weights(cfg, 89, gain_jitter=0.1)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 5 + b, 6 + b) for b in range(4)]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL[dtype], max_steps=1)
    print(s)
    assert s["rows_stat"] > 0


@pytest.mark.parametrize("dtype,hq,d,f,block,k", [
    ("bf16", 4, 288, 11520, 24, 2),   # 2 row tiles x 11520: the shortest split down projection there
    ("bf16", 4, 288, 7680, 40, 8),    # 3 row tiles; 18 weight tiles in groups of four
    ("bf16", 8, 512, 4608, 70, 20),   # 6 row tiles
    ("fp8w", 4, 320, 7744, 40, 8),    # e4m3 codes, 121 k-steps over four ranges of four waves
    ("fp8w", 4, 256, 4672, 70, 25),
])
def test_partial_step_with_split_down_projection(dtype, hq, d, f, block, k):
    """Few-row steps whose down projection is split along K over blocks."""
    cfg = small_cfg(dtype, hq, 2, 64, d=d, f=f, vocab=512, scale=8.0)
    w = ec_inputs.make_weights(cfg, 71, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=2 * block, block=block, k_recent=k, tokens_per_step=4, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, 30, 6), TOL[dtype], max_steps=6)
    print(s)
    assert s["modes"][eco.PARTIAL] == 5 and s["rows_stat"] > 0


@pytest.mark.parametrize("dtype,hq,hkv,hd,d,T,shape", [
    ("bf16", 32, 32, 64, 96, 523, (192, 128, 1)),     # head_dim 64: 16 chunks of factors to a row
    ("bf16", 48, 16, 64, 96, 1700, (192, 256, 1)),
    ("fp8w", 32, 32, 64, 128, 771, (192, 192, 1)),    # three tiles a wave: they straddle heads and q | k | v
    ("bf16", 16, 16, 128, 96, 771, (192, 192, 1)),
    ("bf16", 40, 8, 128, 96, 1030, (192, 256, 1)),    # grouped queries, the last row block 70 rows
    ("bf16", 32, 32, 128, 96, 1300, (192, 384, 1)),
])
def test_rotation_and_cache_stores_of_wide_blocks(dtype, hq, hkv, hd, d, T, shape):
    """The q / k / v epilogue that stages its rows' rotation factors in LDS, at every block shape and both
    head dimensions (192 x 320 and 256 x 256: above)."""
    cfg = small_cfg(dtype, hq, hkv, hd, d=d, f=256, vocab=512, layers=1, scale=4.0)
    assert block_shape(cfg, ec.EC_K_QKV, T) == shape
    w = ec_inputs.make_weights(cfg, 107, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=11, block=4, k_recent=2, tokens_per_step=1, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, T - 11, 6), TOL[dtype], max_steps=2)
    print(s)
    assert s["rows_stat"] > 0


@pytest.mark.parametrize("block", [30, 44])
def test_split_down_projection_three_steps_ahead(block):
    """Few-row down projection (split from 3 row tiles on) whose K ranges are whole pairs of sets of three
    k-steps: 9216 = 3 x 3072."""
    cfg = small_cfg("bf16", 4, 2, 64, d=288, f=9216, vocab=512, scale=8.0)
    w = ec_inputs.make_weights(cfg, 103, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=2 * block, block=block, k_recent=4, tokens_per_step=4, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, 30, 6), TOL["bf16"], max_steps=6)
    print(s)
    assert s["modes"][eco.PARTIAL] == 5 and s["rows_stat"] > 0


@pytest.mark.parametrize("dtype,d,f,P,block,down", [
    ("bf16", 4128, 4096, 520, 40, (192, 320, 4)),   # 52 tiles of 4: four of them over several XCDs
    ("bf16", 4128, 6176, 1089, 80, (256, 256, 3)),  # 85 tiles of 3
    ("fp8w", 4160, 4096, 520, 60, (192, 320, 4)),
    ("bf16", 96, 4128, 150, 70, (96, 128, 4)),      # 4 waves; one column of tiles, few k-steps to a range
    ("bf16", 1056, 1024, 2060, 20, (192, 128, 2)),  # two ranges; a row block with few rows
])
def test_blocks_that_meet_give_the_same_bits(dtype, d, f, P, block, down):
    """K split over blocks, full steps and the few-row steps behind them (which stream their weights and
    read what the full step left): the same logits whether the blocks wait for each other, give up at once (the
    last one finishes everything) or take each other to be on different XCDs.
    Their values are checked against the oracle by the tests above, which run the default."""
    cfg = small_cfg(dtype, 4, 4, 64, d=d, f=f, vocab=512, scale=4.0)
    assert block_shape(cfg, ec.EC_K_DOWN, P + 2 * block) == down
    w = ec_inputs.make_weights(cfg, 101, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=2 * block, block=block, k_recent=2, tokens_per_step=1, tau=1e9)
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, ec_inputs.make_prompt(cfg.vocab, P, 6))
    g.keep_logits(True)
    want = None
    few = [(p, a) for p in (0, 1, 2, 3, 5, 8) for a in (False, True)]   # (who gives up depends on the moment)
    for polls, apart in [(20000, False), (20000, True)] + few + [(20000, False)]:
        g.debug_meeting(polls, apart)
        got = []
        for mode in (ec.EC_FULL, ec.EC_PARTIAL, ec.EC_PARTIAL):
            g.step_forced(mode, [], [])
            got.append(g.debug_read(ec.EC_DBG_LOGITS, count=block))
        if want is None:
            want = got
            assert all(np.isfinite(z).all() and z.std() > 0 for z in want)
        assert all(np.array_equal(a, b) for a, b in zip(want, got)), (polls, apart)
    g.close()


@pytest.mark.parametrize("dtype,d,partial,mixed", [
    ("bf16", 4128, (192, 128, 4), (192, 320, 4)),
    ("bf16", 1056, (96, 128, 4), (96, 128, 4)),
    ("fp8w", 1088, (96, 128, 4), (96, 128, 4)),
])
def test_blocks_of_a_batch_that_meet(dtype, d, partial, mixed):
    """Six ragged sequences whose partial steps (30 rows each, back to back) and mixed steps (two segments
    padded to 256 rows before them) split K over blocks that meet: against the oracle, and the same bits
    however the blocks find each other."""
    B, block = 6, 30
    cfg = small_cfg(dtype, 4, 4, 64, d=d, f=4096, vocab=512, scale=4.0)
    assert ec.block_shape(cfg, ec.EC_K_DOWN, 192, 192) == partial
    assert ec.block_shape(cfg, ec.EC_K_DOWN, 640, 640) == mixed
    w = ec_inputs.make_weights(cfg, 113, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(batch=B, gen_len=2 * block, block=block, k_recent=2, tokens_per_step=1, tau=1e9)
    prompts = [ec_inputs.make_prompt(cfg.vocab, 130 + 3 * b, 6 + b) for b in range(B)]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL[dtype], max_steps=3, check_cache_every=3)
    print(s)
    assert s["modes"][eco.PARTIAL] == 2 * B and s["rows_stat"] > 0

    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompts)
    g.keep_logits(True)
    full, part, none = [ec.EC_FULL] * B, [ec.EC_PARTIAL] * B, [[]] * B
    want = None
    for polls, apart in [(20000, False), (20000, True), (0, False), (0, True), (2, False), (5, True), (20000, False)]:
        g.debug_meeting(polls, apart)
        got = []
        for modes in (full, part, full[:2] + part[2:]):
            g.step_forced_batch(modes, none, none)
            got += [g.debug_read(ec.EC_DBG_LOGITS, count=block, seq=b) for b in range(B)]
        if want is None:
            want = got
            assert all(np.isfinite(z).all() and z.std() > 0 for z in want)
        assert all(np.array_equal(a, b) for a, b in zip(want, got)), (polls, apart)
    g.close()


def test_blocks_meet_while_another_context_runs():
    """Two contexts stepping at once on two streams: their blocks take each other's compute units, so those of a
    tile need not run at the same time.  Every step's logits are those of the context alone."""
    import threading

    import torch
    cfgs = [small_cfg("bf16", 4, 4, 64, d=d, f=4096, vocab=512, scale=4.0) for d in (4128, 1056)]
    assert [block_shape(c, ec.EC_K_DOWN, 600) for c in cfgs] == [(192, 320, 4), (128, 128, 4)]
    dec = ec_inputs.DecodeCfg(gen_len=40, block=20, k_recent=2, tokens_per_step=1, tau=1e9)
    ctx, want, bad = [], [], []

    def step(g):
        g.step_forced(ec.EC_FULL, [], [])
        return g.debug_read(ec.EC_DBG_LOGITS, count=20)

    for i, cfg in enumerate(cfgs):
        dw = ec.weights_to_device(cfg, ec_inputs.make_weights(cfg, 127 + i, gain_jitter=0.1))
        torch.cuda.synchronize()
        g = ec.EntropyCache(cfg, dw, dec, ec_inputs.make_prompt(cfg.vocab, 560, 6), stream=torch.cuda.Stream())
        g.keep_logits(True)
        ctx.append(g)
        want.append(step(g))
    gate = threading.Barrier(2)

    def work(i):
        gate.wait(timeout=30)
        for _ in range(60):
            if not np.array_equal(step(ctx[i]), want[i]):
                bad.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in threads]
    [t.join(timeout=60) for t in threads]
    assert not any(t.is_alive() for t in threads) and not bad
    [g.close() for g in ctx]


@pytest.mark.parametrize("dtype,d,f,P,block,k,down", [
    ("bf16", 4128, 4096, 520, 40, 8, (192, 320, 4)),   # K split over blocks that meet; few rows: over the grid
    ("fp8w", 4160, 4096, 520, 40, 8, (192, 320, 4)),
    ("bf16", 1056, 1024, 260, 20, 2, (96, 128, 4)),    # the 4-wave kernels meet; few rows: K whole
    ("bf16", 4128, 64, 520, 20, 2, (128, 128, 1)),     # K whole, 4 waves and 8
    ("bf16", 4128, 64, 860, 20, 2, (192, 128, 1)),
])
def test_one_large_residual_channel(dtype, d, f, P, block, k, down):
    """A residual channel of 3e5, as trained models have them in a few columns: its square, 9e10, is one
    block's contribution to the row's sum of squares, which must not saturate it.  The gains of the channel are small,
    so that the other channels decide the logits."""
    cfg = small_cfg(dtype, 4, 4, 64, d=d, f=f, vocab=512, layers=2, scale=1000.0)
    assert block_shape(cfg, ec.EC_K_DOWN, P + 2 * block) == down
    w = ec_inputs.make_weights(cfg, 109, gain_jitter=0.1)
    # (tensors are bfloat16 bit patterns: 0x4892 is 299008, 0x3880 is 2^-14)
    emb = (w["tok_emb"].astype(np.uint32) << np.uint32(16)).view(np.float32) * np.float32(64)   # exact
    w["tok_emb"] = (emb.view(np.uint32) >> np.uint32(16)).astype(np.uint16)
    w["tok_emb"][:, d // 2 + 5] = 0x4892
    for gain in [w["final_norm"], *w["attn_norm"], *w["mlp_norm"]]:
        gain[d // 2 + 5] = 0x3880
    dec = ec_inputs.DecodeCfg(gen_len=2 * block, block=block, k_recent=k, tokens_per_step=4, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, P, 6), TOL[dtype], max_steps=3)
    print(s)
    assert s["modes"][eco.PARTIAL] == 2 and s["rows_stat"] > 0


@pytest.mark.parametrize("N,block,k,n,sliding", [
    (512, 128, 30, 30, 0),     # the most slots the waves count for themselves, the largest block
    (513, 100, 3, 32, 1),      # one more; sliding window
    (1100, 65, 64, 32, 0),     # more slots than threads
    (1030, 7, 0, 7, 1),        # nothing recent; two rounds of the row lists
])
def test_decision_bookkeeping_sizes(N, block, k, n, sliding):
    """Row sets, history and flags over whole generations whose slot counts cross the decision
    kernel's limits (bit-exact against the oracle, teacher forced)."""
    cfg = small_cfg("f32", 2, 1, 64, d=64, f=64, vocab=300, layers=1, scale=6.0)
    w = ec_inputs.make_weights(cfg, 73, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=N, block=block, k_recent=k, tokens_per_step=n, tau=1e9,
                              schedule=sliding)
    prompt = ec_inputs.make_prompt(cfg.vocab, 3, 6)
    st = eco.eco_init(eco.OracleModel(cfg, w), dec, prompt)
    g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, w), dec, prompt)
    while not st.done:
        r = eco.eco_step(st, eco.AUTO, keep_logits=False)
        q = g.step_forced(r["mode"], r["positions"], r["tokens"])
        assert q["done"] == st.done and q["n_block_rows"] == len(r["Mb"]) and q["n_query_rows"] == len(r["S"])
        assert q["n_recent_next"] == len(r["R"])
        if not st.done:
            rows = sorted(set(eco.current_block_masked(st).tolist()) | set(r["R"]))
            assert g.debug_read(ec.EC_DBG_ROWS, count=len(rows)).tolist() == rows
    assert np.array_equal(g.debug_read(ec.EC_DBG_X), st.x.astype(np.int32))
    assert g.debug_read(ec.EC_DBG_HIST).tolist() == [int(h) for h in st.hist]
    g.close()


@pytest.mark.parametrize("P,gain", [(230, 1.0), (230, 12.0), (2120, 6.0)])
def test_attention_scores_that_keep_growing(P, gain):
    """Keys whose scores grow along the context, slowly and fast, so that the running maximum moves now
    and then, and often (full and partial steps, key slices over blocks)."""
    cfg = small_cfg("bf16", 4, 2, 64, layers=1, scale=8.0)
    w = ec_inputs.make_weights(cfg, 79, gain_jitter=0.1)
    # sharper scores: larger queries (the attention norm's gain also scales k and v, both sides see it)
    from tests.gpu_harness import bf16_bits_to_f32
    w["wq"][0] = ec_inputs.f32_to_bf16_bits(bf16_bits_to_f32(w["wq"][0]) * np.float32(gain))
    dec = ec_inputs.DecodeCfg(gen_len=24, block=16, k_recent=2, tokens_per_step=2, tau=1e9)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, P, 7), TOL["bf16"], max_steps=4)
    print(s)
    assert s["tokens_exact"] > 0


@pytest.mark.parametrize("hq,hkv,hd,P,batch,tiles", [
    (4, 2, 64, 70, 1, 8), (4, 4, 128, 900, 1, 8), (8, 2, 128, 2600, 1, 8),   # one visit, key slices over blocks
    (16, 4, 64, 300, 16, 8),                        # a batch: one block per (sequence, head)
    (32, 8, 128, 2100, 1, 12), (64, 8, 64, 1060, 1, 12),   # full steps with three tiles a wave
])
@pytest.mark.parametrize("gain", [4.0, 30.0, 300.0])
def test_attention_weights_sum_to_one(hq, hkv, hd, P, batch, tiles, gain):
    """With one and the same embedding for every token all values are equal, and attention returns that
    value whatever the scores are: the weights' sum is one to float32 rounding (at most T + 32 roundings
    of 2^-24, far inside half a bf16 step), so the logits are those of a model with zero queries, bit
    for bit.  (A denominator of unrounded probabilities misses the value by up to 2^-9.)"""
    from tests.gpu_harness import bf16_bits_to_f32
    cfg = small_cfg("bf16", hq, hkv, hd, layers=1, scale=8.0, vocab=512)
    w = ec_inputs.make_weights(cfg, 97, gain_jitter=0.1)
    w["tok_emb"][:] = w["tok_emb"][0]
    dec = ec_inputs.DecodeCfg(batch=batch, gen_len=48, block=20, k_recent=2, tokens_per_step=1, tau=1e9)
    prompts = [ec_inputs.make_prompt(cfg.vocab, P + b, 7) for b in range(batch)]
    assert full_step_attn_tiles(cfg, [P + b + 48 for b in range(batch)]) == tiles
    got = []
    for c in (0.0, gain):
        wc = dict(w, wq=[ec_inputs.f32_to_bf16_bits(bf16_bits_to_f32(w["wq"][0]) * np.float32(c))])
        g = ec.EntropyCache(cfg, ec.weights_to_device(cfg, wc), dec, prompts if batch > 1 else prompts[0])
        g.keep_logits(True)
        z = []
        for mode in (ec.EC_FULL, ec.EC_PARTIAL):
            g.step_forced_batch([mode] * batch, [[]] * batch, [[]] * batch)
            z += [g.debug_read(ec.EC_DBG_LOGITS, seq=b) for b in range(batch)]
        g.close()
        got.append(np.stack(z))
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("plens", [[5, 9, 3], [3 + 5 * (i % 7) for i in range(64)], [97, 4, 113, 30, 6]])
def test_row_lists_of_batches(plens):
    """Row lists of under and over 128 rows, from few sequences and from the most a batch can have (a lane looks for
    each), some of which recompute everything where others do not, with a last row tile that is not full."""
    cfg = small_cfg("bf16", 4, 2, 64, d=64, f=64, vocab=512, layers=1, scale=8.0)
    w = ec_inputs.make_weights(cfg, 149, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(batch=len(plens), gen_len=12, block=6, k_recent=2, tokens_per_step=1, tau=2.5)
    prompts = [ec_inputs.make_prompt(cfg.vocab, P, 40 + i) for i, P in enumerate(plens)]
    s = run_teacher_forced_batch(cfg, w, dec, prompts, TOL["bf16"], max_steps=4)
    print(s)
    assert s["modes"][eco.FULL] >= len(plens) and s["rows_stat"] > 0


@pytest.mark.parametrize("tiles,gen_len,block,k_recent,threshold", [
    (128, 128, 40, 3, 0.0), (129, 129, 7, 2, 0.02),     # 64 and 65 parts of a row; the last wave with slots full, and one more
    (256, 512, 64, 3, 0.0), (257, 513, 33, 2, 0.0),     # 128 and 129; history counted by each wave, and by the block
    (128, 1030, 128, 4, 0.0), (1024, 64, 64, 0, 0.02),  # more slots than threads; four rounds of rows; no recency
])
def test_decisions_at_the_edges_of_rows_parts_and_slots(tiles, gen_len, block, k_recent, threshold):
    """The decision kernel where a lane's parts, a wave's slots and a round of rows begin or end: tokens, ranks, history threshold
    and row lists of a few steps."""
    cfg = small_cfg("bf16", 4, 2, 64, d=64, f=64, vocab=16 * tiles, layers=1, scale=24.0)
    w = ec_inputs.make_weights(cfg, 151, gain_jitter=0.1)
    dec = ec_inputs.DecodeCfg(gen_len=gen_len, block=block, k_recent=k_recent, tokens_per_step=3, tau=2.0,
                              conf_threshold=threshold)
    s = run_teacher_forced(cfg, w, dec, ec_inputs.make_prompt(cfg.vocab, 9, 6), TOL["bf16"], max_steps=6)
    print(s)
    assert s["rows_stat"] > 0
