"""The work whose speed counts: denoising steps of the model shapes this repository describes
(`ec_inputs`), whole small generations, and the vocabulary reduction as a call of its own.

`listed()` names the fixed cases, `draw()` gives more of the same ranges, `prepare()` makes what a
program holds before the call, `run()` is one pass through the public entry points, `work()` what a
pass cannot do without, `exact()` the result in 64 bits by plain torch, and `tolerance()` how far
another correct implementation of the same precision may be from it.

What one pass is, by `kind`:
  full      a new prompt: reset() and the first step, which recomputes every position
  partial   one step that recomputes the block's masked positions and the recent tokens only
  mixed     one step of a batch in which the first `n_full` sequences recompute everything and the
            others do not - what a batch does whenever some sequence's entropy was too high
  generate  reset() and generate(): the entropy-gated loop to the last token
  entropy   the reduction of logits that are on the device to (token, confidence, entropy, maximum)

Partial and mixed passes go through the teacher-forced step with nothing to commit: the whole step
runs, the state stays, and the same pass can be made again.  The tokens that the state holds were
committed by earlier such steps, so that a step sees a stale cache and a set of recent tokens.

The steps return their logits where the library leaves them: `keep_logits` stores them in the
workspace, which is the program's own tensor, and `prepare()` looks up where.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2603_18489_amd as ec

# n_layers is each case's own: most take a few layers of the full-size models
MODELS = {
    "llada8b": dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=12288,
                    vocab=126464, rope_base=500000.0),
    "dream7b": dict(d_model=3584, n_heads=28, n_kv_heads=4, head_dim=128, d_ffn=18944,
                    vocab=152064, rope_base=1e6),
}
MATRICES = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


def _step_case(name, kind, model, layers, prompt, gen, block=32, k=2, n=1, batch=1, dtype="bf16",
               scale=8.0, tau=1.0, n_full=0, ragged=0, sliding=False):
    return dict(name=name, kind=kind, n_layers=layers, **MODELS[model], dtype=dtype, scale=scale,
                prompt=prompt, gen=gen, block=block, k=k, n=n, batch=batch, tau=tau,
                n_full=n_full, ragged=ragged, sliding=sliding)


def _small_case(name, kind, d, heads, kv_heads, hd, ffn, vocab, layers, prompt, gen, block=32, k=2,
                n=1, batch=1, dtype="bf16", scale=16.0, tau=2.0, n_full=0, ragged=0, sliding=False):
    return dict(name=name, kind=kind, n_layers=layers, d_model=d, n_heads=heads,
                n_kv_heads=kv_heads, head_dim=hd, d_ffn=ffn, vocab=vocab, rope_base=10000.0,
                dtype=dtype, scale=scale, prompt=prompt, gen=gen, block=block, k=k, n=n,
                batch=batch, tau=tau, n_full=n_full, ragged=ragged, sliding=sliding)


def listed():
    return [
        # a sampler that asks for the statistics of a few rows, inside a loop that cannot allocate
        dict(name="entropy_few", kind="entropy", rows=7, vocab=4096, pad=0, alloc=False),
        # the same for a whole block at a full-size vocabulary
        dict(name="entropy_many", kind="entropy", rows=128, vocab=126464, pad=0, alloc=True),
        # the float32 model's whole generation: 64 small steps, launches and latency
        _small_case("tiny_f32_generate", "generate", 256, 4, 4, 64, 768, 4096, 2, 64, 64,
                    dtype="f32"),
        # a small bf16 model's step: nothing to stream, launches and latency
        _small_case("small_partial", "partial", 256, 4, 2, 64, 768, 4096, 2, 64, 64),
        # the two modes of the headline model at full depth
        _step_case("llada8b_partial", "partial", "llada8b", 32, 512, 256),
        _step_case("llada8b_full", "full", "llada8b", 32, 512, 256),
        # grouped-query attention, the widest feed-forward, 1280 positions
        _step_case("dream7b_full", "full", "dream7b", 8, 1024, 256, n=2),
        # the paper's own budget of 64 recent tokens: 96 rows
        _step_case("llada8b_recent64_partial", "partial", "llada8b", 8, 512, 256, k=64,
                   sliding=True),
        # 16 sequences: every one partial, two of them full, and the first step
        _step_case("llada8b_b16_partial", "partial", "llada8b", 8, 1024, 512, batch=16),
        _step_case("llada8b_b16_mixed", "mixed", "llada8b", 8, 1024, 512, batch=16, n_full=2),
        _step_case("llada8b_b16_full", "full", "llada8b", 4, 1024, 512, batch=16),
        # matrices as e4m3 codes
        _step_case("llada8b_fp8_partial", "partial", "llada8b", 8, 512, 256, dtype="fp8w"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    most = 2.6e13   # the largest listed case's flops
    while True:
        what = rng.random()
        if what < 0.2:
            return dict(kind="entropy", rows=_log_int(rng, 1, 128), vocab=_log_int(rng, 1000, 163840),
                        pad=rng.choice([0, 0, 1, 3, 64]), alloc=rng.random() < 0.5)
        if what < 0.3:
            heads = rng.choice([2, 4, 8])
            c = _small_case("", "generate", rng.choice([128, 256, 512]), heads,
                            rng.choice([heads, heads // 2]), rng.choice([64, 128]),
                            8 * rng.randint(32, 192), _log_int(rng, 1000, 8192), rng.randint(1, 3),
                            _log_int(rng, 8, 200), rng.randint(24, 80), block=rng.choice([8, 16, 32]),
                            k=rng.randint(0, 8), n=rng.randint(1, 4), dtype="f32")
        else:
            kind = "partial" if what < 0.65 else "full" if what < 0.85 else "mixed"
            batch = 1 if rng.random() < 0.6 else _log_int(rng, 2, 16)
            if kind == "mixed":
                batch = _log_int(rng, 2, 16)
            block = rng.choice([16, 32, 32, 32, rng.randint(5, 64)])
            k = rng.choice([0, 2, 2, 4, rng.randint(1, 64)])
            common = dict(block=block, k=k, n=rng.choice([1, 1, 2]), batch=batch,
                          dtype=rng.choice(["bf16", "bf16", "fp8w"]),
                          n_full=rng.randint(1, max(1, batch - 1)) if kind == "mixed" else 0,
                          ragged=rng.choice([0, rng.randint(1, 50)]) if batch > 1 else 0,
                          sliding=rng.random() < 0.3)
            prompt = _log_int(rng, 16, 3000)
            gen = 2 * block + (k + block - 1) // block * block + rng.randint(1, 300)
            if rng.random() < 0.6:
                c = _step_case("", kind, rng.choice(["llada8b", "llada8b", "dream7b"]),
                               rng.randint(1, 6), prompt, gen, **common)
            else:
                hd, heads = rng.choice([64, 128]), rng.choice([4, 8, 12, 16])
                c = _small_case("", kind, 64 * rng.randint(4, 32), heads,
                                rng.choice([heads, heads // 2, heads // 4]), hd,
                                64 * rng.randint(8, 96), 16 * _log_int(rng, 256, 4000),
                                rng.randint(1, 6), prompt, gen, **common)
        del c["name"]
        if work(c)["flops"] <= most:
            return c


# ---- inputs ------------------------------------------------------------------------------------
def _cfg(case):
    return SimpleNamespace(
        n_layers=case["n_layers"], d_model=case["d_model"], n_heads=case["n_heads"],
        n_kv_heads=case["n_kv_heads"], head_dim=case["head_dim"], d_ffn=case["d_ffn"],
        vocab=case["vocab"], mask_id=case["vocab"] - 1, rms_eps=1e-5,
        rope_base=case["rope_base"], logit_scale=case["scale"], dtype=case["dtype"])


def _dec(case):
    return SimpleNamespace(
        batch=case["batch"], gen_len=case["gen"], block=case["block"], k_recent=case["k"],
        tokens_per_step=case["n"], tau=case["tau"], conf_threshold=0.0, gate_metric=0,
        schedule=1 if case["sliding"] else 0)


def _weights(case, seed):
    """Matrices N(0, 0.02), norm gains around 1, in the model's storage type."""
    c = _cfg(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = torch.float32 if c.dtype == "f32" else torch.bfloat16

    def normal(*shape):
        return torch.empty(shape, dtype=kind, device="cuda").normal_(0.0, 0.02, generator=gen)

    def gain():
        g = torch.empty(c.d_model, device="cuda").normal_(1.0, 0.1, generator=gen)
        return g.to(kind)

    nq, nkv = c.n_heads * c.head_dim, c.n_kv_heads * c.head_dim
    shapes = {"wq": (nq, c.d_model), "wk": (nkv, c.d_model), "wv": (nkv, c.d_model),
              "wo": (c.d_model, nq), "w_gate": (c.d_ffn, c.d_model), "w_up": (c.d_ffn, c.d_model),
              "w_down": (c.d_model, c.d_ffn)}
    w = {"tok_emb": normal(c.vocab, c.d_model), "lm_head": normal(c.vocab, c.d_model),
         "final_norm": gain(), "attn_norm": [], "mlp_norm": []}
    w.update({m: [] for m in MATRICES})
    for _ in range(c.n_layers):
        w["attn_norm"].append(gain())
        w["mlp_norm"].append(gain())
        for m in MATRICES:
            w[m].append(normal(*shapes[m]))
    if c.dtype == "fp8w":
        def coded(x):
            scale = x.abs().amax(dim=1).float() / 448.0
            return (x.float() / scale[:, None]).to(torch.float8_e4m3fn).view(torch.uint8), scale
        w["lm_head"], w["lm_head_scale"] = coded(w["lm_head"])
        for m in MATRICES:
            pairs = [coded(x) for x in w[m]]
            w[m], w[m + "_scale"] = [p[0] for p in pairs], [p[1] for p in pairs]
    return w


def _prompts(case, seed):
    rng = np.random.default_rng(seed)
    return [[int(t) for t in rng.integers(0, case["vocab"] - 96, size=n)]
            for n in _prompt_lengths(case)]


def _prompt_lengths(case):
    return [max(1, case["prompt"] - b * case["ragged"] % max(1, case["prompt"] // 2 + 1))
            for b in range(case["batch"])]


def _commits(case, seed):
    """Per sequence, what earlier steps committed: a list of (slots, tokens), one per step.  Whole
    blocks are decoded, the last k tokens of them in the last steps, so that the state's step sees
    a full block of masked positions and k recent tokens."""
    block, k = case["block"], case["k"]
    total = block * max(1, -(-k // block))
    cuts = []
    for lo, hi in ((0, total - k), (total - k, total)):
        cuts += [(a, min(a + 32, hi)) for a in range(lo, hi, 32)]
    rng = np.random.default_rng(seed + 1)
    return [[(list(range(a, b)), [int(t) for t in rng.integers(0, case["vocab"] - 96, size=b - a)])
             for a, b in cuts] for _ in range(case["batch"])]


def _logits_in(workspace, block, rows, vocab):
    """The part of the workspace that holds `rows` rows of logits, the first of them `block`."""
    words = workspace[: workspace.numel() // 256 * 256].view(torch.int32)[::64]
    block = torch.from_numpy(block).cuda()
    first = block.view(torch.int32).reshape(-1)[0]
    for at in (words == first).nonzero().reshape(-1).tolist():
        z = workspace[at * 256: at * 256 + rows * vocab * 4]
        if z.numel() == rows * vocab * 4:
            z = z.view(torch.float32).view(rows, vocab)
            if torch.equal(z[: block.shape[0]], block):
                return z
    raise RuntimeError("the step's logits are not in the workspace")


def prepare(case, seed):
    if case["kind"] == "entropy":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        rows, vocab = case["rows"], case["vocab"]
        # rows of different sharpness
        sharp = torch.empty(rows, 1, device="cuda").uniform_(0.5, 12.0, generator=gen)
        buf = torch.empty(rows, vocab + case["pad"], device="cuda").normal_(0.0, 1.0, generator=gen)
        buf *= sharp
        return {"case": case, "logits": buf[:, :vocab],
                "stats": torch.empty(rows, 4, device="cuda")}
    batch = case["batch"]
    prompts = _prompts(case, seed)
    g = ec.EntropyCache(_cfg(case), _weights(case, seed), _dec(case),
                        prompts if batch > 1 else prompts[0])
    g.keep_logits(True)
    if case["kind"] in ("full", "generate"):
        r = g.step(ec.EC_AUTO)
    else:
        none = [[]] * batch
        r = _forced(g, [ec.EC_FULL] * batch, none, none)
        commits = _commits(case, seed)
        for i in range(len(commits[0])):
            _forced(g, [ec.EC_PARTIAL] * batch,
                    [[len(p) + s for s in c[i][0]] for p, c in zip(prompts, commits)],
                    [c[i][1] for c in commits])
        r = _forced(g, [ec.EC_PARTIAL] * batch, none, none)
    rows = [x["n_block_rows"] for x in (r if isinstance(r, list) else [r])]
    state = {"case": case, "g": g, "prompts": prompts if batch > 1 else prompts[0],
             "modes": [ec.EC_FULL if b < case["n_full"] else ec.EC_PARTIAL for b in range(batch)],
             "none": [[]] * batch}
    state["logits"] = _logits_in(g._workspace, g.debug_read(ec.EC_DBG_LOGITS, count=rows[0]),
                                 sum(rows), case["vocab"])
    return state


# ---- one pass ----------------------------------------------------------------------------------
def _forced(g, modes, positions, tokens):
    if g.B == 1:
        return g.step_forced(modes[0], positions[0], tokens[0])
    return g.step_forced_batch(modes, positions, tokens)


def run(state):
    kind = state["case"]["kind"]
    if kind == "entropy":
        if state["case"]["alloc"]:
            s = ec.row_entropy(state["logits"])
        else:
            s = state["stats"]
            ec.row_entropy_noalloc(state["logits"], s)
        return {"token": s[:, 0], "confidence": s[:, 1], "entropy": s[:, 2], "maximum": s[:, 3]}
    g = state["g"]
    if kind == "full":
        g.reset(state["prompts"])
        g.step(ec.EC_AUTO)
        return {"logits": state["logits"]}
    if kind == "generate":
        g.reset(state["prompts"])
        tokens, stats = g.generate()
        # the last step decodes what is left of the last block
        left = (state["case"]["gen"] - 1) % state["case"]["block"] % state["case"]["n"] + 1
        return {"tokens": tokens, "full_steps": stats["full_steps"],
                "rows": stats["rows_recomputed"], "logits": state["logits"][:left]}
    _forced(g, state["modes"], state["none"], state["none"])
    return {"logits": state["logits"]}


# ---- what a pass cannot do without -------------------------------------------------------------
def work(case):
    if case["kind"] == "entropy":
        n = case["rows"] * case["vocab"]
        return {"bytes": 4 * n + 16 * case["rows"], "flops": 6 * n}
    d, f, v, n_layers = case["d_model"], case["d_ffn"], case["vocab"], case["n_layers"]
    nq, nkv = case["n_heads"] * case["head_dim"], case["n_kv_heads"] * case["head_dim"]
    es = 4 if case["dtype"] == "f32" else 2
    ws = {"f32": 4, "bf16": 2, "fp8w": 1}[case["dtype"]]
    params = n_layers * ((nq + 2 * nkv) * d + d * nq + 3 * f * d)
    lengths = [n + case["gen"] for n in _prompt_lengths(case)]

    def step(modes):
        rows = [t if full else case["block"] + case["k"] for t, full in zip(lengths, modes)]
        lm = len(lengths) * case["block"]
        kv = n_layers * 2 * nkv * es
        nbytes = (params + v * d) * ws + sum(rows) * d * es + lm * v * 4
        # every cached key and value that the step does not make itself is read, every new one written
        nbytes += sum(max(0, t - r) + r for t, r in zip(lengths, rows)) * kv
        flops = 2.0 * params * sum(rows) + 2.0 * lm * v * d
        flops += sum(4.0 * n_layers * r * t * nq for r, t in zip(rows, lengths))
        return np.array([nbytes, flops])

    if case["kind"] == "generate":
        total = step([True]) + (-(-case["gen"] // case["n"]) - 1) * step([False])
    elif case["kind"] == "full":
        total = step([True] * case["batch"])
    else:
        total = step([b < case["n_full"] for b in range(case["batch"])])
    return {"bytes": float(total[0]), "flops": float(total[1])}


def tolerance(case):
    if case["kind"] == "entropy":
        return {"rel": 4e-6}    # float32 sums over the vocabulary: up to 2e-7 off the exact result
    if case["dtype"] == "f32":
        return {"rel": 4e-6}    # up to 8e-7 off
    # bfloat16 operands, keys, values and probabilities: 4e-3 off the exact logits at 2 layers, 1e-2
    # at 8 and 2e-2 at 32, where the same rounding in every layer has travelled through the others
    return {"rel": min(0.03, 0.016 * math.sqrt(case["n_layers"]))}


# ---- the same in 64 bits -----------------------------------------------------------------------
class _Exact:
    """One sequence of the model in float64: the rows of a step recompute their keys and values in
    every layer, which replace the cached ones before they attend to the whole cache."""

    def __init__(self, case, w, prompt):
        self.c, self.w, self.case = _cfg(case), w, case
        self.P, self.T = len(prompt), len(prompt) + case["gen"]
        self.x = torch.full((self.T,), self.c.mask_id, dtype=torch.long, device="cuda")
        self.x[: self.P] = torch.tensor(prompt, device="cuda")
        self.masked = [False] * self.P + [True] * case["gen"]
        shape = (self.c.n_layers, self.c.n_kv_heads, self.T, self.c.head_dim)
        self.K = torch.zeros(shape, dtype=torch.float64, device="cuda")
        self.V = torch.zeros(shape, dtype=torch.float64, device="cuda")
        half = self.c.head_dim // 2
        j = torch.arange(half, dtype=torch.float64, device="cuda")
        base = float(np.float32(self.c.rope_base))
        a = torch.arange(self.T, dtype=torch.float64, device="cuda")[:, None] * base ** (-2.0 * j / self.c.head_dim)
        self.cos, self.sin = a.cos(), a.sin()

    def norm(self, h, gain):
        return h / (h.square().mean(dim=1, keepdim=True) + float(np.float32(self.c.rms_eps))).sqrt() * gain.double()

    def rope(self, v, rows):
        c, s = self.cos[rows][:, None], self.sin[rows][:, None]
        a, b = v.chunk(2, dim=-1)
        return torch.cat([a * c - b * s, b * c + a * s], dim=-1)

    def block(self):
        left = [p for p in range(self.P, self.T) if self.masked[p]]
        if self.case["sliding"] or not left:
            return left[: self.case["block"]]
        at = (left[0] - self.P) // self.case["block"]
        return [p for p in left if (p - self.P) // self.case["block"] == at]

    def layer(self, l, m, h, rows):
        """Layer l on the rows' residual stream; m: its matrices in float64, transposed."""
        c = self.c
        u = self.norm(h, self.w["attn_norm"][l])
        q = self.rope((u @ m["wq"]).view(-1, c.n_heads, c.head_dim), rows)
        self.K[l][:, rows] = self.rope((u @ m["wk"]).view(-1, c.n_kv_heads, c.head_dim), rows).transpose(0, 1)
        self.V[l][:, rows] = (u @ m["wv"]).view(-1, c.n_kv_heads, c.head_dim).transpose(0, 1)
        group = c.n_heads // c.n_kv_heads
        q = q.transpose(0, 1).reshape(c.n_kv_heads, group * len(rows), c.head_dim)
        o = torch.empty_like(q)
        for kv in range(c.n_kv_heads):
            s = q[kv] @ self.K[l, kv].t() / math.sqrt(c.head_dim)
            o[kv] = torch.softmax(s, dim=1) @ self.V[l, kv]
        o = o.view(c.n_heads, len(rows), c.head_dim).transpose(0, 1).reshape(len(rows), -1)
        h = h + o @ m["wo"]
        u = self.norm(h, self.w["mlp_norm"][l])
        return h + (torch.nn.functional.silu(u @ m["w_gate"]) * (u @ m["w_up"])) @ m["w_down"]


def _matrix64(w, name, at=None):
    x = w[name] if at is None else w[name][at]
    if x.dtype == torch.uint8:
        s = w[name + "_scale"] if at is None else w[name + "_scale"][at]
        return x.view(torch.float8_e4m3fn).float().double() * s.double()[:, None]
    return x.double()


def _exact_step(seqs, w, rows, scale):
    """Logits of the sequences' block rows after one step that recomputes rows[b] of sequence b."""
    rows = [torch.tensor(r, device="cuda") for r in rows]
    h = [w["tok_emb"][s.x[r]].double() for s, r in zip(seqs, rows)]
    for l in range(seqs[0].c.n_layers):
        m = {name: _matrix64(w, name, l).t() for name in MATRICES}
        h = [s.layer(l, m, x, r) for s, x, r in zip(seqs, h, rows)]
    u = []
    for s, x, r in zip(seqs, h, rows):
        at = torch.isin(r, torch.tensor(s.block(), device="cuda"))
        u.append(s.norm(x[at], w["final_norm"]))
    return torch.cat(u) @ _matrix64(w, "lm_head").t() * float(np.float32(scale))


def _exact_generate(case, s, w):
    """The entropy-gated loop: everything is recomputed while a step's largest entropy is over tau."""
    hist, t, last_full, full, n_full, n_rows = {}, 1, 0, True, 0, 0
    while any(s.masked):
        if full:
            rows, last_full = list(range(s.T)), t
        else:
            rows = sorted(set(s.block()) | recent)  # noqa: F821 (the first step is full)
        n_full, n_rows, block = n_full + full, n_rows + len(rows), s.block()
        z = _exact_step([s], w, [rows], case["scale"])
        p = torch.softmax(z, dim=1)
        conf, tok = p.max(dim=1)
        ent = -torch.special.xlogy(p, p).sum(dim=1)
        best = sorted(range(len(block)), key=lambda i: (-conf[i].item(), i))[: case["n"]]
        for i in best:
            s.x[block[i]] = tok[i]
            s.masked[block[i]] = False
            hist[block[i]] = t
        kth = sorted(hist.values(), reverse=True)[case["k"] - 1] if 0 < case["k"] <= len(hist) else 0
        since = max(kth, last_full) if case["k"] else t + 1
        recent = {q for q, at in hist.items() if at >= since}
        full = max(ent[i].item() for i in best) > case["tau"]
        t += 1
    return {"tokens": s.x[s.P:].to(torch.int32), "full_steps": n_full, "rows": n_rows, "logits": z}


def exact(case, seed):
    if case["kind"] == "entropy":
        z = prepare(case, seed)["logits"].double()
        p = torch.softmax(z, dim=1)
        return {"token": z.argmax(dim=1).double(), "confidence": p.amax(dim=1),
                "entropy": -torch.special.xlogy(p, p).sum(dim=1), "maximum": z.amax(dim=1)}
    w = _weights(case, seed)
    seqs = [_Exact(case, w, p) for p in _prompts(case, seed)]
    if case["kind"] == "generate":
        return _exact_generate(case, seqs[0], w)
    every = [list(range(s.T)) for s in seqs]
    z = _exact_step(seqs, w, every, case["scale"])
    if case["kind"] == "full":
        return {"logits": z}
    # the steps that committed the state's tokens, then the one that counts
    commits = _commits(case, seed)
    recent = [[(0, p) for p in ()] for _ in seqs]
    for i in range(len(commits[0]) + 1):
        rows = []
        for b, s in enumerate(seqs):
            last = i == len(commits[0])
            full = last and case["kind"] == "mixed" and b < case["n_full"]
            rows.append(every[b] if full else sorted(set(s.block()) | set(_recent(recent[b], case["k"]))))
        z = _exact_step(seqs, w, rows, case["scale"])
        if i < len(commits[0]):
            for b, s in enumerate(seqs):
                slots, tokens = commits[b][i]
                for slot, tok in zip(slots, tokens):
                    s.x[s.P + slot] = tok
                    s.masked[s.P + slot] = False
                    recent[b].append((i + 2, s.P + slot))
    return {"logits": z}


def _recent(hist, k):
    """Positions decoded at or after the step of the k-th latest one (any since the full step)."""
    if k == 0:
        return []
    at = sorted((t for t, _ in hist), reverse=True)
    since = at[k - 1] if k <= len(at) else 1
    return [p for t, p in hist if t >= since]
