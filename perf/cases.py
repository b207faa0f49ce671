"""Performance cases of the rollout engine: the calls that a reinforcement-learning program makes,
at the layer shapes of the benchmark configurations, through the public entry points.

Kinds of case
  step    one april_rollout_step (prefill, then decode until `n` of `n_over` rollouts are complete);
          `steps` = 2 parks the unfinished rollouts and resumes them in a second step
  resume  token-level rollouts imported, resumed by re-prefill and decoded to their limit
  score   prompts prefilled in parity mode, the logits after each prompt returned
  sample  the sampler alone on a device array of logits

Rollouts return their tokens and the log-probability of each over the whole vocabulary (what a
trainer's importance ratio needs).  The models are random-init decoders whose LM head also holds the
embedding of the preceding token of a fixed cycle: as in a trained model the next token is likely
(p around one half) and the arg-max does not hang on the last bits of the arithmetic.  Projections
into the residual stream are scaled by 1 / sqrt(layers), a usual initialisation.
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2509_18521_amd as ap

# Layer shapes: the benchmark configurations, and one whose dimensions are odd multiples of 32.
SHAPES = {
    "tiny": dict(d_model=128, n_q_heads=4, n_kv_heads=4, head_dim=32, d_ffn=512, vocab=512, dtype=0),
    "small": dict(d_model=896, n_q_heads=14, n_kv_heads=2, head_dim=64, d_ffn=4864, vocab=151936),
    "mid": dict(d_model=2560, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ffn=9728, vocab=151936),
    "8b": dict(d_model=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ffn=14336, vocab=128256),
    "moe": dict(d_model=2048, n_q_heads=32, n_kv_heads=4, head_dim=128, d_ffn=0, vocab=151936,
                n_experts=128, experts_per_tok=8, d_expert_ffn=768),
    "odd": dict(d_model=1184, n_q_heads=20, n_kv_heads=4, head_dim=64, d_ffn=3104, vocab=32032),
}
CYCLE = 7919            # the likely token after t is (t + CYCLE) mod vocab


def listed():
    return [
        # the fp32 configuration as it is run: 24 short rollouts in flight, 16 wanted
        dict(name="tiny_fp32_step", kind="step", shape="tiny", layers=2, n=16, n_over=24, p_lo=32, p_hi=32,
             g_lo=8, g_hi=96, sampler="greedy", steps=1),
        # a single interactive rollout on the whole 0.6 B model: nothing but latency
        dict(name="small_single", kind="step", shape="small", layers=24, n=1, n_over=1, p_lo=37, p_hi=37,
             g_lo=24, g_hi=24, sampler="greedy", steps=1),
        # the whole 0.6 B model with the evaluation sampling (top-k, top-p), over-provisioned
        dict(name="small_step", kind="step", shape="small", layers=24, n=64, n_over=96, p_lo=256, p_hi=256,
             g_lo=32, g_hi=160, sampler="topk", steps=1),
        # layers of the 4.4 B model at the default workload's batch: 512-token prompts, 192 in flight
        dict(name="mid_step", kind="step", shape="mid", layers=4, n=128, n_over=192, p_lo=512, p_hi=512,
             g_lo=48, g_hi=192, sampler="greedy", steps=1),
        # layers of the 8 B model with 384 rollouts in flight and short ragged prompts: decode projections
        dict(name="8b_wide_step", kind="step", shape="8b", layers=2, n=256, n_over=384, p_lo=16, p_hi=250,
             g_lo=48, g_hi=160, sampler="greedy", steps=1),
        # layers of the routed-expert model
        dict(name="moe_step", kind="step", shape="moe", layers=2, n=160, n_over=240, p_lo=64, p_hi=400,
             g_lo=32, g_hi=96, sampler="greedy", steps=1),
        # a few rollouts deep in the response tail: long contexts, split over several KV ranges
        dict(name="8b_long_context", kind="step", shape="8b", layers=2, n=7, n_over=7, p_lo=4500, p_hi=8001,
             g_lo=64, g_hi=96, sampler="greedy", steps=1),
        # two steps with parking and resumption, dimensions that are odd multiples of 32, ragged prompts
        dict(name="odd_two_steps", kind="step", shape="odd", layers=3, n=33, n_over=47, p_lo=3, p_hi=301,
             g_lo=16, g_hi=90, sampler="topk", steps=2),
        # parked rollouts continued under a new policy: prompt and response so far prefilled again
        dict(name="small_resume", kind="resume", shape="small", layers=6, n=19, n_over=19, p_lo=700, p_hi=3301,
             g_lo=8, g_hi=16, sampler="greedy", steps=1),
        # prompts of very different length scored in one call, logits wanted
        dict(name="mid_score", kind="score", shape="mid", layers=3, n=21, n_over=21, p_lo=1, p_hi=1999,
             g_lo=1, g_hi=1, sampler="greedy", steps=1),
        # the sampler of a training rollout: temperature over the whole vocabulary, log-probabilities
        dict(name="sample_categorical", kind="sample", mode="categorical", rows=192, vocab=151936),
        # the allocation-free sampler of a small serving loop
        dict(name="sample_topk_few", kind="sample", mode="topk", rows=5, vocab=151936),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = [_cost(c) for c in listed()]
    most = max(limit)
    while True:
        kind = rng.choice(["step", "step", "step", "step", "resume", "score", "sample"])
        if kind == "sample":
            return dict(kind="sample", mode=rng.choice(["categorical", "topk", "greedy"]), rows=_log_uniform(rng, 1, 384),
                        vocab=rng.choice([151936, 128256, 32032, 50257]))
        shape = rng.choice(list(SHAPES))
        if kind != "step" and shape == "tiny":
            continue
        n = _log_uniform(rng, 1, 24 if kind != "step" else 200)
        n_over = n if kind != "step" else min(300, n + rng.randrange(0, n // 2 + 1))
        p_hi = _log_uniform(rng, 1, 96 if shape == "tiny" else 6000)
        p_lo = rng.randrange(1, p_hi + 1)
        g_hi = 1 if kind == "score" else _log_uniform(rng, 2, 128)
        g_lo = 1 if kind == "score" else rng.randrange(1, g_hi + 1)
        c = dict(kind=kind, shape=shape, layers=rng.choice([1, 2, 3]), n=n, n_over=n_over, p_lo=p_lo, p_hi=p_hi, g_lo=g_lo,
                 g_hi=g_hi, sampler=rng.choice(["greedy", "topk"]), steps=rng.choice([1, 2]) if kind == "step" else 1)
        if _cost(c) <= 0.6 * most:
            return c


# ---------------------------------------------------------------------------
# sizes of a case (a function of the case alone, so that every seed does the same work)
# ---------------------------------------------------------------------------
def _shape(case):
    s = dict(n_experts=0, experts_per_tok=0, d_expert_ffn=0, dtype=1, rope_theta=10000.0, rms_eps=1e-6, n_layers=case["layers"])
    s.update(SHAPES[case["shape"]])
    return SimpleNamespace(**s)


def _lengths(case):
    """Prompt lengths and response limits of every request that the case can admit."""
    count = case["n_over"] + (case["steps"] - 1) * case["n"]
    rng = random.Random(1000003 * case["n_over"] + 1009 * case["p_hi"] + case["g_hi"])
    prompts = [round(case["p_lo"] + (case["p_hi"] - case["p_lo"]) * (i + 0.5) / count) for i in range(count)]
    # long-tailed responses: lognormal, clipped to the range
    mid, sigma = math.sqrt(case["g_lo"] * case["g_hi"]), 0.8
    gens = [min(case["g_hi"], max(case["g_lo"], round(mid * math.exp(sigma * rng.gauss(0, 1))))) for _ in range(count)]
    rng.shuffle(prompts)
    return prompts, gens


def _given(case):
    """Tokens a resumed rollout has already generated (a third of its length)."""
    return [p // 3 for p in _lengths(case)[0]]


def _schedule(case):
    """Per step: the delivered (id, tokens generated) in order, and for each rollout in flight
    (id, tokens before the step, tokens made in it, whether it is prefilled)."""
    prompts, gens = _lengths(case)
    nxt, buffered, out = 0, [], []                      # buffered: (id, generated, done)
    for _ in range(case["steps"]):
        done = [b for b in buffered if b[2]]
        live = [(b[0], b[1], False) for b in buffered if not b[2]]
        while len(live) < case["n_over"] - len(done) and nxt < len(prompts):
            live.append((nxt, 0, True))
            nxt += 1
        want = case["n"] - len(done)
        rest = sorted(gens[i] - g for i, g, _ in live)
        iters = rest[want - 1] if want > 0 else 0
        fins = sorted((gens[i] - g, i) for i, g, _ in live if gens[i] - g <= iters) if want > 0 else []
        order = [b[0] for b in done] + [i for _, i in fins]
        out.append(([(i, gens[i]) for i in order[:case["n"]]], [(i, g, min(iters, gens[i] - g), new) for i, g, new in live], iters))
        over = set(order[case["n"]:])
        ended = set(order)
        buffered = sorted([(i, gens[i], True) for i in over] +
                          [(i, g + iters, False) for i, g, _ in live if i not in ended])
    return out


def _layer_params(s):
    attn = s.d_model * s.head_dim * (2 * s.n_q_heads + 2 * s.n_kv_heads)
    return attn, (s.n_experts * s.d_model if s.n_experts else 3 * s.d_model * s.d_ffn), 3 * s.d_model * s.d_expert_ffn


def work(case):
    if case["kind"] == "sample":
        return {"bytes": 4.0 * case["rows"] * case["vocab"], "flops": 2.0 * case["rows"] * case["vocab"]}
    s = _shape(case)
    e = 2 if s.dtype else 4
    prompts, _ = _lengths(case)
    attn, mlp, expert = _layer_params(s)
    per_token = 2.0 * s.n_layers * (attn + mlp + s.experts_per_tok * expert)
    kv = 2.0 * s.n_layers * s.n_kv_heads * s.head_dim * e
    score = 4.0 * s.n_layers * s.n_q_heads * s.head_dim
    head = float(s.d_model * s.vocab)
    given = _given(case) if case["kind"] == "resume" else [0] * len(prompts)
    nbytes = flops = 0.0

    def weights(rows):
        hit = s.n_experts * (1 - (1 - s.experts_per_tok / s.n_experts) ** rows) if s.n_experts else 0
        return e * (s.n_layers * (attn + mlp + hit * expert) + head)

    for _, flight, iters in _schedule(case):
        pre = [(prompts[i] + given[i]) for i, _, _, new in flight if new]
        if pre:
            nbytes += weights(sum(pre)) + kv * sum(pre)
            flops += per_token * sum(pre) + score * sum(p * (p + 1) / 2 for p in pre) + 2 * head * len(pre)
        for it in range(1, iters + 1):
            rows = [(prompts[i] + given[i] + g + it - 1) for i, g, made, new in flight if made >= it and not (new and it == 1)]
            if rows:
                nbytes += weights(len(rows)) + kv * sum(rows)
                flops += len(rows) * (per_token + 2 * head) + score * sum(rows)
    return {"bytes": nbytes, "flops": flops}


def _cost(case):
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / 1e15


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _weights(case, seed):
    s = _shape(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7 + 1)
    dt = torch.bfloat16 if s.dtype else torch.float32

    def lin(*shape, by=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * (by / math.sqrt(shape[-1]))).to(dt)

    def gain():
        return 1 + 0.1 * torch.randn(s.d_model, generator=g, device="cuda")

    nq, nkv, d = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.d_model
    into = 1 / math.sqrt(s.n_layers)
    w = {"tok_emb": torch.randn(s.vocab, d, generator=g, device="cuda").to(dt)}
    for l in range(s.n_layers):
        w[f"attn_norm.{l}"], w[f"mlp_norm.{l}"] = gain(), gain()
        w[f"wq.{l}"], w[f"wk.{l}"], w[f"wv.{l}"], w[f"wo.{l}"] = lin(nq, d), lin(nkv, d), lin(nkv, d), lin(d, nq, by=into)
        if s.n_experts:
            w[f"router.{l}"] = lin(s.n_experts, d)
            w[f"e_gate.{l}"], w[f"e_up.{l}"] = lin(s.n_experts, s.d_expert_ffn, d), lin(s.n_experts, s.d_expert_ffn, d)
            w[f"e_down.{l}"] = lin(s.n_experts, d, s.d_expert_ffn, by=into)
        else:
            w[f"w_gate.{l}"], w[f"w_up.{l}"], w[f"w_down.{l}"] = lin(s.d_ffn, d), lin(s.d_ffn, d), lin(d, s.d_ffn, by=into)
    w["final_norm"] = gain()
    # the embedding keeps about 1 / sqrt(1.5) of the final residual stream
    tied = (math.log(s.vocab) + 0.5) * math.sqrt(1.5 / d)
    w["lm_head"] = ((0.25 * torch.randn(s.vocab, d, generator=g, device="cuda") +
                     tied * torch.roll(w["tok_emb"].float(), CYCLE % s.vocab, 0)) / math.sqrt(d)).to(dt)
    return s, w


def _tokens(case, seed):
    """Prompts of every request, and their responses: the cycle of likely tokens."""
    s = _shape(case)
    prompts, gens = _lengths(case)
    given = _given(case) if case["kind"] == "resume" else [0] * len(prompts)
    rng = np.random.default_rng([seed, 5])
    p = [rng.integers(0, s.vocab, n, dtype=np.int32) for n in prompts]
    before = [rng.integers(0, s.vocab, n, dtype=np.int32) for n in given]
    chain = []
    for i in range(len(p)):
        last = int((before[i] if given[i] else p[i])[-1])
        chain.append(np.array([(last + CYCLE * (k + 1)) % s.vocab for k in range(gens[i])], dtype=np.int32))
    return p, before, chain


class State:
    """An engine and what a program passes to it."""

    ctx = None

    def __del__(self):
        if self.ctx is not None:
            ap.april_destroy(self.ctx)


def prepare(case, seed):
    st = State()
    st.case = case
    if case["kind"] == "sample":
        s = SimpleNamespace(n_layers=1, d_model=8, n_q_heads=1, n_kv_heads=1, head_dim=32, d_ffn=8, vocab=case["vocab"],
                            n_experts=0, experts_per_tok=0, d_expert_ffn=0, dtype=0, rope_theta=10000.0, rms_eps=1e-6)
        z = lambda *n: np.zeros(n, np.float32)  # noqa: E731
        w = {"tok_emb": z(s.vocab, 8), "attn_norm.0": z(8), "mlp_norm.0": z(8), "wq.0": z(32, 8), "wk.0": z(32, 8), "wv.0": z(32, 8),
             "wo.0": z(8, 32), "w_gate.0": z(8, 8), "w_up.0": z(8, 8), "w_down.0": z(8, 8), "final_norm": z(8), "lm_head": z(s.vocab, 8)}
        cfg = ap.make_cfg(s, max_inflight=4, max_ctx=32, seed=seed, **_sampling(case["mode"]))
        st.logits, st.ids, st.index = _rows(case, seed)
        st.ctx = ap.april_init(cfg, w)
        return st
    s, w = _weights(case, seed)
    p, before, chain = _tokens(case, seed)
    given = [len(b) for b in before]
    longest = max(len(a) + b + len(c) for a, b, c in zip(p, given, chain))
    score = case["kind"] == "score"
    cfg = ap.make_cfg(s, max_inflight=case["n_over"] + 4, max_ctx=longest + 16, seed=seed, logprobs=not score,
                      debug_logits=score, **_sampling(case["sampler"]))
    torch.cuda.synchronize()
    st.ctx = ap.april_init(cfg, w)
    st.max_new = max(len(c) for c in chain) + max(given)
    st.vocab = s.vocab
    if case["kind"] == "resume":
        rng = np.random.default_rng([seed, 6])
        st.partials = [dict(request_id=i, prompt=p[i], generated=before[i], limit=given[i] + len(chain[i]),
                            logprobs=-rng.random(given[i]).astype(np.float32)) for i in range(len(p))]
    else:
        st.requests = [dict(request_id=i, tokens=p[i], forced_len=len(chain[i])) for i in range(len(p))]
    if score:
        for i in range(len(p)):
            ap.april_debug_watch(st.ctx, i, 0, 1)
    return st


def _sampling(mode):
    if mode == "greedy":
        return dict(sampler=ap.APRIL_SAMPLER_GREEDY)
    if mode == "topk":
        return dict(sampler=ap.APRIL_SAMPLER_TOPK, top_k=50, top_p=0.7, temperature=1.0)
    return dict(sampler=ap.APRIL_SAMPLER_CATEGORICAL, temperature=0.8)


def _rows(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    logits = 2.5 * torch.randn(case["rows"], case["vocab"], generator=g, device="cuda")
    rng = np.random.default_rng([seed, 7])
    return logits, np.arange(case["rows"], dtype=np.int64) + 17, rng.integers(0, 4096, case["rows"], dtype=np.int32)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st.case
    if case["kind"] == "sample":
        args = (st.ctx, st.logits.data_ptr(), case["rows"], st.ids, st.index)
        if case["mode"] == "categorical":
            tokens, logprobs = ap.april_sample_rows_logprobs(*args)
            return {"tokens": tokens, "logprobs": logprobs}
        return {"tokens": ap.april_sample_rows_noalloc(*args) if case["rows"] * (case["vocab"] // 64) <= 1 << 20
                else ap.april_sample_rows(*args)}
    out = {}
    if case["kind"] == "resume":
        ap.april_resume(st.ctx, ap.april_buffer_import(st.ctx, st.partials))
        res = ap.april_rollout_step(st.ctx, [], case["n"], case["n"], st.max_new)
        _collect(out, 0, res)
    elif case["kind"] == "score":
        res = ap.april_rollout_step(st.ctx, st.requests, case["n"], case["n"], st.max_new)
        out["ids"] = np.array(res.request_id)
        out["logits"] = np.stack([ap.april_debug_logits(st.ctx, i, 0, st.vocab)[0] for i in range(case["n"])])
    else:
        used = 0
        for k in range(case["steps"]):
            if k:
                ap.april_resume(st.ctx, res.buffer)
            res = ap.april_rollout_step(st.ctx, st.requests[used:], case["n"], case["n_over"], st.max_new)
            used += res.n_new_consumed
            _collect(out, k, res)
    ap.april_buffer_free(st.ctx, res.buffer)
    return out


def _collect(out, k, res):
    out[f"ids{k}"] = np.array(res.request_id)
    out[f"tokens{k}"] = np.concatenate(res.tokens)
    out[f"logprobs{k}"] = np.concatenate(res.logprobs)


def tolerance(case):
    if case["kind"] == "sample":
        # 32-bit exponentials and 64-bit sums (3e-8 off the same in 64 bits); chosen tokens are whole numbers
        return {"rel": 1e-6, "differ": 0.0} if case["mode"] == "categorical" else "exact"
    if case["shape"] == "tiny":
        return {"rel": 2e-6, "max": 5e-5, "differ": 0.0}          # 32-bit sums: 2.6e-7 off 64 bits
    if case["shape"] == "moe":
        return {"rel": 0.012, "max": 0.5, "differ": 0.0}          # 2.6e-3 off; a near tie may pick another expert
    return {"rel": 0.01, "max": 0.3, "differ": 0.0}               # bf16 operands: 0.8e-3 to 2.4e-3 off


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _norm(x, g, eps):
    return x * g / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _rope(v, theta):
    half = v.shape[-1] // 2
    f = theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=v.device) / v.shape[-1])
    ang = (torch.arange(v.shape[0], dtype=torch.float64, device=v.device)[:, None] * f)[:, None, :]
    c, s, a, b = torch.cos(ang), torch.sin(ang), v[..., :half], v[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attention(q, k, v):
    """One sequence, causal: q [T, Hq, dh], k and v [T, Hkv, dh]."""
    T, group = q.shape[0], q.shape[1] // k.shape[1]
    out = torch.empty_like(q)
    hidden = torch.ones(T, T, dtype=torch.bool, device=q.device).triu(1)
    for h in range(k.shape[1]):
        for a in range(h * group, (h + 1) * group):
            sc = (q[:, a] @ k[:, h].T / math.sqrt(q.shape[2])).masked_fill_(hidden, -math.inf)
            out[:, a] = torch.softmax(sc, -1) @ v[:, h]
    return out


def _forward64(s, w, seqs):
    """Final hidden states of every sequence (all rows of all sequences go through a layer together)."""
    f = lambda n: w[n].double()  # noqa: E731
    cuts = np.cumsum([0] + [len(q) for q in seqs])
    x = w["tok_emb"][torch.from_numpy(np.concatenate(seqs)).cuda().long()].double()
    for l in range(s.n_layers):
        h = _norm(x, f(f"attn_norm.{l}"), s.rms_eps)
        q, k, v = ((h @ f(n).T).reshape(x.shape[0], -1, s.head_dim) for n in (f"wq.{l}", f"wk.{l}", f"wv.{l}"))
        o = [_attention(_rope(q[a:b], s.rope_theta), _rope(k[a:b], s.rope_theta), v[a:b]) for a, b in zip(cuts, cuts[1:])]
        x = x + torch.cat(o).reshape(x.shape[0], -1) @ f(f"wo.{l}").T
        h = _norm(x, f(f"mlp_norm.{l}"), s.rms_eps)
        if s.n_experts:
            r = torch.softmax(h @ f(f"router.{l}").T, -1)
            wt, ids = torch.topk(r, s.experts_per_tok, -1)
            wt = wt / wt.sum(-1, keepdim=True)
            y = torch.zeros_like(h)
            for e in range(s.n_experts):
                row, pick = torch.where(ids == e)
                z = h[row]
                a = torch.nn.functional.silu(z @ w[f"e_gate.{l}"][e].double().T) * (z @ w[f"e_up.{l}"][e].double().T)
                y[row] += wt[row, pick][:, None] * (a @ w[f"e_down.{l}"][e].double().T)
            x = x + y
        else:
            for a in range(0, x.shape[0], 16384):
                z = h[a:a + 16384]
                x[a:a + 16384] += (torch.nn.functional.silu(z @ f(f"w_gate.{l}").T) * (z @ f(f"w_up.{l}").T)) @ f(f"w_down.{l}").T
    return torch.split(_norm(x, f("final_norm"), s.rms_eps), [len(q) for q in seqs])


def _uniform(seed, ids, index):
    """Philox4x32-10 (Salmon et al., 2011): key = the sampler's seed, counter = (id, token index), 24 bits of word 0."""
    m = np.uint64(0xFFFFFFFF)
    c = [np.uint64(i) & m for i in (ids.astype(np.uint64), ids.astype(np.uint64) >> np.uint64(32), index.astype(np.uint64), 0 * ids.astype(np.uint64))]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & m, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return (c[0] >> np.uint64(8)).astype(np.float64) * 2.0 ** -24


def _sampled64(case, seed):
    logits, ids, index = _rows(case, seed)
    z = logits.double() / (0.8 if case["mode"] == "categorical" else 1.0)
    if case["mode"] == "greedy":
        return {"tokens": z.argmax(-1).int()}
    u = torch.from_numpy(_uniform(seed, ids, index)).cuda()[:, None]
    logp = torch.log_softmax(z, -1)
    if case["mode"] == "categorical":
        token = (logp.exp().cumsum(-1) <= u).sum(-1).clamp(max=case["vocab"] - 1)
        return {"tokens": token.int(), "logprobs": logp.gather(1, token[:, None])[:, 0]}
    top, at = torch.topk(z, 50, -1)
    p = torch.softmax(top, -1)
    before = p.cumsum(-1) - p
    p = torch.where(before >= np.float32(0.7), 0.0, p)
    pick = ((p / p.sum(-1, keepdim=True)).cumsum(-1) <= u).sum(-1).clamp(max=49)
    return {"tokens": at.gather(1, pick[:, None])[:, 0].int()}


def exact(case, seed):
    if case["kind"] == "sample":
        return _sampled64(case, seed)
    prompts, _ = _lengths(case)
    s = _shape(case)
    if work(case)["flops"] > 3e14:
        return None
    s, w = _weights(case, seed)
    p, before, chain = _tokens(case, seed)
    plan = _schedule(case)
    wanted = sorted({i for done, _, _ in plan for i, _ in done})
    hid = {}
    for a in range(0, len(wanted), 48):
        part = wanted[a:a + 48]
        for i, h in zip(part, _forward64(s, w, [np.concatenate([p[i], before[i], chain[i][:-1]]) for i in part])):
            hid[i] = h[-len(chain[i]):].clone()
    head = w["lm_head"].double()
    if case["kind"] == "score":
        return {"ids": np.arange(case["n"]), "logits": torch.cat([hid[i] for i in range(case["n"])]) @ head.T}
    logp = {}
    for i in wanted:
        z = torch.log_softmax(hid[i] @ head.T, -1)
        own = torch.from_numpy(chain[i]).cuda().long()
        if not torch.equal(z.argmax(-1), own):
            return None                                  # not the likely token everywhere: no closed answer
        logp[i] = z.gather(1, own[:, None])[:, 0].cpu().numpy()
    rng = np.random.default_rng([seed, 6])
    old = [-rng.random(len(b)).astype(np.float32) for b in before]
    out = {}
    for k, (done, _, _) in enumerate(plan):
        out[f"ids{k}"] = np.array([i for i, _ in done])
        out[f"tokens{k}"] = np.concatenate([np.concatenate([before[i], chain[i]]) for i, _ in done])
        out[f"logprobs{k}"] = np.concatenate([np.concatenate([old[i].astype(np.float64), logp[i]]) for i, _ in done])
    return out
