"""The fp32 kernels against the oracle at ragged sizes: inner dimensions that 4 or 16 do not divide, one
output column, contexts around the attention's steps of 64 tokens, every head size.
Bound: a dot product of at most 200 fp32 terms of size about 1 (2^-24 x sqrt(200) relative), a dozen of
them in a row, on logits of size below 10: 1e-4, as for the other fp32 comparisons."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts
from oracle.model import Decoder

pytestmark = pytest.mark.gpu
LENGTHS = [1, 2, 15, 17, 63, 64, 65, 127, 129, 200]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("head_dim,n_q,n_kv,d_model,d_ffn,vocab", [
    (32, 3, 1, 40, 13, 37), (64, 2, 2, 8, 1, 1), (128, 4, 2, 72, 50, 130), (32, 4, 4, 128, 200, 257)])
def test_ragged_fp32_models(head_dim, n_q, n_kv, d_model, d_ffn, vocab):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, d_model, n_q, n_kv, head_dim, d_ffn, vocab, dtype=ai.DTYPE_FP32)
    n, gen = len(LENGTHS), 4
    w = ai.Workload("fp32", shape, 1, max(LENGTHS), n, n, gen, 0.0, 0.1, gen, gen, ai.SAMPLER_GREEDY, 0, 1, 7)
    weights = ai.make_weights(shape, w.seed)
    rng = np.random.default_rng(d_model)
    reqs = [ai.Request(i, rng.integers(0, vocab, t, dtype=np.int32), gen) for i, t in enumerate(LENGTHS)]
    forced = {i: rng.integers(0, vocab, gen, dtype=np.int32) for i in range(n)}
    dec = Decoder(shape, weights)
    ctx = make_engine(w, weights, debug=True)
    try:
        for r in reqs:
            ap.april_debug_watch(ctx, r.request_id, 0, gen)
        ap.april_rollout_step(ctx, req_dicts(reqs, forced), n, n, gen)
        for r in reqs:
            ref = dec.forward_block(np.concatenate([r.tokens, forced[r.request_id][:-1]]), dec.new_cache())[-gen:]
            for g in range(gen):
                got, _ = ap.april_debug_logits(ctx, r.request_id, g, vocab)
                assert np.max(np.abs(got - ref[g])) <= 1e-4, (len(r.tokens), g)
    finally:
        ap.april_destroy(ctx)


@pytest.mark.parametrize("head_dim,n_q,n_kv,d_model,d_ffn,vocab,n", [
    (32, 4, 4, 128, 512, 512, 24), (32, 6, 2, 72, 52, 131, 40), (64, 2, 1, 40, 4, 1, 9), (128, 2, 1, 128, 320, 700, 300)])
def test_decode_in_one_launch_keeps_a_prefilled_rollouts_bits(head_dim, n_q, n_kv, d_model, d_ffn, vocab, n):
    """Models whose decode pass is one launch: logits of positions reached by decoding are those of the same tokens
    prefilled, bit for bit, alone and in a batch, across page and attention-step boundaries; and the oracle's."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, d_model, n_q, n_kv, head_dim, d_ffn, vocab, dtype=ai.DTYPE_FP32)
    gen, prompt = 3, [1, 14, 15, 16, 61, 62, 63, 64, 126, 127, 190]
    w = ai.Workload("fp32", shape, 1, 200, n, n, gen, 0.0, 0.1, gen, gen, ai.SAMPLER_GREEDY, 0, 1, 7)
    weights = ai.make_weights(shape, w.seed)
    rng = np.random.default_rng(d_model)
    text = rng.integers(0, vocab, 256, dtype=np.int32)
    dec = Decoder(shape, weights)
    ref = dec.forward_block(text[:200], dec.new_cache())
    got = {}
    for shift in (0, 1):                     # shift 1: what was decoded first is now the prompt's last token
        ctx = make_engine(w, weights, debug=True, max_inflight=n)
        reqs = [ai.Request(i, text[:prompt[i % len(prompt)] + shift], gen - shift) for i in range(n)]
        forced = {r.request_id: text[len(r.tokens):len(r.tokens) + gen] for r in reqs}
        try:
            for r in reqs[:22]:
                ap.april_debug_watch(ctx, r.request_id, 0, gen - shift)
            ap.april_rollout_step(ctx, req_dicts(reqs, forced), n, n, gen)
            for r in reqs[:22]:
                for g in range(gen - shift):
                    at, row = len(r.tokens) + g - 1, ap.april_debug_logits(ctx, r.request_id, g, vocab)[0]
                    assert np.max(np.abs(row - ref[at])) <= 1e-4, (len(r.tokens), g)
                    got.setdefault(at, []).append(row)
        finally:
            ap.april_destroy(ctx)
    for at, rows in got.items():
        assert all(np.array_equal(rows[0], x) for x in rows[1:]), at


@pytest.mark.parametrize("head_dim,n_q,n_kv,d_model,d_ffn,vocab", [(32, 6, 2, 72, 52, 131), (64, 2, 1, 40, 4, 65), (32, 4, 4, 128, 512, 512)])
def test_small_models_prompt_bits_do_not_depend_on_the_pass(head_dim, n_q, n_kv, d_model, d_ffn, vocab):
    """The rows of a pass pick the columns per workgroup of its products (32, 64 and 128, with ends inside one): same sums."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, d_model, n_q, n_kv, head_dim, d_ffn, vocab, dtype=ai.DTYPE_FP32)
    weights = ai.make_weights(shape, 3)
    rng = np.random.default_rng(vocab)
    prompts = [rng.integers(0, vocab, t, dtype=np.int32) for t in (5, 33, 64)]
    dec = Decoder(shape, weights)
    ref = [dec.forward_block(p, dec.new_cache())[-1] for p in prompts]
    alone = None
    for n in (3, 1, 12, 30, 150):
        w = ai.Workload("fp32", shape, 1, 64, n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 3)
        ctx = make_engine(w, weights, debug=True, max_inflight=n)
        try:
            for i in range(n):
                ap.april_debug_watch(ctx, i, 0, 1)
            ap.april_rollout_step(ctx, req_dicts([ai.Request(i, prompts[i % 3], 1) for i in range(n)]), n, n, 1)
            got = [ap.april_debug_logits(ctx, i, 0, vocab)[0] for i in range(n)]
        finally:
            ap.april_destroy(ctx)
        alone = alone or got
        for i, row in enumerate(got):
            assert np.max(np.abs(row - ref[i % 3])) <= 1e-4 and np.array_equal(row, alone[i % 3]), (n, i)


@pytest.mark.parametrize("d_ffn", [512, 600, 800])
def test_small_models_bits_do_not_depend_on_capacity_or_batch(d_ffn):
    """Layers of 1.0, 1.2 and 1.4 MiB (the last beyond the one-launch pass): the same rollouts in contexts of few and many slots, alone
    and among so many that a decode pass runs as separate launches."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, 128, 4, 4, 32, d_ffn, 300, dtype=ai.DTYPE_FP32)
    weights = ai.make_weights(shape, 11)
    rng = np.random.default_rng(d_ffn)
    gen = 5
    prompts = [rng.integers(0, 300, t, dtype=np.int32) for t in (1, 15, 40, 62, 70)]
    forced = rng.integers(0, 300, (5, gen), dtype=np.int32)
    dec = Decoder(shape, weights)
    first = None
    for n, slots in ((5, 5), (5, 256), (5, 257), (5, 321), (260, 260), (300, 330)):
        w = ai.Workload("fp32", shape, 1, 70, n, n, gen, 0.0, 0.1, gen, gen, ai.SAMPLER_GREEDY, 0, 1, 11)
        ctx = make_engine(w, weights, debug=True, max_inflight=slots)
        try:
            for i in range(5):
                ap.april_debug_watch(ctx, i, 0, gen)
            ap.april_rollout_step(ctx, req_dicts([ai.Request(i, prompts[i % 5], gen) for i in range(n)], {i: forced[i % 5] for i in range(n)}), n, n, gen)
            got = [[ap.april_debug_logits(ctx, i, g, 300)[0] for g in range(gen)] for i in range(5)]
        finally:
            ap.april_destroy(ctx)
        if first is None:
            first = got
            for i in range(5):
                ref = dec.forward_block(np.concatenate([prompts[i], forced[i][:-1]]), dec.new_cache())[-gen:]
                assert np.max(np.abs(np.array(got[i]) - ref)) <= 1e-4, i
        assert np.array_equal(np.array(first), np.array(got)), (n, slots)


def test_small_models_bits_do_not_depend_on_where_decode_turns_to_separate_launches():
    """16 heads: contexts up to 160 tokens decode in one launch, up to 480 where there are many rows, longer ones in separate launches,
    within a step.  Logits of positions around the turns: the same bits as prefilled there, alone, beside a longer rollout and among
    many short ones, and as the oracle's."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, 64, 16, 4, 32, 256, 200, dtype=ai.DTYPE_FP32)
    weights = ai.make_weights(shape, 2)
    text = np.random.default_rng(5).integers(0, 200, 560, dtype=np.int32)
    dec = Decoder(shape, weights)
    ref = dec.forward_block(text[:500], dec.new_cache())
    rows = {}
    for prompt, gen, others in ((150, 20, []), (150, 20, [300]), (150, 20, [5] * 140), (470, 20, [5] * 140), (157, 4, []), (158, 4, []),
                                (159, 4, []), (160, 4, []), (165, 4, []), (477, 4, []), (480, 4, [])):
        n = 1 + len(others)
        w = ai.Workload("fp32", shape, 1, 500, n, n, 24, 0.0, 0.1, 24, 24, ai.SAMPLER_GREEDY, 0, 1, 2)
        ctx = make_engine(w, weights, debug=True, max_inflight=n, max_ctx=560 if others else 32768)     # (a page list of every length in LDS)
        reqs = [ai.Request(i, text[:t], gen) for i, t in enumerate([prompt] + others)]
        try:
            ap.april_debug_watch(ctx, 0, 0, gen)
            ap.april_rollout_step(ctx, req_dicts(reqs, {r.request_id: text[len(r.tokens):len(r.tokens) + gen] for r in reqs}), n, n, gen)
            for g in range(gen):
                got, at = ap.april_debug_logits(ctx, 0, g, 200)[0], prompt + g - 1
                assert np.max(np.abs(got - ref[at])) <= 1e-4, (prompt, g)
                rows.setdefault(at, []).append(got)
        finally:
            ap.april_destroy(ctx)
    for at, got in rows.items():
        assert all(np.array_equal(got[0], x) for x in got[1:]), at


@pytest.mark.parametrize("vocab,d_model,temperature", [(1, 8, 1.0), (63, 40, 0.7), (512, 128, 1.0), (1030, 64, 1.3)])
def test_greedy_in_the_decode_pass_equals_the_sampler(vocab, d_model, temperature):
    """A greedy decode pass of a small fp32 model picks the token itself, a context that watches logits leaves that to the sampler's
    kernel: same tokens (ties included: the upper half of the vocabulary repeats the lower) and log-probabilities, bit for bit."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, d_model, 2, 1, 32, 36, vocab, dtype=ai.DTYPE_FP32)
    w = ai.Workload("greedy", shape, 1, 20, 6, 9, 30, 0.0, 0.1, 3, 30, ai.SAMPLER_GREEDY, 0, 1, 3)
    weights = ai.make_weights(shape, w.seed)
    weights["lm_head"][vocab - vocab // 2:] = weights["lm_head"][:vocab // 2]
    rng = np.random.default_rng(vocab)
    reqs = [dict(request_id=i, tokens=rng.integers(0, vocab, 1 + 2 * i, dtype=np.int32), forced_len=3 + 3 * i) for i in range(9)]
    seen = []
    for debug in (False, True):
        ctx = make_engine(w, weights, debug=debug, temperature=temperature, logprobs=True)
        try:
            res = ap.april_rollout_step(ctx, reqs, 6, 9, 30)
            ap.april_resume(ctx, res.buffer)
            res2 = ap.april_rollout_step(ctx, [], 3, 3, 30)
            seen.append((list(res.request_id) + list(res2.request_id), np.concatenate(list(res.tokens) + list(res2.tokens)),
                         np.concatenate(list(res.logprobs) + list(res2.logprobs))))
        finally:
            ap.april_destroy(ctx)
    assert seen[0][0] == seen[1][0] and np.array_equal(seen[0][1], seen[1][1]) and np.array_equal(seen[0][2], seen[1][2])
    assert np.isfinite(seen[0][2]).all() and seen[0][1].min() >= 0 and seen[0][1].max() < vocab
