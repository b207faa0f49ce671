"""Records of 64-logit groups (maximum, its column, sum of exponentials): the sampler entry points on
logits in memory and the LM head epilogue, where the vocabulary, the row count or the values end a
group, a wavefront or a part of the call early.

Bounds on log-probabilities: the fp32 result is at most 20 in size (2^-24 relative: 1e-6), the fp32
difference from the maximum adds as much, and fp32 exponentials (2^-21 relative at these arguments)
enter a sum: 1e-5 covers them."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import assert_schedule_equal, have_gpu, make_engine, run_gpu
from oracle import sampler as osampler
from oracle.philox import uniform_for

pytestmark = pytest.mark.gpu
LP_TOL = 1e-5


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


def ap():
    import paper_2509_18521_amd
    return paper_2509_18521_amd


def sampler_engine(vocab, sampler, top_k=1, temperature=1.0, seed=11):
    shape = ai.ModelShape(1, 32, 1, 1, 32, 32, vocab, dtype=ai.DTYPE_FP32)
    cfg = ap().make_cfg(shape, max_inflight=4, max_ctx=32, sampler=sampler, top_k=top_k, temperature=temperature, seed=seed)
    return ap().april_init(cfg, ap().pack_weights(shape, ai.make_weights(shape, 0)))


@pytest.mark.parametrize("vocab", [1, 63, 65, 1023, 4097, 50257])
@pytest.mark.parametrize("sampler", [ai.SAMPLER_GREEDY, ai.SAMPLER_TOPK, ai.SAMPLER_CATEGORICAL])
def test_sampling_rows_of_ragged_vocabularies(vocab, sampler):
    import torch
    rng = np.random.default_rng(vocab)
    n, seed, T = 9, 11, float(np.float32(0.8))
    logits = (2.5 * rng.standard_normal((n, vocab))).astype(np.float32)
    logits[1, : vocab // 2] = -np.inf                     # masked ranges: whole groups of -inf, and the first columns
    if vocab > 64:
        logits[2, 64:] = -np.inf
        logits[3, :64] = np.finfo(np.float32).min
    ctx = sampler_engine(vocab, sampler, 20, 0.8, seed)
    try:
        d = torch.from_numpy(logits).cuda()
        ids, idx = np.arange(n, dtype=np.int64) + 2 ** 33, np.arange(n, dtype=np.int32) * 7
        got, lp = ap().april_sample_rows_logprobs(ctx, d.data_ptr(), n, ids, idx)
        assert np.array_equal(got, ap().april_sample_rows_noalloc(ctx, d.data_ptr(), n, ids, idx))
        # rows that start at an odd multiple of 4 bytes
        shifted = torch.empty(n * vocab + 1, device="cuda")
        shifted[1:] = d.reshape(-1)
        assert np.array_equal(got, ap().april_sample_rows(ctx, shifted.data_ptr() + 4, n, ids, idx))
        for r in range(n):
            z = logits[r].astype(np.float64) / T
            u = uniform_for(seed, int(ids[r]), int(idx[r]))
            with np.errstate(invalid="ignore"):
                if sampler == ai.SAMPLER_GREEDY:
                    want = osampler.greedy(logits[r])
                elif sampler == ai.SAMPLER_TOPK:
                    want = osampler.top_k_sample(logits[r], 20, T, u)
                else:
                    want = osampler.categorical_sample(logits[r], T, u)
            assert int(got[r]) == want, r
            assert abs(float(lp[r]) - osampler.token_logprob(logits[r], T, int(got[r]))) <= LP_TOL, r
        assert np.isfinite(z).all()
    finally:
        ap().april_destroy(ctx)


def test_rows_beyond_one_part_of_the_workspace():
    """2 500 rows of 151 936 logits exceed the workspace the call keeps: it runs in parts."""
    import torch
    n, vocab = 2500, 151936
    d = torch.randn((n, vocab), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    ctx = sampler_engine(vocab, ai.SAMPLER_CATEGORICAL, 1, 0.8)
    try:
        ids, idx = np.arange(n, dtype=np.int64), np.arange(n, dtype=np.int32) % 5
        got, lp = ap().april_sample_rows_logprobs(ctx, d.data_ptr(), n, ids, idx)
        for r0 in (0, 2300, n - 3):
            part, lpp = ap().april_sample_rows_logprobs(ctx, d[r0:].data_ptr(), 3, ids[r0:r0 + 3], idx[r0:r0 + 3])
            assert np.array_equal(part, got[r0:r0 + 3]) and np.array_equal(lpp, lp[r0:r0 + 3])
    finally:
        ap().april_destroy(ctx)


@pytest.mark.parametrize("vocab", [1056, 1024, 32])
@pytest.mark.parametrize("n_target,n_over", [(13, 18), (110, 150)])
def test_logprobs_without_logits(monkeypatch, vocab, n_target, n_over):
    """Greedy rollouts with log-probabilities: from the LM head's records alone (both its kernels, up
    to and beyond 128 rows; odd numbers of 32-column tiles) the same tokens and the same bits as
    when the logits are written too, and what the logits themselves give."""
    shape = ai.ModelShape(1, 128, 4, 2, 32, 256, vocab)
    w = ai.Workload("records", shape, 8, 9, n_target, n_over, 7, 1.6, 0.3, 3, 7, ai.SAMPLER_GREEDY, 0, 2, 13)
    weights = ai.make_weights(shape, w.seed)
    reqs = ai.make_requests(w, ai.requests_needed(w))
    runs = []
    for flag in ("1", "0"):
        monkeypatch.setenv("APRIL_WRITE_LOGITS", flag)
        ctx = make_engine(w, weights, logprobs=True, temperature=0.9)
        try:
            runs.append(run_gpu(ctx, reqs, w.n_target, w.n_overprovision, w.max_new, w.steps))
        finally:
            ap().april_destroy(ctx)
    a, b = runs
    assert_schedule_equal(b, a)
    assert [g["tokens"] for g in a] == [g["tokens"] for g in b]
    assert [g["logprobs"] for g in a] == [g["logprobs"] for g in b]
    ctx = make_engine(w, weights, logprobs=True, temperature=0.9, debug=True)
    try:
        rid, toks, lps = b[0]["ids"][0], b[0]["tokens"][0], b[0]["logprobs"][0]
        ap().april_debug_watch(ctx, rid, 0, len(toks))
        run_gpu(ctx, reqs, w.n_target, w.n_overprovision, w.max_new, 1)
        for g, t in enumerate(toks):
            row, _ = ap().april_debug_logits(ctx, rid, g, vocab)
            assert abs(lps[g] - osampler.token_logprob(row, float(np.float32(0.9)), t)) <= LP_TOL
    finally:
        ap().april_destroy(ctx)


@pytest.mark.parametrize("vocab", [1024, 1056, 6176])
@pytest.mark.parametrize("n_target,n_over", [(13, 18), (110, 150)])
@pytest.mark.parametrize("sampler,top_k", [(ai.SAMPLER_CATEGORICAL, 0), (ai.SAMPLER_TOPK, 5), (ai.SAMPLER_TOPK, 40)])
def test_sampled_bf16_rollouts(vocab, n_target, n_over, sampler, top_k):
    """Sampling modes of bf16 rollouts, in iterations whose row count falls (records of rows that are gone stay behind in
    the arrays): every token and log-probability is the oracle sampler's on the logits row it was drawn from."""
    shape = ai.ModelShape(1, 128, 4, 2, 32, 256, vocab)
    w = ai.Workload("sampled", shape, 8, 9, n_target, n_over, 7, 1.4, 0.5, 1, 7, ai.SAMPLER_GREEDY, top_k, 2, 13)
    weights = ai.make_weights(shape, w.seed)
    reqs = ai.make_requests(w, ai.requests_needed(w))
    T, steps = float(np.float32(0.8)), []
    for debug in (True, False):
        ctx = make_engine(w, weights, logprobs=True, temperature=0.8, debug=debug, sampler=sampler)
        try:
            for r in reqs if debug else []:
                ap().april_debug_watch(ctx, r.request_id, 0, w.max_new)
            steps.append(run_gpu(ctx, reqs, w.n_target, w.n_overprovision, w.max_new, w.steps))
            for g in steps[0] if debug else []:
                assert g["iters"] > 1 and g["sum_live"] < g["iters"] * n_over
                for rid, toks, lps in zip(g["ids"], g["tokens"], g["logprobs"]):
                    for i, t in enumerate(toks):
                        row, chosen = ap().april_debug_logits(ctx, rid, i, vocab)
                        u = uniform_for(w.seed, rid, i)
                        want = (osampler.categorical_sample(row, T, u) if sampler == ai.SAMPLER_CATEGORICAL
                                else osampler.top_k_sample(row, top_k, T, u))
                        assert t == chosen == want, (rid, i)
                        assert abs(lps[i] - osampler.token_logprob(row, T, t)) <= LP_TOL, (rid, i)
        finally:
            ap().april_destroy(ctx)
    assert [g["tokens"] for g in steps[0]] == [g["tokens"] for g in steps[1]]
    assert [g["logprobs"] for g in steps[0]] == [g["logprobs"] for g in steps[1]]
