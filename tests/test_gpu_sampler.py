"""The device sampler alone, on identical logits rows and identical uniforms."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu
from oracle import sampler as osampler
from oracle.philox import uniform_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


def engine(vocab, sampler, top_k, temperature, seed, top_p=0.0):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(1, 32, 1, 1, 32, 32, vocab, dtype=ai.DTYPE_FP32)
    cfg = ap.make_cfg(shape, max_inflight=4, max_ctx=32, sampler=sampler, top_k=top_k, temperature=temperature,
                      seed=seed, top_p=top_p)
    return ap, ap.april_init(cfg, ap.pack_weights(shape, ai.make_weights(shape, 0)))


@pytest.mark.parametrize("vocab,top_k,temperature,quant", [
    (151936, 50, 1.0, None), (151936, 50, 0.75, None), (1000, 50, 1.0, 0.25), (37, 64, 1.0, 0.5),
    (512, 1, 1.0, None), (4096, 7, 0.5, 1.0), (8192, 50, 1.0, 0.5), (65536, 64, 1.0, 2.0), (4160, 50, 1.0, None)])
def test_topk_sampler_matches_oracle(vocab, top_k, temperature, quant):
    import torch
    rng = np.random.default_rng(vocab + top_k)
    n = 48
    logits = (3.0 * rng.standard_normal((n, vocab))).astype(np.float32)
    if quant:                                    # many exact ties, also across the k-th place
        logits = (np.round(logits / quant) * quant).astype(np.float32)
    seed = 1234567 + vocab
    ap, ctx = engine(vocab, ai.SAMPLER_TOPK, top_k, temperature, seed)
    try:
        rid = rng.integers(0, 2 ** 40, size=n)
        gi = rng.integers(0, 9000, size=n)
        d = torch.from_numpy(logits).cuda()
        got = ap.april_sample_rows(ctx, d.data_ptr(), n, rid, gi)
        exact = 0
        for r in range(n):
            u = uniform_for(seed, int(rid[r]), int(gi[r]))
            idx, p = osampler.top_k_probs(logits[r], top_k, float(np.float32(temperature)))
            if np.min(np.abs(np.cumsum(p)[:-1] - u)) < 1e-9 if len(p) > 1 else False:
                continue                         # u on a CDF boundary: either neighbour is right
            assert int(got[r]) == osampler.top_k_sample(logits[r], top_k, float(np.float32(temperature)), u), r
            exact += 1
        assert exact >= n - 2
    finally:
        ap.april_destroy(ctx)


@pytest.mark.parametrize("vocab,top_k,quant", [(4095, 64, None), (4097, 64, 0.5), (4097, 33, None), (4097, 32, 0.5),
                                               (6337, 50, 1.0), (6335, 50, 1.0), (8129, 64, 0.5)])
def test_topk_search_of_ragged_vocabularies(vocab, top_k, quant):
    """Either side of where the search turns from whole rows to groups (4096 logits, 2 k groups)."""
    test_topk_sampler_matches_oracle(vocab, top_k, 1.0, quant)


def test_greedy_sampler_lowest_index_on_ties():
    import torch
    rng = np.random.default_rng(5)
    n, vocab = 32, 3001
    logits = np.round(rng.standard_normal((n, vocab)) * 2).astype(np.float32)     # heavy ties at the max
    logits[3] = 0.0
    logits[4] = -0.0
    logits[5, 100] = np.float32(-0.0)
    ap, ctx = engine(vocab, ai.SAMPLER_GREEDY, 1, 1.0, 0)
    try:
        d = torch.from_numpy(logits).cuda()
        got = ap.april_sample_rows(ctx, d.data_ptr(), n, np.arange(n), np.zeros(n, dtype=np.int32))
        for r in range(n):
            assert int(got[r]) == osampler.greedy(logits[r]), r
    finally:
        ap.april_destroy(ctx)


@pytest.mark.parametrize("vocab,top_k,temperature,top_p,quant", [
    (151936, 64, 0.8, 0.7, None),      # the paper's appendix values: temperature 0.8, top_p 0.7
    (4096, 50, 1.0, 0.9, 0.5), (1000, 20, 0.5, 0.3, 0.25), (512, 64, 1.0, 0.999, None), (8192, 8, 1.3, 0.05, None)])
def test_nucleus_sampler_matches_oracle(vocab, top_k, temperature, top_p, quant):
    """top-k then top-p on the device against the oracle on identical logits and uniforms; rows
    where the uniform or top_p lies within 1e-9 of a step of the cumulative distribution are
    not compared (either neighbour is right there)."""
    import torch
    rng = np.random.default_rng(vocab + top_k + 7)
    n = 64
    logits = (3.0 * rng.standard_normal((n, vocab))).astype(np.float32)
    if quant:
        logits = (np.round(logits / quant) * quant).astype(np.float32)
    seed = 99 + vocab
    T, P = float(np.float32(temperature)), float(np.float32(top_p))
    ap, ctx = engine(vocab, ai.SAMPLER_TOPK, top_k, temperature, seed, top_p=top_p)
    try:
        rid = rng.integers(0, 2 ** 40, size=n)
        gi = rng.integers(0, 9000, size=n)
        d = torch.from_numpy(logits).cuda()
        got = ap.april_sample_rows(ctx, d.data_ptr(), n, rid, gi)
        exact, sizes = 0, set()
        for r in range(n):
            u = uniform_for(seed, int(rid[r]), int(gi[r]))
            _, pk = osampler.top_k_probs(logits[r], top_k, T)
            if np.min(np.abs(np.cumsum(pk) - P)) < 1e-9:
                continue
            idx, q = osampler.top_k_top_p_probs(logits[r], top_k, T, P)
            sizes.add(len(idx))
            if len(q) > 1 and np.min(np.abs(np.cumsum(q)[:-1] - u)) < 1e-9:
                continue
            assert int(got[r]) == osampler.top_k_top_p_sample(logits[r], top_k, T, P, u), r
            exact += 1
        assert exact >= n - 3 and (len(sizes) > 1 or top_p < 0.1)
    finally:
        ap.april_destroy(ctx)


@pytest.mark.parametrize("vocab,temperature", [(151936, 0.8), (3001, 1.0), (64, 0.5), (5000, 2.0)])
def test_categorical_sampler_and_logprobs_match_oracle(vocab, temperature):
    """Temperature sampling over the whole vocabulary (index-order inverse CDF) and the
    log-probability of the chosen token, on identical logits and uniforms."""
    import torch
    rng = np.random.default_rng(vocab)
    n = 40
    logits = (2.5 * rng.standard_normal((n, vocab))).astype(np.float32)
    logits[0] = 0.0                                        # uniform row: log-probability -log V
    seed = 5 + vocab
    T = float(np.float32(temperature))
    ap, ctx = engine(vocab, ai.SAMPLER_CATEGORICAL, 1, temperature, seed)
    try:
        rid = rng.integers(0, 2 ** 40, size=n)
        gi = rng.integers(0, 9000, size=n)
        d = torch.from_numpy(logits).cuda()
        got, lp = ap.april_sample_rows_logprobs(ctx, d.data_ptr(), n, rid, gi)
        assert np.array_equal(got, ap.april_sample_rows(ctx, d.data_ptr(), n, rid, gi))
        exact = 0
        for r in range(n):
            u = uniform_for(seed, int(rid[r]), int(gi[r]))
            z = logits[r].astype(np.float64) / T
            p = np.exp(z - z.max()); p /= p.sum()
            assert abs(float(lp[r]) - osampler.token_logprob(logits[r], T, int(got[r]))) < 2e-5, r
            if np.min(np.abs(np.cumsum(p) - u)) < 1e-9:
                continue
            assert int(got[r]) == osampler.categorical_sample(logits[r], T, u), r
            exact += 1
        assert exact >= n - 2
        assert abs(float(lp[0]) + np.log(vocab)) < 2e-5
    finally:
        ap.april_destroy(ctx)


def test_logprobs_of_greedy_and_topk_choices():
    import torch
    rng = np.random.default_rng(77)
    n, vocab = 24, 4160
    logits = (3.0 * rng.standard_normal((n, vocab))).astype(np.float32)
    for sampler, top_k, temperature in ((ai.SAMPLER_GREEDY, 1, 1.0), (ai.SAMPLER_TOPK, 50, 0.8)):
        T = float(np.float32(temperature))
        ap, ctx = engine(vocab, sampler, top_k, temperature, 3)
        try:
            d = torch.from_numpy(logits).cuda()
            got, lp = ap.april_sample_rows_logprobs(ctx, d.data_ptr(), n, np.arange(n), np.arange(n, dtype=np.int32))
            for r in range(n):
                assert abs(float(lp[r]) - osampler.token_logprob(logits[r], T, int(got[r]))) < 2e-5
        finally:
            ap.april_destroy(ctx)


@pytest.mark.parametrize("n_groups,top_k", [(64, 64), (65, 50), (1025, 1), (4096, 50), (4097, 50)])
@pytest.mark.parametrize("sampler", [ai.SAMPLER_GREEDY, ai.SAMPLER_TOPK, ai.SAMPLER_CATEGORICAL])
def test_records_of_every_register_count(sampler, n_groups, top_k):
    """Vocabularies of one group per lane, one and several groups per thread, and more than the records kernel keeps in
    registers (4096 groups); ties, masked logits and all of the mass in one place, among ordinary rows."""
    import torch
    vocab, T, seed = 64 * n_groups, 0.7, 9
    rng = np.random.default_rng([n_groups, top_k, sampler])
    logits = rng.standard_normal((5, vocab)).astype(np.float32)
    logits[1] = np.round(logits[1] * 4) / 4                       # ties, also between groups
    logits[2, rng.random(vocab) < 0.97] = -np.inf                 # most of the row masked
    logits[3, vocab // 3] = 40.0                                  # one logit holds the mass
    logits[4, :] = np.finfo(np.float32).min
    logits[4, 7::1999] = 0.5
    ids, idx = np.arange(5, dtype=np.int64) + 3, np.array([0, 1, 2, 3, 4], dtype=np.int32)
    ap, ctx = engine(vocab, sampler, top_k, T, seed)
    try:
        dev = torch.from_numpy(logits).cuda()
        tok, lp = ap.april_sample_rows_logprobs(ctx, dev.data_ptr(), 5, ids, idx)
        alone = ap.april_sample_rows_noalloc(ctx, dev.data_ptr(), 5, ids, idx)
    finally:
        ap.april_destroy(ctx)
    assert np.array_equal(tok, alone)
    for r in range(5):
        z = logits[r].astype(np.float64) / T
        logp = z - z.max() - np.log(np.exp(z - z.max()).sum())
        # fp32 results and differences to the maximum
        assert abs(lp[r] - logp[tok[r]]) <= 2e-6 * max(1.0, abs(logp[tok[r]])), (r, lp[r], logp[tok[r]])
        u = uniform_for(seed, int(ids[r]), int(idx[r]))
        if sampler == ai.SAMPLER_GREEDY or (sampler == ai.SAMPLER_TOPK and top_k <= 1):
            assert tok[r] == int(np.argmax(logits[r])), r
            continue
        order = np.arange(vocab) if sampler == ai.SAMPLER_CATEGORICAL else np.lexsort((np.arange(vocab), -z))[:top_k]
        p = np.exp(z[order] - z.max())
        c = np.cumsum(p) / p.sum()
        if np.min(np.abs(c - u)) > 1e-9:                          # not on a step of the distribution
            assert tok[r] == order[np.argmax(c > u)], r


@pytest.mark.parametrize("n_groups,ragged,top_k", [(1, 0, 1), (64, 0, 64), (65, 0, 50), (65, 31, 20), (1025, 0, 50), (1025, 31, 50),
                                                   (4096, 0, 64), (4097, 0, 50), (4097, 31, 50)])
@pytest.mark.parametrize("sampler", [ai.SAMPLER_GREEDY, ai.SAMPLER_TOPK, ai.SAMPLER_CATEGORICAL])
def test_rows_of_nan_give_tokens_of_the_vocabulary(sampler, n_groups, ragged, top_k):
    """NaN of either sign in the whole row, and in all of it but a few logits (fewer than k groups): a NaN with the sign set
    comes below -inf in the order of the searches, any other above +inf.  A distribution without a sum gives its last token.
    A row of signalling NaN: any token."""
    import torch
    vocab, T = 64 * n_groups - ragged, float(np.float32(0.7))
    k = min(top_k, vocab)
    neg, pos = np.uint32(0xffc00000).view(np.float32), np.uint32(0x7fc00000).view(np.float32)
    logits = np.full((6, vocab), neg, dtype=np.float32)
    logits[1] = pos
    few = np.unique(np.array([vocab // 3, vocab // 2, vocab - 1]))
    logits[2, few] = np.arange(len(few), dtype=np.float32) - 1.5
    logits[3, few] = -np.inf
    logits[4] = np.random.default_rng(n_groups).standard_normal(vocab).astype(np.float32)
    logits[4, :vocab // 2] = neg
    logits.view(np.uint32)[5] = 0x7f800001
    ids, idx = np.arange(6, dtype=np.int64) + 3, np.arange(6, dtype=np.int32)
    ap, ctx = engine(vocab, sampler, top_k, T, 9)
    try:
        dev = torch.from_numpy(logits).cuda()
        tok, _ = ap.april_sample_rows_logprobs(ctx, dev.data_ptr(), 6, ids, idx)
        plain = ap.april_sample_rows(ctx, dev.data_ptr(), 6, ids, idx)
        alone = ap.april_sample_rows_noalloc(ctx, dev.data_ptr(), 6, ids, idx)
    finally:
        ap.april_destroy(ctx)
    assert np.array_equal(tok, plain) and np.array_equal(tok, alone)
    assert tok.min() >= 0 and tok.max() < vocab
    if sampler == ai.SAMPLER_CATEGORICAL:
        assert all(t == vocab - 1 for t in tok)
        return
    bits = logits.view(np.uint32)
    keys = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000))
    for r in range(5):
        order = np.lexsort((np.arange(vocab), -keys[r].astype(np.int64)))[:k]
        if sampler == ai.SAMPLER_GREEDY or top_k <= 1:
            # (a short last group counts as if it were filled up with -inf, which comes above a row of such NaN)
            assert tok[r] == order[0] or (r == 0 and ragged and tok[r] == vocab // 64 * 64), r
        elif np.isnan(logits[r, order]).any() or np.isinf(logits[r, order[0]]):
            assert tok[r] == order[k - 1], r
        else:
            p = np.exp((logits[r, order].astype(np.float64) - logits[r, order[0]]) / T)
            c, u = np.cumsum(p) / p.sum(), uniform_for(9, int(ids[r]), int(idx[r]))
            assert np.min(np.abs(c - u)) <= 1e-9 or tok[r] == order[np.argmax(c > u)], r


@pytest.mark.parametrize("vocab,top_k", [(4032, 64), (4095, 50)])
def test_whole_row_searches_make_no_group_records(vocab, top_k):
    """Top-k searches that read whole rows (fewer than k groups; a short row) leave group records alone: no pass over the logits
    for them, so no workspace either (8192 rows of them would take 2 MiB, with sums 6).  Same tokens and log-probabilities."""
    import torch
    n, T, seed = 8192, float(np.float32(0.8)), 3
    logits = 2.0 * torch.randn(n, vocab, generator=torch.Generator("cuda").manual_seed(vocab), device="cuda")
    ids, idx = np.arange(n, dtype=np.int64), np.zeros(n, dtype=np.int32)
    ap, ctx = engine(vocab, ai.SAMPLER_TOPK, top_k, T, seed)
    try:
        ap.april_sample_rows_logprobs(ctx, logits.data_ptr(), 1, ids[:1], idx[:1])      # (whatever the first launch allocates)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        tok, lp = ap.april_sample_rows_logprobs(ctx, logits.data_ptr(), n, ids, idx)
        plain = ap.april_sample_rows(ctx, logits.data_ptr(), n, ids, idx)
        assert free - torch.cuda.mem_get_info()[0] < 1 << 20
    finally:
        ap.april_destroy(ctx)
    assert np.array_equal(tok, plain)
    for r in range(0, n, 331):
        row = logits[r].cpu().numpy()
        assert abs(float(lp[r]) - osampler.token_logprob(row, T, int(tok[r]))) < 2e-5
        _, p = osampler.top_k_probs(row, top_k, T)
        u = uniform_for(seed, int(ids[r]), 0)
        assert np.min(np.abs(np.cumsum(p)[:-1] - u)) < 1e-9 or int(tok[r]) == osampler.top_k_sample(row, top_k, T, u), r


@pytest.mark.parametrize("n_groups", [4096, 4097])
@pytest.mark.parametrize("top_k", [50, 64])
def test_topk_lists_that_overflow_fall_back_to_the_whole_row(n_groups, top_k):
    """More groups at the bound than the list of groups holds (1024: a constant row, a row of two values), and more candidates in
    few groups than the list of candidates holds (2048: 40 and 100 groups full of the maximum), among ordinary rows."""
    import torch
    vocab, T, seed = 64 * n_groups, float(np.float32(0.8)), 21
    rng = np.random.default_rng([n_groups, top_k])
    logits = rng.standard_normal((6, vocab)).astype(np.float32)
    logits[0] = 0.25
    logits[1] = np.where(rng.random(vocab) < 0.5, 1.0, -1.0)
    for r, full in ((2, 40), (3, 100)):
        for g in rng.choice(n_groups, full, replace=False):
            logits[r, 64 * g:64 * g + 64] = 6.0
    logits[4] = 0.25
    logits[4, -1] = 9.0                                           # the maximum in the last group, ties behind it
    ids, idx = np.arange(6, dtype=np.int64) + 40, np.arange(6, dtype=np.int32)
    ap, ctx = engine(vocab, ai.SAMPLER_TOPK, top_k, T, seed)
    try:
        dev = torch.from_numpy(logits).cuda()
        tok, lp = ap.april_sample_rows_logprobs(ctx, dev.data_ptr(), 6, ids, idx)
        alone = ap.april_sample_rows_noalloc(ctx, dev.data_ptr(), 6, ids, idx)
    finally:
        ap.april_destroy(ctx)
    assert np.array_equal(tok, alone)
    for r in range(6):
        _, p = osampler.top_k_probs(logits[r], top_k, T)
        u = uniform_for(seed, int(ids[r]), int(idx[r]))
        assert np.min(np.abs(np.cumsum(p)[:-1] - u)) < 1e-9 or int(tok[r]) == osampler.top_k_sample(logits[r], top_k, T, u), r
        assert abs(float(lp[r]) - osampler.token_logprob(logits[r], T, int(tok[r]))) < 2e-5, r
