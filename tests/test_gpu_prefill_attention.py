"""Query-tiled prefill attention against the oracle where its tiles end: prompts around the page (16), half
stage (32), stage (64) and page-id group (1024 tokens) boundaries in one call, every padding of the
query heads of a KV head, all head sizes."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts
from oracle.model import Decoder

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 255, 257, 1023, 1024, 1025, 1100]
# bf16 operands: weights are exact on both sides, a dozen roundings of 2^-9 relative size in one layer
LOGIT_TOL = 1e-2                # max-abs relative to the logit scale max(1, max|l_ref|)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("head_dim,n_q,n_kv", [(32, 4, 4), (32, 6, 2), (64, 14, 2), (64, 16, 1), (128, 4, 2), (128, 4, 1)])
def test_prompts_of_every_boundary_length(head_dim, n_q, n_kv):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(1, 64, n_q, n_kv, head_dim, 64, 256)
    n = len(LENGTHS)
    w = ai.Workload("lengths", shape, 1, max(LENGTHS), n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 29)
    weights = ai.make_weights(shape, w.seed)
    rng = np.random.default_rng(head_dim + n_q)
    reqs = [ai.Request(i, rng.integers(0, shape.vocab, t, dtype=np.int32), 1) for i, t in enumerate(LENGTHS)]
    dec = Decoder(shape, weights)
    ctx = make_engine(w, weights, debug=True)
    try:
        for r in reqs:
            ap.april_debug_watch(ctx, r.request_id, 0, 1)
        ap.april_rollout_step(ctx, req_dicts(reqs), n, n, 1)
        for r in reqs:
            ref = dec.forward_block(r.tokens, dec.new_cache())[-1]
            got, _ = ap.april_debug_logits(ctx, r.request_id, 0, shape.vocab)
            assert np.max(np.abs(got - ref)) <= LOGIT_TOL * max(1.0, np.max(np.abs(ref))), len(r.tokens)
    finally:
        ap.april_destroy(ctx)
