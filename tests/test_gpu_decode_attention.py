"""Decode attention against the oracle where its tiles end: prompts around the page (16), tile (32), round of the
wavefronts (128), ring (256) and KV split boundaries, two decode iterations behind each; several head sizes, query
heads per KV head, and QKV split factors (by the model's width: 1, 2, 4 and 8 partials)."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts
from oracle.model import Decoder

pytestmark = pytest.mark.gpu

LENGTHS = [1, 14, 15, 16, 30, 31, 32, 62, 63, 95, 126, 127, 128, 159, 255, 257, 383, 511, 1022, 1023, 1024, 1100]
# bf16 operands: weights are exact on both sides, a dozen roundings of 2^-9 relative size in one layer
LOGIT_TOL = 1e-2                # max-abs relative to the logit scale max(1, max|l_ref|)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("head_dim,n_q,n_kv,d_model", [
    (32, 4, 4, 64), (32, 16, 1, 416), (64, 14, 2, 896), (64, 10, 2, 1664), (128, 4, 2, 64), (128, 16, 1, 416)])
def test_contexts_of_every_boundary_length(head_dim, n_q, n_kv, d_model):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(1, d_model, n_q, n_kv, head_dim, 64, 256)
    n, gen = len(LENGTHS), 3
    w = ai.Workload("lengths", shape, 1, max(LENGTHS), n, n, gen, 0.0, 0.1, gen, gen, ai.SAMPLER_GREEDY, 0, 1, 31)
    weights = ai.make_weights(shape, w.seed)
    rng = np.random.default_rng(head_dim + n_q)
    reqs = [ai.Request(i, rng.integers(0, shape.vocab, t, dtype=np.int32), gen) for i, t in enumerate(LENGTHS)]
    forced = {r.request_id: rng.integers(0, shape.vocab, gen, dtype=np.int32) for r in reqs}
    dec = Decoder(shape, weights)
    ctx = make_engine(w, weights, debug=True)
    try:
        for r in reqs:
            ap.april_debug_watch(ctx, r.request_id, 0, gen)
        ap.april_rollout_step(ctx, req_dicts(reqs, forced=forced), n, n, gen)
        for r in reqs:
            ref = dec.forward_block(np.concatenate([r.tokens, forced[r.request_id][:gen - 1]]), dec.new_cache())[-(gen - 1):]
            for i in range(1, gen):
                got, _ = ap.april_debug_logits(ctx, r.request_id, i, shape.vocab)
                assert np.max(np.abs(got - ref[i - 1])) <= LOGIT_TOL * max(1.0, np.max(np.abs(ref[i - 1]))), (len(r.tokens), i)
    finally:
        ap.april_destroy(ctx)
