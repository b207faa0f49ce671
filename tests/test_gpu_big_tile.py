"""The 256 x 256 GEMM tile against the oracle where its stage ring is barely filled (1 to 5 stages of 32
values of k) and its row and column tiles end early: the gate/up projection and the LM head of 140
short prompts in one prefill pass (977 rows)."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts
from oracle.model import Decoder

pytestmark = pytest.mark.gpu
# bf16 operands: weights are exact on both sides, a dozen roundings of 2^-9 relative size in one layer
LOGIT_TOL = 1e-2                # max-abs relative to the logit scale max(1, max|l_ref|)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("d_model", [32, 64, 96, 128, 160])
def test_short_k_and_ragged_edges(d_model):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(1, d_model, 2, 1, 32, 4064, 1056)
    n, lengths = 140, [7, 6, 8, 7, 7]
    w = ai.Workload("big", shape, 1, 8, n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, d_model)
    weights = ai.make_weights(shape, w.seed)
    rng = np.random.default_rng(d_model)
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in lengths]
    reqs = [ai.Request(i, prompts[i % 5], 1) for i in range(n)]
    dec = Decoder(shape, weights)
    refs = [dec.forward_block(p, dec.new_cache())[-1] for p in prompts]
    ctx = make_engine(w, weights, debug=True)
    try:
        for i in range(n):
            ap.april_debug_watch(ctx, i, 0, 1)
        ap.april_rollout_step(ctx, req_dicts(reqs), n, n, 1)
        for i in range(n):
            got, _ = ap.april_debug_logits(ctx, i, 0, shape.vocab)
            ref = refs[i % 5]
            assert np.max(np.abs(got - ref)) <= LOGIT_TOL * max(1.0, np.max(np.abs(ref))), i
    finally:
        ap.april_destroy(ctx)
