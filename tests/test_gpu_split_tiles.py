"""Prefill products whose last round of 256 x 256 tiles goes as halves of 128 columns, and whose columns end in one of 128
(17 or 33 units of 128 columns, of 64 features): a prompt's logits keep the bits of a pass of few rows."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


# 75 prompts are 2550 rows (10 row tiles), 265 are 9010 (36): all tiles as halves, or those past the first 256
@pytest.mark.parametrize("d_model,d_ffn,n_q,n_kv,head_dim", [
    (2176, 1120, 15, 1, 128), (1056, 2112, 30, 2, 64), (416, 2080, 60, 4, 32), (128, 224, 2, 1, 32),
    (928, 256, 2, 1, 64),            # 29 column tiles: at 36 row tiles whole tiles of 256, whose last ends in the middle of a wavefront
    (896, 448, 5, 1, 128)])          # 7 units everywhere: the halves' last sixteen is partial, pieces of the odd column fill it
def test_halves_keep_the_bits(d_model, d_ffn, n_q, n_kv, head_dim):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, d_model, n_q, n_kv, head_dim, d_ffn, 512)
    weights = ai.make_weights(shape, 4)
    rng = np.random.default_rng(d_model)
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in (5, 33, 64)]
    alone = None
    for n in (3, 75, 265) + ((560,) if d_model == 128 else ()):        # 560: 19 040 rows in one pass
        w = ai.Workload("split", shape, 1, 64, n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 4)
        ctx = make_engine(w, weights, debug=True, max_inflight=n)
        try:
            for i in range(n):
                ap.april_debug_watch(ctx, i, 0, 1)
            ap.april_rollout_step(ctx, req_dicts([ai.Request(i, prompts[i % 3], 1) for i in range(n)]), n, n, 1)
            got = [ap.april_debug_logits(ctx, i, 0, shape.vocab)[0] for i in range(n)]
        finally:
            ap.april_destroy(ctx)
        alone = alone or got
        for i, row in enumerate(got):
            assert np.isfinite(row).all() and np.array_equal(row, alone[i % 3]), (n, i)
