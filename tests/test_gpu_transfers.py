"""Token and log-probability transfers of a step through the pinned buffer, which holds what all slots hold up to 2^18
ints: one rollout, the most a context admits (one piece per rollout and array), and more ints than the buffer, where
pieces are split as it fills.  Imported rollouts deliver what they brought."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,length", [(1, 1), (3, 700), (2048, 3), (40, 7000)])
def test_imported_rollouts_come_back_whole(n, length):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(1, 32, 1, 1, 32, 32, 64)
    w = ai.Workload("xfer", shape, 1, 1, n, n, 2, 0.0, 0.1, 2, 2, ai.SAMPLER_GREEDY, 0, 1, 3)
    rng = np.random.default_rng(n)
    lengths = [length - (i % 5 if length > 10 else 0) for i in range(n)]
    parts = [dict(request_id=i, prompt=rng.integers(0, 64, 1 + i % 3), generated=rng.integers(0, 64, t), limit=t + 2,
                  logprobs=-rng.random(t).astype(np.float32)) for i, t in enumerate(lengths)]
    ctx = make_engine(w, ai.make_weights(shape, 1), logprobs=True, max_inflight=n, max_ctx=length + 16)
    try:
        ap.april_resume(ctx, ap.april_buffer_import(ctx, parts))
        res = ap.april_rollout_step(ctx, [], n, n, length + 2)
        assert res.request_id == list(range(n))
        for p, t, toks, lps in zip(parts, lengths, res.tokens, res.logprobs):
            assert len(toks) == t + 2 and np.array_equal(toks[:t], p["generated"])
            assert np.array_equal(lps[:t], p["logprobs"]) and np.all(lps[t:] < 0)
    finally:
        ap.april_destroy(ctx)
