"""The rows of a prefill pass pick its GEMM tiles (64 x 32, 128 x 64, 256 x 128, 256 x 256): a prompt's logits
keep their bits alone and among however many others, at inner dimensions that fill the stage rings
only partly."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("d_model,d_ffn,head_dim,n_q", [(64, 96, 32, 1), (160, 4128, 64, 3), (1024, 2080, 128, 4)])
def test_prompt_bits_do_not_depend_on_the_pass(d_model, d_ffn, head_dim, n_q):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, d_model, n_q, 1, head_dim, d_ffn, 512)
    weights = ai.make_weights(shape, 3)
    rng = np.random.default_rng(d_model)
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in (5, 33, 64)]
    alone = None
    for n in (3, 6, 12, 24, 48, 120, 200):
        w = ai.Workload("tiles", shape, 1, 64, n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 3)
        reqs = [ai.Request(i, prompts[i % 3], 1) for i in range(n)]
        ctx = make_engine(w, weights, debug=True, max_inflight=n)
        try:
            for i in range(n):
                ap.april_debug_watch(ctx, i, 0, 1)
            ap.april_rollout_step(ctx, req_dicts(reqs), n, n, 1)
            got = [ap.april_debug_logits(ctx, i, 0, shape.vocab)[0] for i in range(n)]
        finally:
            ap.april_destroy(ctx)
        alone = alone or got
        for i, row in enumerate(got):
            assert np.isfinite(row).all() and np.array_equal(row, alone[i % 3]), (n, i)


@pytest.mark.parametrize("n_q,n_kv,head_dim", [(64, 32, 32), (64, 16, 64), (32, 8, 128), (3, 1, 128), (5, 1, 32)])
def test_qkv_tiles_give_the_same_queries_keys_and_values(n_q, n_kv, head_dim):
    """The rows of a pass pick the QKV projection's tile (64 x 64, 128 x 128, 256 x 128, 256 x 256: all four for the wide
    shapes, and ends inside a tile); heads are whole or split over wavefronts by it.  Same sums, same rotation: same bits."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, 160, n_q, n_kv, head_dim, 256, 512)
    weights = ai.make_weights(shape, 9)
    rng = np.random.default_rng(head_dim)
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in (5, 33, 64)]
    alone = None
    for n in (130, 3, 9, 30, 64):
        w = ai.Workload("qkv", shape, 1, 64, n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 9)
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


@pytest.mark.parametrize("experts", [32, 64, 160])
def test_expert_groups_take_every_row_once(experts):
    """Routed experts: the number of row groups picks how many of them an XCD takes in a row (0 below 64
    groups); neither that nor a ragged last round may leave out or mix up a row."""
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(2, 320, 5, 1, 64, 0, 512, n_experts=experts, experts_per_tok=4, d_expert_ffn=160)
    weights = ai.make_weights(shape, 5)
    rng = np.random.default_rng(experts)
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in (5, 33, 64)]
    alone = None
    for n in (3, 24, 60, 200):
        w = ai.Workload("experts", shape, 1, 64, n, n, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 5)
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
