"""Prefill passes of enough rows take only the sampling rows past the last layer's keys and values: a prompt's logits and those of the
tokens decoded behind it keep the bits of a pass that takes every row (the prompt alone, below the row count of that rule)."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


@pytest.mark.parametrize("layers,d_model,n_q,n_kv,head_dim,experts", [
    (1, 160, 5, 1, 32, 0), (3, 192, 6, 2, 64, 0), (2, 2048, 4, 2, 128, 0), (1, 192, 4, 2, 64, 32), (2, 320, 3, 1, 128, 32)])
def test_sampling_rows_alone_behind_the_last_keys(layers, d_model, n_q, n_kv, head_dim, experts):
    import paper_2509_18521_amd as ap
    kw = dict(n_experts=experts, experts_per_tok=4, d_expert_ffn=96) if experts else {}
    shape = ai.ModelShape(layers, d_model, n_q, n_kv, head_dim, 0 if experts else 224, 512, **kw)
    weights = ai.make_weights(shape, 11)
    rng = np.random.default_rng(d_model + layers)
    # (5000 rows spared are enough for every width)
    lengths = [1, 2, 7] if experts else [1, 2, 31, 77]
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in lengths + [5000]]
    w = ai.Workload("last", shape, 1, 5010, 8, 8, 3, 0.0, 0.1, 3, 1, ai.SAMPLER_GREEDY, 0, 1, 11)
    ctx = make_engine(w, weights, debug=True, max_inflight=8)

    def logits(ids, which):
        for i in ids:
            ap.april_debug_watch(ctx, i, 0, 3)
        reqs = [ai.Request(i, prompts[p], 3) for i, p in zip(ids, which)]
        ap.april_buffer_free(ctx, ap.april_rollout_step(ctx, req_dicts(reqs), len(ids), len(ids), 3).buffer)
        return [[ap.april_debug_logits(ctx, i, g, shape.vocab)[0] for g in range(3)] for i in ids]

    try:
        together = logits(range(len(prompts)), range(len(prompts)))
        for p in range(len(lengths)):
            alone = logits([100 + p], [p])[0]
            assert np.isfinite(alone[0]).all() and all(np.array_equal(a, b) for a, b in zip(alone, together[p])), lengths[p]
    finally:
        ap.april_destroy(ctx)


@pytest.mark.parametrize("d_model,n_q,n_kv,head_dim,experts", [(160, 5, 1, 32, 0), (192, 6, 2, 64, 0), (2048, 4, 2, 128, 0), (320, 3, 1, 128, 32)])
def test_sampling_rows_alone_equal_a_pass_of_all_rows(d_model, n_q, n_kv, head_dim, experts):
    """A further layer whose output and down projections are zero changes no bit of the residual stream, and makes the layer before it one that takes
    every row.  Prompts up to 1100 tokens (more than the 64 pages that an attention workgroup knows at a time), with the tokens decoded behind them."""
    import paper_2509_18521_amd as ap
    kw = dict(n_experts=experts, experts_per_tok=4, d_expert_ffn=96) if experts else {}
    shapes = [ai.ModelShape(layers, d_model, n_q, n_kv, head_dim, 0 if experts else 224, 512, **kw) for layers in (2, 3)]
    weights = ai.make_weights(shapes[1], 13)
    for name in ("wo.2", "e_down.2" if experts else "w_down.2"):
        weights[name] = np.zeros_like(weights[name])
    rng = np.random.default_rng(d_model)
    prompts = [rng.integers(0, shapes[0].vocab, t, dtype=np.int32) for t in (1, 31, 420, 1023, 1024, 1025, 1100)]
    w = ai.Workload("last", shapes[0], 1, 1110, 8, 8, 3, 0.0, 0.1, 3, 1, ai.SAMPLER_GREEDY, 0, 1, 13)
    seen = []
    for shape in shapes:
        ctx = make_engine(ai.reduced(w, n_layers=shape.n_layers), {n: t for n, t in weights.items() if shape.n_layers == 3 or not n.endswith(".2")}, debug=True,
                          max_inflight=8)
        try:
            for i in range(len(prompts)):
                ap.april_debug_watch(ctx, i, 0, 3)
            ap.april_rollout_step(ctx, req_dicts([ai.Request(i, p, 3) for i, p in enumerate(prompts)]), len(prompts), len(prompts), 3)
            seen.append([ap.april_debug_logits(ctx, i, g, shape.vocab)[0] for i in range(len(prompts)) for g in range(3)])
        finally:
            ap.april_destroy(ctx)
    for at, (cut, whole) in enumerate(zip(*seen)):
        assert np.isfinite(cut).all() and np.array_equal(cut, whole), (len(prompts[at // 3]), at % 3)
