"""Prefill passes of more than 16 384 rows, and prompts that take two passes: the second finds the workspaces of the first (residual
stream, packed rows of the last layer, staging block) and gives the bits that the same prompts have alone."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import have_gpu, make_engine, req_dicts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


def pass_rows(s):
    """Rows that april_init gives a pass (more slots than those rows, short contexts): 4 GiB of workspace, 16384 to 65536."""
    nq, moe = s.n_q_heads * s.head_dim, s.n_experts > 0
    row = 7 * s.d_model + 6 * nq + 2 * s.d_ffn
    if moe:
        row += 4 * s.n_experts + s.experts_per_tok * (2 * s.d_expert_ffn + 4 * s.d_model + 16)
    return max(16384, min((4 << 30) // row, 65536))


def prompt_kinds(limit, behind):
    """Prompts of 5, 33, 64 tokens in turn, then of 5 until no other fits into the first pass; `behind` more."""
    kinds, room, lengths = [], limit, (5, 33, 64)
    while room >= 64:
        kinds.append(len(kinds) % 3)
        room -= lengths[kinds[-1]]
    kinds += [0] * (room // 5)
    return kinds + [i % 3 for i in range(behind)]


# row bytes of 156 544 (8 x 16 heads of 128, 28 672 features) and 241 664 (8 of 32 experts, rows of 6144): passes of 27 436 and 17 772 rows.
# Last passes on both sides of the rule that takes the sampling rows alone past the last layer's keys and values (384 rows spared, of routed experts 8).
# None behind the first: one full pass; a wide layer of 4096, whose passes hold 65 536 rows, with 19 040.
DENSE = dict(n_layers=2, d_model=128, n_q_heads=128, n_kv_heads=8, head_dim=128, d_ffn=28672, vocab=512)
MOE = dict(n_layers=2, d_model=6144, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=0, vocab=512, n_experts=32, experts_per_tok=8, d_expert_ffn=64)
WIDE = dict(n_layers=2, d_model=4096, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ffn=512, vocab=512)


@pytest.mark.parametrize("shape,behind", [(DENSE, (0, 9, 40)), (MOE, (0, 1, 40)), (WIDE, (None,))], ids=["dense", "experts", "wide"])
def test_prompts_keep_their_bits_in_passes_of_any_size(shape, behind):
    import paper_2509_18521_amd as ap
    shape = ai.ModelShape(**shape)
    weights = ai.make_weights(shape, 6)
    rng = np.random.default_rng(shape.d_model)
    prompts = [rng.integers(0, shape.vocab, t, dtype=np.int32) for t in (5, 33, 64)]
    limit = pass_rows(shape)
    runs = [[0, 1, 2]] + [[i % 3 for i in range(560)] if b is None else prompt_kinds(limit, b) for b in behind]
    n_most = max(len(r) for r in runs)
    w = ai.Workload("passes", shape, 1, 64, n_most, n_most, 1, 0.0, 0.1, 1, 1, ai.SAMPLER_GREEDY, 0, 1, 6)
    ctx = make_engine(w, weights, debug=True, max_inflight=n_most)
    alone, first_id = None, 0
    try:
        for kinds in runs:
            n = len(kinds)
            ids = range(first_id, first_id + n)
            first_id += n
            watched = [i for i in range(n) if i < 6 or i % 37 == 0 or i >= n - 45]
            for i in watched:
                ap.april_debug_watch(ctx, ids[i], 0, 1)
            res = ap.april_rollout_step(ctx, req_dicts([ai.Request(ids[i], prompts[kinds[i]], 1) for i in range(n)]), n, n, 1)
            got = {i: ap.april_debug_logits(ctx, ids[i], 0, shape.vocab)[0] for i in watched}
            ap.april_buffer_free(ctx, res.buffer)
            alone = alone or got
            for i, row in got.items():
                assert np.isfinite(row).all() and np.array_equal(row, alone[kinds[i]]), (n, i, kinds[i])
    finally:
        ap.april_destroy(ctx)
