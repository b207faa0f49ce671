"""GPU parity for routed experts (router soft-max, top-k, grouped expert GEMMs)."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import assert_schedule_equal, class_forced_tokens, have_gpu, make_engine, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

BF16_LOGIT_TOL = 2e-2
ROUTE_MARGIN = 3e-2      # relative gap between the last kept and first dropped router probability


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


def ap():
    import paper_2509_18521_amd
    return paper_2509_18521_amd


def moe_parity(w, steps, n_requests, min_rows):
    """Teacher-forced logits parity.  The routing decision is an integer decided by floating
    point: positions where the oracle's own decision (at any layer) is within ROUTE_MARGIN of
    a tie are not compared.  Above the first layer a flipped decision also perturbs that
    position's K/V for later positions; that effect is diluted by attention and stays inside
    the tolerance, so later positions are still compared."""
    weights = ai.make_weights(w.shape, w.seed)
    reqs = ai.make_requests(w, n_requests)
    want, eng = run_oracle(w, weights, reqs, w.n_target, w.n_overprovision, w.max_new, steps, keep_logits=True)
    ref_tokens = {}
    for o in want:
        ref_tokens.update(dict(zip(o["ids"], o["tokens"])))
    ref_tokens.update(want[-1]["buffer_tokens"])
    # per-rollout routing margins from an oracle replay of each rollout alone
    from oracle.model import Decoder
    dec = Decoder(w.shape, weights)
    first_bad = {}
    for rid, toks in ref_tokens.items():
        dec.route_margins = []
        seq = list(reqs[rid].tokens) + list(toks[:-1])
        dec.forward_block(seq, dec.new_cache())
        P = len(reqs[rid].tokens)
        # generated token i is predicted from position P - 1 + i; near-ties inside the prompt
        # are not filtered (their effect on later positions is diluted by attention)
        bad = {p - (P - 1) for p, l, m in dec.route_margins if m < ROUTE_MARGIN and p >= P - 1}
        first_bad[rid] = bad
    ctx = make_engine(w, weights, debug=True)
    try:
        for rid in ref_tokens:
            ap().april_debug_watch(ctx, rid, 0, w.max_new)
        got = run_gpu(ctx, reqs, w.n_target, w.n_overprovision, w.max_new, steps, forced=ref_tokens)
        assert_schedule_equal(got, want)
        worst, rows, skipped = 0.0, 0, 0
        for rid, toks in ref_tokens.items():
            for i in range(len(toks)):
                fb = first_bad[rid]
                if (isinstance(fb, set) and i in fb) or (isinstance(fb, int) and i >= fb):
                    skipped += 1
                    continue
                lg, sampled = ap().april_debug_logits(ctx, rid, i, w.shape.vocab)
                ref = eng.logits[(rid, i)]
                scale = max(1.0, float(np.max(np.abs(ref))))
                worst = max(worst, float(np.max(np.abs(lg - ref))) / scale)
                rows += 1
        print(f"moe parity: rows={rows} skipped={skipped} worst={worst:.4g}")
        share = f"skipped {skipped} of {rows + skipped} positions ({skipped / max(rows + skipped, 1):.0%}) as routing near-ties"
        assert rows >= min_rows, f"compared only {rows} rows; {share}"
        assert worst <= BF16_LOGIT_TOL, f"worst {worst:.4g}; {share}"
    finally:
        ap().april_destroy(ctx)


def test_moe_small_two_layers():
    shape = ai.ModelShape(2, 128, 4, 2, 32, 0, 512, n_experts=32, experts_per_tok=4, d_expert_ffn=64)
    w = ai.Workload("moe_small", shape, 6, 24, 3, 5, 14, 2.0, 0.5, 3, 14, ai.SAMPLER_GREEDY, 0, 2, 17)
    moe_parity(w, 2, 10, min_rows=30)


def test_moe_cfg5_layer_shape():
    """One layer with configuration 5's widths: 128 experts, top-8, expert ffn 768, d 2048,
    32 query / 4 KV heads of 128; reduced vocabulary."""
    base = ai.WORKLOADS["cfg5_moe_bf16"]
    shape = ai.reduced(base, n_layers=1, vocab=4096).shape
    w = ai.Workload("cfg5_L1", shape, 4, 40, 2, 4, 10, 1.8, 0.4, 3, 10, ai.SAMPLER_GREEDY, 0, 2, base.seed)
    moe_parity(w, 2, 8, min_rows=12)


@pytest.mark.parametrize("experts,top_k", [(96, 1), (224, 6), (256, 8)])
def test_moe_router_takes_the_oracles_experts(experts, top_k):
    """One and a half, three and a half and four experts per lane; one and many arg-max steps."""
    shape = ai.ModelShape(1, 128, 4, 2, 32, 0, 512, n_experts=experts, experts_per_tok=top_k, d_expert_ffn=32)
    w = ai.Workload("moe_route", shape, 6, 24, 3, 5, 14, 2.0, 0.5, 3, 14, ai.SAMPLER_GREEDY, 0, 2, 19)
    moe_parity(w, 2, 10, min_rows=10)


def test_moe_resumed_equals_uninterrupted():
    shape = ai.ModelShape(2, 128, 4, 2, 32, 0, 512, n_experts=32, experts_per_tok=4, d_expert_ffn=64)
    w = ai.Workload("moe_small", shape, 8, 20, 5, 9, 30, 2.4, 0.6, 2, 30, ai.SAMPLER_GREEDY, 0, 4, 23)
    weights = ai.make_weights(shape, w.seed)
    reqs = ai.make_requests(w, ai.requests_needed(w))
    c1, c2 = make_engine(w, weights), make_engine(w, weights)
    try:
        a = run_gpu(c1, reqs, w.n_target, w.n_overprovision, w.max_new, w.steps)
        b = run_gpu(c2, reqs, w.n_target, w.n_target, w.max_new, w.steps)
        ta = {rid: t for g in a for rid, t in zip(g["ids"], g["tokens"])}
        tb = {rid: t for g in b for rid, t in zip(g["ids"], g["tokens"])}
        common = set(ta) & set(tb)
        assert len(common) >= w.n_target and any(r > 0 for g in a for r in g["n_resumes"])
        for rid in common:
            assert ta[rid] == tb[rid], rid
    finally:
        ap().april_destroy(c1)
        ap().april_destroy(c2)


def check_grouping(monkeypatch, w, n, n_classes=None):
    """Runs w with 4 m-tiles of an expert's rows per workgroup in every decode launch, then with 2, and compares the bits."""
    weights = ai.make_weights(w.shape, w.seed)
    reqs = ai.make_requests(w, n)
    forced = None
    if n_classes:
        ctoks = class_forced_tokens(w, n_classes)
        forced = {r.request_id: ctoks[r.request_id % n_classes][:w.max_new] for r in reqs}
    runs = []
    for tall in ("1", "1000000000"):              # always 4 m-tiles / always 2
        monkeypatch.setenv("APRIL_MOE_TALL_ROWS", tall)
        ctx = make_engine(w, weights, debug=True)
        try:
            for r in reqs:
                ap().april_debug_watch(ctx, r.request_id, 0, w.max_new)
            got = run_gpu(ctx, reqs, w.n_target, w.n_overprovision, w.max_new, w.steps, forced=forced)
            logits = {}
            for g in got:
                for rid, toks in list(zip(g["ids"], g["tokens"])) + list(g["buffer_tokens"].items()):
                    for i in range(len(toks)):
                        logits[(rid, i)] = ap().april_debug_logits(ctx, rid, i, w.shape.vocab)[0]
            runs.append((got, logits))
        finally:
            ap().april_destroy(ctx)
    (a, la), (b, lb) = runs
    assert_schedule_equal(b, a)
    assert [g["tokens"] for g in a] == [g["tokens"] for g in b]
    assert la.keys() == lb.keys() and len(la) > 40
    assert all(np.array_equal(la[k], lb[k]) for k in la)
    return a, la


def test_expert_gemm_grouping_changes_no_bit(monkeypatch):
    """Decode batches beyond a row bound give a workgroup 4 m-tiles of an expert's rows instead of
    2; the grouping is not part of any summation chain.  Here an expert has at most 9 rows, one m-tile, which runs the
    same body under either bound: the segments' alignment and the two steps' bookkeeping are what differs.
    (Prefill passes run the LDS-tiled expert kernels, whatever the bound.)"""
    shape = ai.ModelShape(2, 128, 4, 2, 32, 0, 512, n_experts=32, experts_per_tok=2, d_expert_ffn=64)
    w = ai.Workload("moe_group", shape, 6, 150, 6, 9, 6, 1.5, 0.3, 3, 6, ai.SAMPLER_GREEDY, 0, 2, 23)
    check_grouping(monkeypatch, w, ai.requests_needed(w))


@pytest.mark.parametrize("n_classes", [2, 3, 5, 13])
def test_expert_gemm_grouping_of_full_batches_changes_no_bit(monkeypatch, n_classes):
    """200 rollouts of n_classes prompts, the same forced tokens within a class: its 100, 66, 40 or 15 rows take the same
    experts, which get 4, 3, 2 or 1 m-tiles of rows (more where classes share one).  Same bits from workgroups
    of 4 and of 2 m-tiles, and from every row of a class: also from the 64th on, where the groups of 2 part."""
    shape = ai.ModelShape(2, 128, 4, 2, 32, 0, 512, n_experts=32, experts_per_tok=2, d_expert_ffn=64)
    n, gen = 200, 4
    w = ai.Workload("moe_full", shape, n_classes, 9, n, n, gen, 1.5, 0.1, gen, gen, ai.SAMPLER_GREEDY, 0, 1, 23)
    got, logits = check_grouping(monkeypatch, w, n, n_classes)
    assert got[0]["iters"] >= gen - 1 and got[0]["sum_live"] >= n * (gen - 1)
    for (rid, i), row in logits.items():
        assert np.isfinite(row).all() and np.array_equal(row, logits[(rid % n_classes, i)]), (rid, i)
