"""The row count picks the tiles of the decode projections (1 to 4 m-tiles per workgroup, 1 to 4 n-tiles,
the LDS-tiled gate/up): every choice keeps each output's summation chain.  Requests of one class (same
prompt, same forced tokens) must get bit-identical logits wherever they sit in a batch of whatever
size - every row tile of it, its last row - and when they run among three others only."""
import numpy as np
import pytest

import april_inputs as ai
from gpu_common import class_forced_tokens, have_gpu, make_engine, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not have_gpu():
        pytest.skip("no GPU")


def check_bits(shape, seed, sizes):
    import paper_2509_18521_amd as ap
    classes, gen = 31, 2
    weights = ai.make_weights(shape, seed)
    alone = None
    for n in (4,) + sizes:
        w = ai.Workload(f"tiles_{n}", shape, classes, 5, n, n, gen, 0.7, 0.1, gen, gen, ai.SAMPLER_GREEDY, 0, 1, seed)
        reqs = ai.make_requests(w, n)
        ctoks = class_forced_tokens(w, classes)
        forced = {r.request_id: ctoks[r.request_id % classes][:gen] for r in reqs}
        watched = sorted(set(r for r in range(n) if r % classes < 4) | {n - 1})
        ctx = make_engine(w, weights, debug=True, max_inflight=n)
        try:
            for rid in watched:
                ap.april_debug_watch(ctx, rid, 0, gen)
            run_gpu(ctx, reqs, n, n, gen, 1, forced=forced)
            got = {(rid, i): ap.april_debug_logits(ctx, rid, i, shape.vocab)[0] for rid in watched for i in range(gen)}
        finally:
            ap.april_destroy(ctx)
        if alone is None:
            alone = got
        for (rid, i), row in got.items():
            if rid % classes < 4:
                assert np.array_equal(row, alone[(rid % classes, i)]), (n, rid, i)
            else:
                assert np.isfinite(row).all(), (n, rid, i)


@pytest.mark.parametrize("name,sizes", [
    ("cfg2_small_bf16", (33, 65, 97, 161, 257)),
    ("cfg4_8b_bf16", (40, 70, 100, 128, 170, 200, 256, 290, 384))])
def test_a_row_keeps_its_bits_in_every_tile(name, sizes):
    base = ai.WORKLOADS[name]
    check_bits(ai.reduced(base, n_layers=1, vocab=2080).shape, base.seed, sizes)          # (an odd number of vocabulary tiles)


@pytest.mark.parametrize("name,sizes", [("cfg4_8b_bf16", (400, 450, 520, 800)), ("cfg3_mid_bf16", (450, 520))])
def test_a_row_keeps_its_bits_beyond_384_rows(name, sizes):
    """More m-groups than the tile rules of smaller batches know: split-k and gate/up tiles by rounds."""
    base = ai.WORKLOADS[name]
    check_bits(ai.reduced(base, n_layers=1, vocab=2080).shape, base.seed, sizes)


@pytest.mark.parametrize("d_model,n_q,n_kv,head_dim,d_ffn,sizes", [
    (1184, 20, 4, 64, 3104, (40, 70, 170, 330)),     # 97 feature tiles: no multiple of the 8 XCDs
    (128, 4, 2, 32, 24576, (24, 40, 70))])           # the LDS-tiled gate/up from 64 rows
def test_a_row_keeps_its_bits_in_gate_up(d_model, n_q, n_kv, head_dim, d_ffn, sizes):
    check_bits(ai.ModelShape(1, d_model, n_q, n_kv, head_dim, d_ffn, 2080), 5, sizes)


def test_a_row_keeps_its_bits_in_the_output_projection():
    """5120 columns: one m-tile per workgroup at 96 rows, pairs of n-tiles at 288, single ones above."""
    check_bits(ai.ModelShape(1, 5120, 40, 8, 128, 1024, 2080), 5, (70, 128, 280, 330))


@pytest.mark.parametrize("vocab,sizes", [(33024, (140, 250, 400)), (8224, (140, 400))])
def test_a_row_keeps_its_bits_in_the_lm_head(vocab, sizes):
    """129 groups of 256 columns: the 256-row tile on 8 wavefronts from 129 rows; 33 groups: never."""
    check_bits(ai.ModelShape(1, 160, 2, 1, 64, 96, vocab), 5, sizes)


@pytest.mark.parametrize("d_model,n_q,n_kv,head_dim,d_ffn,sizes", [
    (128, 4, 2, 32, 1024, (40, 64, 100, 130, 250, 290)),      # gate/up on half and single tiles; k ranges of 2 k-tiles
    (416, 5, 1, 64, 1056, (33, 65, 97, 129, 260)),            # odd counts of n-tiles everywhere
    (1280, 20, 4, 64, 2080, (33, 65, 97, 129, 193, 260))])    # 65 feature tiles; split-k of 2 and 3 m-tiles per workgroup
def test_a_row_keeps_its_bits_in_small_matrices(d_model, n_q, n_kv, head_dim, d_ffn, sizes):
    check_bits(ai.ModelShape(1, d_model, n_q, n_kv, head_dim, d_ffn, 2080), 5, sizes)


def test_a_row_keeps_its_bits_in_large_matrices_of_odd_tile_counts():
    """QKV of 195 n-tiles in one slice, down of 81 in four: one n-tile per workgroup and one to four m-tiles, by the rows."""
    check_bits(ai.ModelShape(1, 2592, 39 * 3, 39, 32, 2688, 2080), 5, (33, 64, 96, 120, 160, 190, 224, 300))


@pytest.mark.parametrize("d_ffn,sizes", [(6208, (90, 96)), (4896, (100, 128)), (5120, (100, 128))])
def test_a_row_keeps_its_bits_in_gate_up_of_three_m_tiles(d_ffn, sizes):
    """194 tiles at 96 rows, 153 and 160 (grid order) at 128 rows: a group of three m-tiles, alone or before one of one."""
    check_bits(ai.ModelShape(1, 128, 4, 2, 32, d_ffn, 2080), 5, sizes)


@pytest.mark.parametrize("d_model,d_ffn,vocab,sizes", [
    (2048, 256, 70016, (100, 140, 230, 300)),        # LM head: whole tiles of 256 columns, then halves, by 128, 192 and 256 rows
    (2048, 256, 50304, (100, 190, 250, 300)),        # all whole, the last one past the end: 393 columns of 128 by one and two row groups
    (2176, 128, 32032, (400, 512)),                  # 385 to 512 rows of a product longer than 2048: two row groups of 256
    (128, 9728, 2080, (64, 128, 300, 384)),          # gate/up of 152 workgroups a row group: two groups of 128 a unit; 4 stages of k, less than the ring
    (384, 12288, 2080, (60, 250, 320, 384)),         # 192: one and two row groups of 256, of 384 rows
    (1280, 9728, 2080, (40, 64, 70, 96)),            # the shortest product that turns to it at 64 rows (64-row tiles, then 128)
    (1152, 9728, 2080, (64, 90, 128))])              # the next shorter one, at 128
def test_a_row_keeps_its_bits_in_tiles_by_rounds(d_model, d_ffn, vocab, sizes):
    check_bits(ai.ModelShape(1, d_model, 2, 1, 64, d_ffn, vocab), 12, sizes)
