"""Sizes on both sides of the lines between the kernels that serve one step, and the remainders of their tiles, against the float64 oracle
(bars and checks as in test_gpu_parity)."""
import pytest

from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


def _cfg(**over):
    cfg = dict(name="tiles", dtype="bf16", B=1, causal=1, bias0=0.0)
    cfg.update(over)
    return cfg


@pytest.mark.parametrize("over, shared", [
    # 16 x 32 tiles: single rows and columns, remainders of rows, columns and 16 reduction indices, rows of no 16 bytes
    (dict(T=1, d_model=1, nheads=1, d_head=1, E=1, k=1), False),
    (dict(T=15, d_model=33, nheads=3, d_head=17, E=4, k=3), False),
    (dict(T=17, d_model=64, nheads=2, d_head=32, E=4, k=2), True),
    (dict(T=129, T_q=47, d_model=412, nheads=2, d_head=76, E=5, k=3), False),
    (dict(T=40, d_model=36, nheads=2, d_head=20, E=3, k=2, qk_experts=1), False),
    (dict(T=90, d_model=100, nheads=2, d_head=20, E=7, k=2), False),               # sorted rows, atomics
    # 64-row tiles
    (dict(T=1300, d_model=410, nheads=2, d_head=42, E=5, k=3), False),
    (dict(T=1400, T_q=1300, d_model=412, nheads=2, d_head=76, E=5, k=3), True),
    # few of those, but many small tiles: a short reduction; 4-byte loads along the reduction
    (dict(T=1040, d_model=128, nheads=4, d_head=76, E=1, k=1), False),
    (dict(T=400, d_model=410, nheads=3, d_head=36, E=5, k=3), False),
])
def test_fp32_tiles(over, shared):
    run_case(_cfg(dtype="f32", **over), shared=shared, seed=211)


@pytest.mark.parametrize("over, dense", [
    # the output experts of a few rows: one row, remainders of rows, columns and 64 reduction indices, 8-byte pieces, more experts than a wave
    # takes at a time, fewer pieces than waves, dense heads; 256 tiles and the next size
    (dict(T=1, d_model=8, nheads=1, d_head=8, E=3, k=2), False),
    (dict(T=33, d_model=72, nheads=2, d_head=24, E=3, k=2), False),
    (dict(T=70, T_q=37, d_model=412, nheads=2, d_head=76, E=5, k=3), False),
    (dict(T=100, d_model=1024, nheads=4, d_head=100, E=8, k=2), False),
    (dict(T=65, d_model=128, nheads=4, d_head=64, E=13, k=4), False),
    (dict(T=50, d_model=256, nheads=20, d_head=80, E=1, k=1), True),
    (dict(T=256, d_model=1024, nheads=4, d_head=128, E=5, k=3), False),
    (dict(T=257, d_model=1024, nheads=4, d_head=128, E=5, k=3), False),
    # too many experts for those a token selects, and few enough: two heads, one head; expert-sorted rows of few columns and of many
    (dict(T=40, d_model=256, nheads=2, d_head=128, E=32, k=1), False),
    (dict(T=40, d_model=256, nheads=1, d_head=64, E=5, k=1), False),
    (dict(T=1, d_model=256, nheads=4, d_head=128, E=16, k=4), False),
    (dict(T=16, d_model=256, nheads=4, d_head=128, E=16, k=4), False),
    (dict(T=40, d_model=256, nheads=1, d_head=64, E=16, k=1), False),
    (dict(T=16, d_model=1024, nheads=4, d_head=128, E=16, k=4), False),
    # ... and on narrow models, whose other path is short; 512 tiles and the next size
    (dict(T=17, d_model=100, nheads=8, d_head=256, E=4, k=1), False),
    (dict(T=40, d_model=64, nheads=2, d_head=76, E=32, k=5), False),
    (dict(T=1024, d_model=512, nheads=1, d_head=16, E=3, k=3), False),
    (dict(T=1025, d_model=512, nheads=1, d_head=16, E=3, k=3), False),
])
def test_output_experts_of_a_few_rows(over, dense):
    run_case(_cfg(**over), dense=dense, backward=False, seed=223)


@pytest.mark.parametrize("over", [
    dict(T=2100, d_model=64, nheads=16, d_head=128, E=2, k=1),      # dense queries and keys: 144 tiles of 256 x 256
    dict(T=2100, d_model=4096, nheads=2, d_head=64, E=5, k=2),      # their input gradient: 144 such tiles
    dict(T=2100, d_model=256, nheads=2, d_head=128, E=5, k=2),      # both: fewer than 128
])
def test_dense_projections_by_tile_count(over):
    run_case(_cfg(**over), seed=227, check_inter=False)


@pytest.mark.parametrize("over", [
    dict(B=2, T=300, d_model=128, nheads=2, d_head=100, E=4, k=2, rope=1),
    dict(B=2, T=517, T_q=130, d_model=128, nheads=2, d_head=68, E=3, k=2),
    dict(B=3, T=256, d_model=412, nheads=2, d_head=76, E=5, k=3, causal=0),
])
def test_query_gradient_from_kept_scores(over):
    """Head widths that are multiples of four but not of eight: the score gradient is kept where it fits over dead buffers."""
    run_case(_cfg(**over), seed=229)


@pytest.mark.parametrize("over", [
    # at most 16 queries per sequence: one and all queries of a block, fewer keys than waves have pieces, remainders of a piece and of a
    # round of pieces, rows of 8 and 16 bytes, every width of the operands; no causal mask; all queries are the sequence
    dict(T=33, T_q=1, d_model=64, nheads=3, d_head=8, E=2, k=1),
    dict(T=300, T_q=16, d_model=72, nheads=2, d_head=36, E=3, k=2, rope=1),
    dict(B=3, T=257, T_q=4, d_model=412, nheads=2, d_head=76, E=5, k=3),
    dict(T=1055, T_q=15, d_model=128, nheads=2, d_head=100, E=4, k=2),
    dict(B=2, T=640, T_q=16, d_model=64, nheads=2, d_head=128, E=2, k=1, causal=0),
    dict(B=9, T=16, d_model=128, nheads=2, d_head=64, E=4, k=2),
    # the other kernel: the next number of queries, more work-groups than a round of few keys
    dict(T=300, T_q=17, d_model=72, nheads=2, d_head=64, E=3, k=2),
    dict(B=129, T=70, T_q=3, d_model=64, nheads=2, d_head=64, E=3, k=2),
    dict(B=129, T=256, T_q=3, d_model=64, nheads=2, d_head=64, E=3, k=2),   # (and enough of them)
    dict(B=129, T=300, T_q=16, d_model=64, nheads=2, d_head=76, E=3, k=2),
    dict(B=65, T=1030, T_q=2, d_model=64, nheads=4, d_head=100, E=3, k=2),  # (and enough of them)
])
def test_attention_of_a_few_queries(over):
    # (a single query of narrow heads: its router gradient is a few cancelling sums of 8 rounded terms, no measure of anything)
    run_case(_cfg(**over), backward=over["d_head"] > 8, seed=233)


@pytest.mark.parametrize("over", [
    # rows of 8 but not 16 bytes in pieces of 16: reductions and outputs that end in a half piece, in the first piece, in the last place of a
    # K step and in the first of the next, or in none; dense and gathered rows, expert sets, concatenated reductions, weight gradients, on both sides of
    # the lines
    dict(T=40, d_model=12, nheads=2, d_head=12, E=4, k=2),
    dict(T=300, d_model=68, nheads=2, d_head=60, E=5, k=3),
    dict(T=300, d_model=124, nheads=3, d_head=132, E=3, k=2),
    dict(B=3, T=1000, d_model=412, nheads=2, d_head=76, E=8, k=2),                 # sorted rows: 94 tiles, sets: 192
    dict(B=17, T=1000, d_model=260, nheads=3, d_head=68, E=5, k=3, qk_experts=1),
    dict(B=17, T=1000, d_model=620, nheads=4, d_head=100, E=4, k=2),               # dense rows 1064 tiles, their gradient 665
    dict(B=9, T=1000, d_model=412, nheads=4, d_head=48, E=1, k=1),                 # rows of a whole number of pieces, outputs that are not
])
def test_rows_of_half_pieces(over):
    run_case(_cfg(**over), seed=239, check_inter=False)
