"""Parity of the HIP path (through the C ABI) with the float64 oracle, element by element,
on the same seeded inputs.  Bars: routing (top-k indices, permutation, offsets) bit-exact;
outputs and gradients max|gpu - ref| / max|ref| <= 1e-4 for fp32 storage and <= 2e-2 for
bf16 storage with fp32 accumulation."""
import numpy as np
import pytest

from oracle import switchhead_oracle as orc
from paper_2312_07987_amd.inputs import config, make_inputs

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}
GRADS = ("dx", "dW_Q", "dW_K", "dW_V", "dW_O", "dW_S", "dW_D", "db_S", "db_D")


def nerr(a, ref):
    ref = np.asarray(ref, dtype=np.float64)
    den = np.max(np.abs(ref))
    return float(np.max(np.abs(np.asarray(a, dtype=np.float64) - ref)) / (den if den > 0 else 1.0))


def block_errs(a, ref, lead):
    """nerr of every block along the first `lead` axes (one head's or one expert's matrix): a wrong block of
    small magnitude cannot hide under the largest entry of the whole tensor."""
    a = np.asarray(a, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    shape = ref.shape[:lead]
    a, ref = a.reshape((-1,) + ref.shape[lead:]), ref.reshape((-1,) + ref.shape[lead:])
    return np.array([nerr(x, r) for x, r in zip(a, ref)]).reshape(shape)


def run_case(cfg, family=0, shared=False, dense=False, backward=True, seed=None, check_inter=True, mutate=None):
    from paper_2312_07987_amd import binding
    from paper_2312_07987_amd.runner import DeviceLayer
    print("case", cfg, "family", family, "shared", shared, "dense", dense, flush=True)
    t = make_inputs(cfg, seed=seed, shared_router=shared)
    if dense:
        t["W_S"] = t["W_D"] = t["b_S"] = t["b_D"] = None
    if mutate is not None:
        mutate(t)
    prev = binding.switchhead_set_kernel_family(family)
    try:
        layer = DeviceLayer(cfg, t, dense=dense)
        layer.forward()
        if backward:
            layer.backward()
        y, routing = layer.outputs(), layer.routing()
        inter = layer.intermediates()
        grads = layer.grads() if backward else None
    finally:
        binding.switchhead_set_kernel_family(prev)
    f = orc.forward(t["x"], t["W_Q"], t["W_K"], t["W_V"], t["W_O"], t["W_S"], t["W_D"], t["b_S"], t["b_D"],
                    k=cfg["k"], causal=bool(cfg["causal"]), rope=bool(cfg.get("rope")), T_q=cfg.get("T_q") or None)
    Tq = cfg.get("T_q") or cfg["T"]
    if Tq != cfg["T"]:   # fewer queries than keys: the destination side's tables hold B*Tq tokens
        routing = dict(routing)
        for nm in ("idx", "gate", "perm"):
            routing[nm] = [routing[nm][0], routing[nm + "_D"]]
    tol = TOL[cfg["dtype"]]
    # integer work: exact
    for s, side in enumerate("SD"):
        bad = np.argwhere(routing["idx"][s] != f["idx_" + side])
        assert bad.size == 0, ("top-k mismatch", side, bad[:4], [f["margin_" + side][b[0], b[1]] for b in bad[:4]])
        assert np.array_equal(routing["offsets"][s], f["offsets_" + side]), side
        assert np.array_equal(routing["perm"][s], f["perm_" + side]), side
        # gates are fp32; on the bf16 path they come from fp32-accumulated logits
        assert nerr(routing["gate"][s], f["gate_" + side]) < (1e-6 if cfg["dtype"] == "f32" else 2e-5)
    if check_inter:
        for n in ("Q", "K", "V", "ctx"):
            assert nerr(inter[n], f[n]) < tol, n
    e = nerr(y, f["y"])
    print("  y err %.3e" % e, flush=True)
    assert e < tol
    if backward:
        b = orc.backward(t["x"], t["W_Q"], t["W_K"], t["W_V"], t["W_O"], t["W_S"], t["W_D"], f, t["dy"][:, cfg["T"] - Tq:])
        errs = {}
        for n in GRADS:
            if b[n] is None:
                continue
            assert grads[n] is not None, n
            errs[n] = nerr(grads[n], b[n])
        print("  grad errs", {n: "%.2e" % v for n, v in errs.items()}, flush=True)
        assert max(errs.values()) < tol, errs
        # the same bar per expert matrix / per head, and for the query rows and the cached rows of dx apart
        # (an expert nobody chose has an all-zero reference: nerr then is the largest absolute entry, i.e. exact zeros pass)
        blocks = {"dW_V": block_errs(grads["dW_V"], b["dW_V"], 2), "dW_O": block_errs(grads["dW_O"], b["dW_O"], 2)}
        for n in ("dW_Q", "dW_K"):
            blocks[n] = block_errs(grads[n], b[n], 2 if cfg.get("qk_experts") else 1)
        if Tq != cfg["T"]:
            blocks["dx_cached_rows"] = np.array(nerr(grads["dx"][:, :cfg["T"] - Tq], b["dx"][:, :cfg["T"] - Tq]))
            blocks["dx_query_rows"] = np.array(nerr(grads["dx"][:, cfg["T"] - Tq:], b["dx"][:, cfg["T"] - Tq:]))
        worst = {n: float(v.max()) for n, v in blocks.items()}
        print("  per-block grad errs", {n: "%.2e" % v for n, v in worst.items()}, flush=True)
        assert max(worst.values()) < tol, worst
    return f, routing


def small(name, **over):
    c = config(name)
    c.update(over)
    return c


@pytest.mark.parametrize("family", [0, 1])
def test_c0_fp32(family):
    run_case(config("c0"), family=family)


@pytest.mark.parametrize("causal", [1, 0])
def test_fp32_ragged_everything(causal):
    # nothing is a multiple of a tile: T=37, d_model=50, d_head=20, E=7, k=3
    run_case(dict(name="rag", dtype="f32", B=3, T=37, d_model=50, nheads=3, d_head=20, E=7, k=3, causal=causal, bias0=0.0),
             seed=5)


@pytest.mark.parametrize("over", [
    dict(B=1, T=257, d_model=76, d_head=76),                     # one row past a chunk: partial sums, and past four 64-row tiles
    dict(B=3, T=100, d_model=412, d_head=80, T_q=99),            # 80-wide tiles, queries packed, two token sets
    dict(B=1, T=320, d_model=48, d_head=33, E=3, k=3),           # rows of no vector width
    dict(B=2, T=97, d_model=64, d_head=130, E=7, k=2),           # experts over twice the active ones: the atomic path
    dict(B=5, T=65, d_model=100, d_head=196, nheads=1, causal=0),
    dict(B=1, T=31, d_model=64, d_head=16, nheads=9, E=4),       # more segments than one concatenated product takes
])
@pytest.mark.parametrize("shared", [False, True])
def test_fp32_tile_edges(over, shared):
    """The fp32 matrix-core kernels at the edges of their tiles (64 rows, 64 or 80 columns, 32 owned attention rows), chunks
    and dispatch rules."""
    run_case(dict(dict(name="edge32", dtype="f32", nheads=2, E=4, k=2, causal=1, bias0=0.0), **over), shared=shared, seed=31)


@pytest.mark.parametrize("over, shared", [
    (dict(B=5, T=261, d_model=412, nheads=2, d_head=76, E=5, k=3), False),              # 8-byte pieces, ragged in both features
    (dict(B=3, T=701, d_model=1024, nheads=4, d_head=128, E=5, k=3), True),             # a last unit of a few rows, one router
    (dict(B=2, T=800, d_model=1024, nheads=4, d_head=128, E=8, k=2, qk_experts=1), False),   # more items than fit at once
    (dict(B=2, T=900, d_model=300, nheads=2, d_head=168, E=4, k=2, T_q=333), False),    # both tile shapes partly filled, two token sets
    (dict(B=2, T=900, d_model=256, nheads=1, d_head=256, E=3, k=2, T_q=450), True),     # a shared router over two token sets
    (dict(B=1, T=1031, d_model=512, nheads=4, d_head=64, E=16, k=1), False),            # 64 groups
])
def test_bf16_weight_gradient_list(over, shared):
    """All weight gradients in one launch: part and tile edges, and an expert nobody chooses (its gradient is zero)."""
    def shun(t):
        for side in ("b_S", "b_D"):
            if t.get("W_" + side[2]) is not None:
                b = np.zeros(cfg["nheads"] * cfg["E"], np.float32)
                b[1::cfg["E"]] = -30.0
                t[side] = b
    cfg = dict(dict(name="wgrads", dtype="bf16", causal=1, bias0=0.0), **over)
    run_case(cfg, shared=shared, seed=47, mutate=shun)


@pytest.mark.parametrize("over, shared", [
    (dict(B=5, T=1161), False),                       # a last tile of 173 rows
    (dict(B=5, T=1160, T_q=1000), False),             # tiles with query rows of two sequences, query rows beside cached ones
    (dict(B=3, T=2600, T_q=1300), True),              # tiles without any query row, one router over two token sets
    (dict(B=5, T=1161, qk_experts=1), False),         # queries and keys over their experts, gates of either side
    (dict(B=6, T=1000, T_q=961, qk_experts=1), True),
])
def test_bf16_gated_concatenation_forms(over, shared):
    """One product for y and one for dx over every (head, expert): token counts that are no multiple of the tile, two token sets,
    expert queries and keys."""
    cfg = dict(dict(name="gated", dtype="bf16", d_model=2048, nheads=2, d_head=64, E=3, k=2, causal=1, bias0=0.0), **over)
    run_case(cfg, shared=shared, seed=53)


@pytest.mark.parametrize("over, how", [
    (dict(T=520, T_q=1), "own"),                      # three blocks of source tokens, one of destination tokens
    (dict(T=257, T_q=256), "shared"),
    (dict(T=300, T_q=7, E=8, k=2), "own"),
    (dict(T=300), "shared"),                          # one selection: all of the destination side's tables are copies
    (dict(T=300, T_q=44, E=1, k=1), "dense"),
    (dict(T=300, E=1, k=1), "dense"),
])
def test_bf16_routing_tables_of_both_sides(over, how):
    """Both sides' selections and sorts in shared launches, tables copied or filled directly."""
    cfg = dict(dict(name="sides", dtype="bf16", B=2, d_model=128, nheads=3, d_head=32, E=4, k=2, causal=1, bias0=0.0), **over)
    run_case(cfg, shared=how == "shared", dense=how == "dense", seed=59)


@pytest.mark.parametrize("over", [
    dict(T=33, d_model=1024, d_head=128),                        # one row past a tile
    dict(T=65, d_model=1000, d_head=72, E=5, k=3),               # a reduction that no wave's share divides, a last tile of 8 columns
    dict(T=70, d_model=2056, d_head=40, qk_experts=1),           # more than one trip per wave
    dict(T=40, d_model=24, d_head=8),                            # waves without any share
    dict(T=300, d_model=264, d_head=64, T_q=3, causal=0),        # three query rows per sequence
])
def test_bf16_projections_of_a_few_rows(over):
    """The 32 x 32 tiles of short calls at the edges of their rows, columns and shares of the reduction."""
    run_case(dict(dict(name="few", dtype="bf16", B=1, nheads=2, E=4, k=2, causal=1, bias0=0.0), **over), seed=61)


def test_fp32_shared_selection_and_dense_mode():
    run_case(small("c0"), shared=True)
    run_case(dict(name="dense", dtype="f32", B=2, T=48, d_model=64, nheads=4, d_head=16, E=1, k=1, causal=1, bias0=0.0),
             dense=True, seed=9)


def test_fp32_k_equals_E_and_single_token_sequences():
    run_case(dict(name="kE", dtype="f32", B=2, T=33, d_model=32, nheads=2, d_head=16, E=3, k=3, causal=1, bias0=0.0), seed=2)
    run_case(dict(name="T1", dtype="f32", B=5, T=1, d_model=32, nheads=2, d_head=16, E=4, k=2, causal=1, bias0=0.0), seed=3)


def test_fp32_empty_expert_and_max_limits():
    # bias -50 on an expert nobody then picks: empty group, zero weight gradient
    cfg = dict(name="empty", dtype="f32", B=2, T=40, d_model=32, nheads=2, d_head=16, E=4, k=2, causal=1, bias0=-50.0)
    f, routing = run_case(cfg, seed=4)
    assert np.all(np.diff(routing["offsets"], axis=-1)[..., 0] == 0)
    # the largest E, k and d_head the library accepts
    run_case(dict(name="max", dtype="f32", B=1, T=70, d_model=24, nheads=1, d_head=256, E=64, k=8, causal=1, bias0=0.0), seed=6)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_small_multi_tile(family):
    # several tiles and a ragged tail in every dimension the kernels tile over
    run_case(small("c2", B=3, T=200, d_model=320, nheads=2, d_head=128), family=family, seed=11)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_ragged_head_dims(family):
    run_case(small("c1", B=3, T=100), family=family, seed=12)


def test_bf16_noncausal_shared_dense():
    run_case(small("c2", B=2, T=130, d_model=256, nheads=2, causal=0), seed=13)
    run_case(small("c2", B=2, T=130, d_model=256, nheads=2), shared=True, seed=14)
    run_case(dict(name="dense16", dtype="bf16", B=2, T=130, d_model=256, nheads=4, d_head=64, E=1, k=1, causal=1, bias0=0.0),
             dense=True, seed=15)


def test_bf16_mac_matched_shapes():
    """Head counts and widths of the MAC-matched models (Sec. 3.5 "MAC-Matched Setup"): 3 heads of 112, 6 heads of 168."""
    run_case(small("c1", B=2, T=160, nheads=3, d_head=112), seed=16)
    run_case(small("c2", B=1, T=200, nheads=6, d_head=168), seed=17)


@pytest.mark.parametrize("family", [0, 1])
def test_fp32_expert_queries_and_keys(family):
    """All four projections as expert mixtures (Sec. 2.2): W_Q, W_K are banks like W_V."""
    run_case(small("c0", qk_experts=1), family=family)
    run_case(dict(name="ragqk", dtype="f32", B=3, T=37, d_model=50, nheads=3, d_head=20, E=7, k=3, causal=1, bias0=0.0,
                  qk_experts=1), family=family, seed=25)


def test_fp32_expert_queries_and_keys_shared_selection():
    run_case(small("c0", qk_experts=1), shared=True, seed=26)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_expert_queries_and_keys(family):
    run_case(small("c2", B=3, T=200, d_model=320, nheads=2, d_head=128, qk_experts=1), family=family, seed=27)
    run_case(small("c1", B=3, T=100, qk_experts=1), family=family, seed=28)
    run_case(small("c2", B=2, T=130, d_model=256, nheads=2, qk_experts=1), family=family, shared=True, seed=29)


def test_full_config_expert_queries_and_keys():
    """c2 at full size with query and key experts, in the launch configuration bench.py times."""
    run_case(small("c2", qk_experts=1), seed=30)


@pytest.mark.parametrize("family", [0, 1])
def test_fp32_rotary_queries_and_keys(family):
    """Rotary position embedding (App. A.4 "RoPE Positional Encodings"), fp32: even, odd and ragged head widths, long sequences."""
    run_case(small("c0", rope=1), family=family)
    run_case(dict(name="ragrope", dtype="f32", B=2, T=37, d_model=50, nheads=3, d_head=21, E=7, k=3, causal=1, bias0=0.0,
                  rope=1), family=family, seed=45)
    run_case(dict(name="longrope", dtype="f32", B=1, T=1500, d_model=32, nheads=1, d_head=16, E=3, k=2, causal=1, bias0=0.0,
                  rope=1, qk_experts=1), family=family, seed=46)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_rotary_queries_and_keys(family):
    # the paper's rotary models: 2 heads of 64 (E=5, k=3, T=512) and 4 heads of 100 (E=4, k=2, T=1024)
    run_case(small("c1", B=2, T=512, d_head=64, rope=1), family=family, seed=47)
    run_case(small("c2", B=1, T=1024, nheads=4, d_head=100, E=4, k=2, rope=1), family=family, seed=48)
    run_case(small("c2", B=2, T=130, d_model=256, nheads=2, rope=1, qk_experts=1, causal=0), family=family, seed=49)


def test_full_config_rotary():
    """c2 at full size with rotary queries and keys, in the launch configuration bench.py times."""
    run_case(small("c2", rope=1), seed=50)


@pytest.mark.parametrize("family", [0, 1])
def test_fp32_fewer_queries_than_keys(family):
    """Attention over a cached context (App. A.2): queries for the last T_q positions only."""
    run_case(small("c0", T_q=32), family=family)
    run_case(dict(name="ragxl", dtype="f32", B=3, T=37, d_model=50, nheads=3, d_head=20, E=7, k=3, causal=1, bias0=0.0,
                  T_q=13, rope=1), family=family, seed=55)
    run_case(dict(name="ragxl2", dtype="f32", B=2, T=45, d_model=32, nheads=2, d_head=16, E=4, k=2, causal=0, bias0=0.0,
                  T_q=1, qk_experts=1), family=family, seed=56)
    run_case(small("c0", T_q=40), family=family, shared=True, seed=57)
    run_case(dict(name="densexl", dtype="f32", B=2, T=48, d_model=64, nheads=4, d_head=16, E=1, k=1, causal=1, bias0=0.0,
                  T_q=16), family=family, dense=True, seed=58)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_fewer_queries_than_keys(family):
    run_case(small("c2", B=3, T=400, d_model=320, nheads=2, d_head=128, T_q=200), family=family, seed=59)
    run_case(small("c1", B=3, T=200, T_q=100, rope=1), family=family, seed=60)
    run_case(small("c2", B=2, T=260, d_model=256, nheads=2, T_q=130, qk_experts=1), family=family, seed=61)
    run_case(small("c2", B=2, T=260, d_model=256, nheads=2, T_q=77, causal=0), family=family, shared=True, seed=62)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_long_ragged_sequences(family):
    """Sequences past 1024 positions (two wave groups share a query tile's key tiles in the forward kernel) whose lengths
    are no multiple of any tile, with and without the causal mask, and with a cached context whose offset is odd: the
    last key tile repeats its last row instead of zeros, and the score gradient kept for the dQ product has ragged
    rows and a region the dK / dV kernel never writes."""
    run_case(small("c2", B=1, T=1100, d_model=256, nheads=2, d_head=128), family=family, seed=64)
    run_case(small("c2", B=1, T=1337, d_model=256, nheads=2, d_head=64, T_q=901), family=family, seed=65)
    run_case(small("c2", B=2, T=1030, d_model=256, nheads=1, d_head=96, causal=0), family=family, seed=66)


@pytest.mark.parametrize("d_head", [48, 128])
def test_bf16_long_causal_context_not_a_multiple_of_the_key_tile(d_head):
    """T >= 1024 (the forward kernel's two wave groups take alternate key tiles) under a causal mask with 22 cached
    positions: queries 32..41 see keys up to position 54..63 only, so for them the second group's first tile (keys
    64..127, visited because the wave's last query sees key 64) is fully masked before any key was seen."""
    run_case(dict(name="off22", dtype="bf16", B=1, T=1100, d_model=64, nheads=2, d_head=d_head, E=5, k=2, causal=1, bias0=0.0,
                  T_q=1078), seed=74)


@pytest.mark.parametrize("T,T_q", [(300, 143), (1024, 143)])
def test_bf16_dense_mode_fewer_queries_than_keys(T, T_q):
    """Dense multi-head attention (no routers) over a cached context on the matrix-core kernels: each side's
    expert-set tables (one set, but the set-path kernels read them) are built on that side's own tokens."""
    run_case(dict(name="dense_ctx", dtype="bf16", B=2, T=T, d_model=64, nheads=2, d_head=64, E=1, k=1, causal=1, bias0=0.0, T_q=T_q),
             dense=True, seed=75)


def test_bf16_mixed_shapes_long_context():
    """Shapes off the beaten track for the attention kernels of head widths 64..128: head widths that are padded to the
    next compiled width (72, 104), cached contexts with odd offsets past 1024 keys, rotary turns, no causal mask, E = 8."""
    run_case(dict(name="mix1", dtype="bf16", B=2, T=2049, d_model=320, nheads=3, d_head=128, E=5, k=3, causal=1, bias0=0.0,
                  T_q=722, rope=1), seed=1012)
    run_case(dict(name="mix2", dtype="bf16", B=2, T=2049, d_model=256, nheads=3, d_head=64, E=8, k=3, causal=0, bias0=0.0,
                  T_q=1482, rope=1), seed=1019)
    run_case(dict(name="mix3", dtype="bf16", B=1, T=2049, d_model=320, nheads=3, d_head=104, E=2, k=2, causal=1, bias0=0.0,
                  T_q=1411), seed=1022)
    run_case(dict(name="mix4", dtype="bf16", B=2, T=1100, d_model=512, nheads=1, d_head=72, E=8, k=2, causal=1, bias0=0.0,
                  T_q=150, rope=1), seed=1006)


def test_full_config_cached_context():
    """The paper's main setting at c2's sizes: a context twice the current chunk (T = 2 * 512 keys, 512
    queries per sequence), in the launch configuration bench.py times."""
    run_case(small("c2", T=1024, T_q=512), seed=63)


@pytest.mark.parametrize("family", [0, 1])
def test_all_variants_together(family):
    """Expert queries and keys, rotary positions, a cached context and one shared selection in one call."""
    run_case(dict(name="allf32", dtype="f32", B=2, T=41, d_model=40, nheads=3, d_head=18, E=6, k=2, causal=1, bias0=0.0,
                  qk_experts=1, rope=1, T_q=17), family=family, shared=True, seed=70)
    run_case(small("c2", B=2, T=300, d_model=256, nheads=2, qk_experts=1, rope=1, T_q=140), family=family, shared=True, seed=71)
    run_case(small("c2", B=2, T=300, d_model=256, nheads=2, qk_experts=1, rope=1, T_q=140), family=family, seed=72)


def test_bf16_router_weight_gradient_forms():
    """The routers' weight gradients either ride along the Q/K weight-gradient launch (2 * H * E, padded,
    fits a head's width) or take a launch of their own: the last size that fits, the first that does not."""
    run_case(small("c2", B=2, T=256, d_model=256, nheads=4, d_head=128, E=16, k=2), seed=73)
    run_case(small("c2", B=2, T=256, d_model=256, nheads=4, d_head=128, E=17, k=2), seed=74)
    run_case(small("c2", B=2, T=256, d_model=256, nheads=4, d_head=128, E=16, k=2), shared=True, seed=75)


@pytest.mark.parametrize("family", [0, 1])
def test_bf16_single_token_sequences(family):
    """T = 1: the attention matrix is the number 1, so the gradients of queries and keys are exactly zero;
    the row sums of the backward pass must come from the same rounded values its products use, or
    rounding noise of the size of a normal gradient is left where the reference has nothing."""
    run_case(dict(name="t1a", dtype="bf16", B=2, T=1, d_model=96, nheads=1, d_head=64, E=12, k=3, causal=1, bias0=1.5),
             family=family, seed=1027)
    run_case(dict(name="t1b", dtype="bf16", B=5, T=1, d_model=64, nheads=1, d_head=16, E=5, k=3, causal=0, bias0=0.0,
                  qk_experts=1, rope=1), family=family, shared=True, seed=1053)


def test_bf16_sort_tables_too_large_for_the_in_block_scan():
    """126 expert sets and 66 token blocks: the counting sorts take their separate scan launch (smaller
    tables are scanned by every scatter block for itself)."""
    run_case(dict(name="bigsort", dtype="bf16", B=66, T=256, d_model=64, nheads=1, d_head=32, E=9, k=4, causal=1, bias0=0.0),
             seed=76)


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c4"])
def test_full_config(name):
    """The paper-shaped workloads at full size, in the launch configuration bench.py times."""
    cfg = config(name)
    f, routing = run_case(cfg, check_inter=True)
    counts = np.diff(routing["offsets"], axis=-1)
    print("  per-expert counts (side, head, expert):", counts.tolist(), flush=True)
    assert counts.sum() == 2 * cfg["nheads"] * cfg["B"] * cfg["T"] * cfg["k"]
    if name == "c4":
        assert np.all(counts[..., 0] > 0.95 * cfg["B"] * cfg["T"])   # the biased expert takes nearly every token


def test_gated_gemms_second_round_of_tiles():
    """c2's layer with more tokens than one round of the 256-row tiles holds (36 sequences: 72 row tiles x 4 column
    tiles = 288 work-groups for 256 CUs): the tiles of the second round, and a token count that is no power of two."""
    run_case(small("c2", B=36), seed=70)


@pytest.mark.parametrize("E,k", [(4, 2), (6, 2)])
def test_bf16_empty_expert(E, k):
    """An expert nobody picks (bias -50) on the matrix-core kernels: an empty group in the sorted tables, in the
    list of non-empty units the weight-gradient work-groups place themselves by, and an all-zero weight gradient.
    E = 4, k = 2 takes the gated concatenation (a gate column that is zero for every token), E = 6 the expert sets."""
    cfg = dict(name="empty16", dtype="bf16", B=8, T=320, d_model=256, nheads=2, d_head=64, E=E, k=k, causal=1, bias0=-50.0)
    f, routing = run_case(cfg, seed=71)   # 2560 tokens, a multiple of 256: what the gated concatenation asks for
    assert np.all(np.diff(routing["offsets"], axis=-1)[..., 0] == 0)


def test_bf16_max_limits():
    """The largest E, k and d_head the library accepts, bf16 storage."""
    run_case(dict(name="max16", dtype="bf16", B=2, T=140, d_model=64, nheads=1, d_head=256, E=64, k=8, causal=1, bias0=0.0), seed=72)
    # more than 64 (head, expert) groups: the weight-gradient work-groups find their unit by the plain decoding
    run_case(dict(name="groups80", dtype="bf16", B=2, T=256, d_model=128, nheads=5, d_head=64, E=16, k=2, causal=1, bias0=0.0), seed=73)


def test_bf16_decoding_and_many_short_sequences():
    """Shapes from random sweeps that the other cases do not reach: one query against a long cached context (with rotary
    turns and expert queries / keys; with shared selection), hundreds of sequences of a few tokens, 64 experts with six
    active over a cached context."""
    run_case(dict(name="dec1", dtype="bf16", B=1, T=3000, d_model=256, nheads=4, d_head=64, E=4, k=3, causal=1, bias0=0.0, T_q=1,
                  rope=1, qk_experts=1), family=1, seed=8014)
    run_case(dict(name="dec2", dtype="bf16", B=1, T=1500, d_model=128, nheads=2, d_head=32, E=2, k=1, causal=1, bias0=0.0, T_q=1),
             shared=True, seed=8017)
    run_case(dict(name="short1", dtype="bf16", B=300, T=17, d_model=512, nheads=2, d_head=64, E=5, k=2, causal=1, bias0=0.0), seed=8021)
    run_case(dict(name="short2", dtype="bf16", B=777, T=3, d_model=128, nheads=4, d_head=32, E=2, k=2, causal=0, bias0=0.0), seed=8022)
    run_case(dict(name="e64", dtype="bf16", B=1, T=1100, d_model=128, nheads=1, d_head=128, E=64, k=6, causal=0, bias0=2.0, T_q=92),
             seed=7019)


def _tie_columns(E):
    """Input edit for the tie cases: in head 0 expert 2 repeats expert 0's router column, in head 1 every
    expert has the same column (all E logits of a token are bitwise equal under any fixed summation order)."""
    def edit(t):
        for W in ("W_S", "W_D"):
            if t[W] is None:
                continue
            w = t[W].copy()
            w[:, 2] = w[:, 0]
            w[:, E:2 * E] = w[:, E:E + 1]
            t[W] = w
    return edit


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("k", [2, 4])
@pytest.mark.parametrize("dtype,family", [("f32", 0), ("f32", 1), ("bf16", 0), ("bf16", 1)])
def test_equal_logits_lowest_index_wins(dtype, family, k, shared):
    """Exactly equal logits (Sec. 2.2, argtopk; the paper gives no tie rule, the reading taken is: lower
    index first): duplicated router columns make ties on both sides, for k < E and k = E, with one shared
    selection too.  Indices, gates, permutation and offsets must be the oracle's in every kernel family: fp32
    storage (fp64 chain), bf16 storage with the two-stage matrix-core router, bf16 with the plain kernels."""
    E = 4
    if dtype == "f32":
        cfg = dict(name="tie32", dtype="f32", B=2, T=70, d_model=48, nheads=2, d_head=16, E=E, k=k, causal=1, bias0=0.0)
    else:
        cfg = small("c2", B=2, T=200, d_model=320, nheads=2, d_head=64, E=E, k=k)
    f, routing = run_case(cfg, family=family, shared=shared, seed=90 + k, mutate=_tie_columns(E))
    for side in ("S", "D"):
        idx = f["idx_" + side]
        if k < E:
            # the tie decided something: expert 0 taken without its copy 2 somewhere, never the other way round
            lo, hi = (idx[0] == 0).any(-1), (idx[0] == 2).any(-1)
            assert (lo & ~hi).any() and not (hi & ~lo).any()
        assert np.array_equal(idx[1], np.broadcast_to(np.arange(k), idx[1].shape))


def test_rerun_is_stable():
    """Two forward calls on the same workspace give the same bits: no atomic add decides the routing
    tables or, on the matrix-core path this shape takes, y."""
    from paper_2312_07987_amd.runner import DeviceLayer
    cfg = small("c2", B=2, T=256)
    t = make_inputs(cfg, seed=3)
    layer = DeviceLayer(cfg, t)
    layer.forward()
    y1, r1 = layer.outputs().copy(), layer.routing()
    layer.forward()
    y2, r2 = layer.outputs(), layer.routing()
    assert all(np.array_equal(r1[n], r2[n]) for n in r1)
    assert np.array_equal(y2, y1)   # the matrix-core path adds its partial sums in a fixed order


def test_matrix_core_path_is_deterministic():
    """bf16 storage, expert-set path: no atomic add decides y, dx or the weight gradients of the
    projections or of the routers (per-chunk and per-block partial sums are added in a fixed order), so
    two runs agree bit for bit."""
    from paper_2312_07987_amd.runner import DeviceLayer
    cfg = small("c2", B=4, T=256)
    t = make_inputs(cfg, seed=5)
    layer = DeviceLayer(cfg, t)
    runs = []
    for _ in range(2):
        layer.forward()
        layer.backward()
        g = layer.grads()
        g["y"] = layer.outputs().copy()
        runs.append({n: np.array(v, copy=True) for n, v in g.items() if v is not None})
    for n in ("y", "dx", "dW_Q", "dW_K", "dW_V", "dW_O", "dW_S", "dW_D", "db_S", "db_D"):
        assert np.array_equal(runs[0][n], runs[1][n]), n
