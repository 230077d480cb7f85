"""Properties of the layer that a choice of kernel path must not change: buffers that may overlap, sums that stay in
fp32, experts that must not be read, results that repeat bit for bit."""
import numpy as np
import pytest

from oracle import switchhead_oracle as orc
from paper_2312_07987_amd.inputs import make_inputs, round_to_bf16
from test_gpu_parity import TOL, nerr, run_case

pytestmark = pytest.mark.gpu


def _cfg(**over):
    return dict(dict(name="kept", dtype="bf16", causal=1, bias0=0.0, qk_experts=0), **over)


def _steps(layer):
    """Labels of the steps that a forward and a backward call run."""
    from paper_2312_07987_amd import binding
    binding.switchhead_profile_enable(1)
    try:
        layer.forward()
        layer.backward()
        return set(binding.switchhead_profile_read())
    finally:
        binding.switchhead_profile_enable(0)


def _layer(cfg, t, dense=False):
    from paper_2312_07987_amd.runner import DeviceLayer
    print("case", cfg, flush=True)
    return DeviceLayer(cfg, t, dense=dense)


@pytest.mark.parametrize("over, dense", [
    (dict(B=2, T=300, d_model=1024, nheads=4, d_head=128, E=5, k=3), False),             # expert sets
    (dict(B=5, T=1161, d_model=2048, nheads=2, d_head=64, E=3, k=2), False),             # one product over every (head, expert)
    (dict(B=5, T=1161, d_model=2048, nheads=2, d_head=64, E=1, k=1), True),
    (dict(B=4, T=300, d_model=512, nheads=4, d_head=64, E=5, k=3, qk_experts=1), False),
    (dict(B=2, T=300, d_model=412, nheads=2, d_head=76, E=5, k=3, dtype="f32"), False),
])
def test_dx_in_the_place_of_dy(over, dense):
    """dx written over dy (square attention): the same gradients as with buffers of their own."""
    cfg = _cfg(**over)
    t = make_inputs(cfg, seed=101)
    runs = []
    for alias in (False, True):
        layer = _layer(cfg, t, dense)
        if alias:
            layer.dx = layer.dy
        layer.forward()
        layer.backward()
        runs.append({n: v for n, v in layer.grads().items() if v is not None})
    for n, ref in runs[0].items():
        # (the same launches on the same values: what is not equal bit for bit was added atomically, in another order)
        e = nerr(runs[1][n], ref)
        assert e < 1e-5, (n, e)


@pytest.mark.parametrize("B", [4, 16])
@pytest.mark.parametrize("what", ["y", "dx"])
def test_heads_are_summed_in_fp32(B, what):
    """B x 512 tokens (whole 256-row tiles): y and dx are one fp32 accumulator over the heads, rounded once.  Two heads with the same
    router, queries, keys and (for y) values, whose output (for dx: value) experts are opposite up to one sixteenth: the sum is a
    sixteenth of what each head adds, so partial sums rounded to bf16 (2^-9 of a head's share each) would show as 2^-5 of the
    result, twice the bar and more; the accumulator leaves the rounding of the operands, which the two heads have in common."""
    cfg = _cfg(B=B, T=512, d_model=1024, nheads=2, d_head=128, E=5, k=3)
    t = make_inputs(cfg, seed=103)
    for n in ("W_S", "W_D"):
        t[n][:, cfg["E"]:] = t[n][:, :cfg["E"]]
    for n in ("W_Q", "W_K", "W_V", "W_O"):
        t[n][1] = t[n][0]
    other = "W_O" if what == "y" else "W_V"
    if what == "dx":   # the shares of the queries, keys and routers have nothing to cancel: keep them small
        for n in ("W_Q", "W_K", "W_S", "W_D"):
            t[n] = round_to_bf16(t[n] * np.float32(2.0 ** -8))
    noise = np.random.default_rng(5).standard_normal(t[other][1].shape).astype(np.float32) * np.std(t[other][0]) / 16
    t[other][1] = round_to_bf16(noise - t[other][0])
    layer = _layer(cfg, t)
    layer.forward()
    layer.backward()
    f = orc.forward(t["x"], t["W_Q"], t["W_K"], t["W_V"], t["W_O"], t["W_S"], t["W_D"], t["b_S"], t["b_D"], k=cfg["k"], causal=True)
    got, ref = layer.outputs(), f["y"]
    if what == "dx":
        got = layer.grads()["dx"]
        ref = orc.backward(t["x"], t["W_Q"], t["W_K"], t["W_V"], t["W_O"], t["W_S"], t["W_D"], f, t["dy"])["dx"]
    e = float(np.sqrt(np.sum((got - ref) ** 2) / np.sum(ref ** 2)))
    print("  %s relative error %.3e" % (what, e), flush=True)
    assert e < 1e-2


@pytest.mark.parametrize("nheads, E, k", [(8, 5, 3), (4, 9, 5)])
def test_many_narrow_heads_keep_the_expert_sets(nheads, E, k):
    """Two routers whose logits do not fit into one row of d_head (2 * 40 columns, heads of 64): dx cannot be one product over
    every (head, expert), so both passes run by expert sets, with sums in a fixed order and no accumulator to clear."""
    cfg = _cfg(B=10, T=520, d_model=2048, nheads=nheads, d_head=64, E=E, k=k)
    run_case(cfg, seed=107)
    layer = _layer(cfg, make_inputs(cfg, seed=107))
    steps = _steps(layer)
    assert "fwd.y_sum" in steps and not steps & {"fwd.y_zero", "fwd.y_cast", "bwd.dx_zero"}, steps
    first = layer.dx.clone()
    layer.dx.zero_()
    layer.backward()
    assert bool((layer.dx == first).all())


def test_gates_scale_fp32_results_where_there_are_too_many_sets():
    """More expert sets (252) than the tables hold: the gate multiplies the fp32 result of a product, not an operand that is rounded
    to bf16 afterwards."""
    cfg = _cfg(B=6, T=1000, d_model=2048, nheads=4, d_head=128, E=10, k=5)
    run_case(cfg, seed=109)
    got = _steps(_layer(cfg, make_inputs(cfg, seed=109)))
    assert {"fwd.y_cast", "bwd.v_dgrad"} <= got and "bwd.dx_gemm" not in got, got


@pytest.mark.parametrize("over, dense", [
    (dict(T=128, d_model=1024, nheads=4, d_head=128, E=10, k=5), False),     # 252 sets
    (dict(T=101, d_model=412, nheads=2, d_head=76, E=5, k=3), False),        # rows that make no set tables
    (dict(T=100, d_model=1024, nheads=4, d_head=128, E=5, k=3), False),      # sets
    (dict(T=60, T_q=33, d_model=132, nheads=3, d_head=36, E=3, k=2), False),
    (dict(T=50, d_model=256, nheads=4, d_head=80, E=1, k=1), True),
])
def test_output_experts_of_a_few_rows_round_once(over, dense):
    """y from the layer's own read-outs and gates: gates on fp32 products, one fp32 sum over heads and experts, so the error is that of
    rounding the result to bf16 and no more (fp32 sums add 1e-6; a rounding of gate x read-out alone would make it 1.4 times that)."""
    cfg = _cfg(B=1, **over)
    t = make_inputs(cfg, seed=113)
    layer = _layer(cfg, t, dense)
    assert not _steps(layer) & {"fwd.y_sum", "fwd.y_zero", "fwd.y_cast"}
    ctx, r = layer.intermediates()["ctx"].astype(np.float64), layer.routing()
    idx, gate = (r["idx_D"], r["gate_D"]) if "idx_D" in r else (r["idx"][1], r["gate"][1])
    want = np.zeros((ctx.shape[0], cfg["d_model"]))
    for h in range(cfg["nheads"]):
        for j in range(cfg["k"]):
            for e in range(cfg["E"]):
                n = np.nonzero(idx[h, :, j] == e)[0]
                want[n] += gate[h, n, j, None].astype(np.float64) * (ctx[n, h] @ t["W_O"][h, e].astype(np.float64))
    rel = lambda v: float(np.sqrt(np.sum((v - want) ** 2) / np.sum(want ** 2)))
    e, once = rel(layer.outputs().reshape(want.shape)), rel(round_to_bf16(want.astype(np.float32)))
    print("  relative error %.3e, of the rounding alone %.3e" % (e, once), flush=True)
    assert e < 1.05 * once


@pytest.mark.parametrize("over, step", [
    (dict(T=17, d_model=100, nheads=8, d_head=256, E=4, k=1), "fwd.y_zero"),
    (dict(T=40, d_model=64, nheads=2, d_head=76, E=32, k=5), "fwd.y_zero"),
    (dict(T=6, d_model=412, nheads=10, d_head=96, E=5, k=3), "fwd.y_sum"),
    (dict(T=17, d_model=256, nheads=4, d_head=128, E=8, k=1), "fwd.y_sum"),
    (dict(T=100, d_model=1024, nheads=4, d_head=128, E=5, k=3), None),
    (dict(T=205, d_model=1024, nheads=4, d_head=112, E=16, k=8), None),
])
def test_output_experts_of_a_few_rows_leave_short_calls_to_the_other_paths(over, step):
    """Every expert is multiplied there: calls with many experts for those a token selects, or of narrow models, were slower."""
    cfg = _cfg(B=1, **over)
    got = _steps(_layer(cfg, make_inputs(cfg, seed=117)))
    assert got & {"fwd.y_sum", "fwd.y_zero"} == ({step} if step else set()), got


def _poison_one(t, n, h, e, i, j):
    t[n] = t[n].copy()
    t[n][h, e, i, j] = np.inf
    t[n][h, e, i + 1, j + 2] = np.nan


@pytest.mark.parametrize("over, shared", [
    (dict(dtype="f32", B=2, T=70, d_model=50, nheads=2, d_head=20, E=4, k=2), False),
    (dict(dtype="f32", B=2, T=70, d_model=412, nheads=2, d_head=76, E=5, k=3, T_q=41), False),
    (dict(B=1, T=70, d_model=412, nheads=2, d_head=76, E=5, k=3), False),                # a few rows, of 8 bytes
    (dict(B=1, T=100, d_model=1024, nheads=4, d_head=128, E=5, k=3), False),             # ... and of 16
    (dict(B=5, T=1161, d_model=2048, nheads=2, d_head=64, E=3, k=2), False),             # a last tile of 173 rows
    (dict(B=5, T=1160, T_q=1000, d_model=2048, nheads=2, d_head=64, E=3, k=2), True),    # two token sets
    (dict(B=5, T=1161, d_model=2048, nheads=2, d_head=64, E=3, k=2, qk_experts=1), False),
])
def test_experts_that_a_token_did_not_select_do_not_reach_it(over, shared):
    """Infinities and NaNs in experts nobody selects leave no trace; in an output expert they reach only the tokens that
    selected it."""
    cfg = _cfg(**over)
    t = make_inputs(cfg, seed=127, shared_router=shared)
    HE, E = cfg["nheads"] * cfg["E"], cfg["E"]
    t["b_S"] = np.zeros(HE, np.float32)
    t["b_S"][E + 1] = -40.0                       # head 1, expert 1: nobody
    t["b_D"] = None if shared else t["b_S"].copy()
    layer = _layer(cfg, t)
    layer.forward()
    layer.backward()
    y, g = layer.outputs(), layer.grads()
    bad = dict(t)
    for n in ("W_V", "W_O") + (("W_Q", "W_K") if cfg["qk_experts"] else ()):
        _poison_one(bad, n, 1, 1, 3, 5)
    layer = _layer(cfg, bad)
    layer.forward()
    layer.backward()
    bar = 1e-5 if cfg["dtype"] == "f32" else 4e-3   # (elements summed in another order: bf16 results may move by one rounding, 2^-8)
    assert nerr(layer.outputs(), y) < bar
    for n, v in layer.grads().items():
        if v is not None:
            assert np.isfinite(v).all() and nerr(v, g[n]) < bar, n
    _poison_one(bad, "W_O", 0, 2, 4, 7)           # head 0, expert 2: some
    layer = _layer(cfg, bad)
    layer.forward()
    got, r = layer.outputs().reshape(-1, cfg["d_model"]), layer.routing()
    sel = (r["idx_D"] if "idx_D" in r else r["idx"][1])[0]
    hit = (sel == 2).any(-1)
    assert 0 < hit.sum() < hit.size
    want = y.reshape(-1, cfg["d_model"])
    assert nerr(got[~hit], want[~hit]) < bar
    ok = np.isfinite(got[hit])
    assert not ok[:, [7, 9]].any() and np.delete(ok, [7, 9], 1).all()


@pytest.mark.parametrize("d_model, d_head", [(50, 20), (76, 36), (33, 17)])
def test_fp32_infinities_past_the_end_of_a_reduction(d_model, d_head):
    """The row that fills up the last step of a reduction is a repeat; an infinity in it stays an infinity of its own place."""
    cfg = _cfg(dtype="f32", B=1, T=45, d_model=d_model, nheads=2, d_head=d_head, E=4, k=2)
    t = make_inputs(cfg, seed=131)
    t["W_K"][0, 0, 3] = np.inf            # the first of d_model reduction indices
    layer = _layer(cfg, t)
    layer.forward()
    assert np.array_equal(layer.intermediates()["K"][:, 0, 3], np.where(t["x"][0, :, 0] > 0, np.inf, -np.inf))
    t = make_inputs(cfg, seed=131)
    t["dy"][0, -1, 5] = np.inf            # the last token: the last row of every group it belongs to
    layer = _layer(cfg, t)
    layer.forward()
    layer.backward()
    got, inter, r = layer.grads()["dW_O"], layer.intermediates(), layer.routing()
    for h in range(cfg["nheads"]):
        for e in range(cfg["E"]):
            col = got[h, e, :, 5]
            if e in r["idx"][1][h, -1]:
                assert np.array_equal(col, np.where(inter["ctx"][-1, h] > 0, np.inf, -np.inf)), (h, e)
            else:
                assert np.isfinite(col).all(), (h, e)


@pytest.mark.parametrize("d_head", [20, 21, 76])
def test_fp32_causal_queries_do_not_meet_what_lies_far_behind_them(d_head):
    """NaNs and infinities in later tokens: under the causal mask the queries of earlier blocks of 32, and the keys and values
    that only later queries with bad gradients do not see, keep their results."""
    cfg = _cfg(dtype="f32", B=1, T=150, d_model=64, nheads=2, d_head=d_head, E=4, k=2)
    t = make_inputs(cfg, seed=137)
    base = _layer(cfg, t)
    base.forward()
    base.backward()
    y, g, want = base.outputs(), base.grads(), base.intermediates()
    for first in (32, 100):                                # the first bad token; its block of 32 starts at `clean`
        clean = first // 32 * 32
        bad = dict(t, x=t["x"].copy())
        bad["x"][0, first:] = np.inf
        bad["x"][0, first + 1::2] = np.nan
        layer = _layer(cfg, bad)
        layer.forward()
        assert nerr(layer.outputs()[:, :clean], y[:, :clean]) < 1e-6
        assert nerr(layer.intermediates()["ctx"][:clean], want["ctx"][:clean]) < 1e-6
    # queries before an owned block of keys never see it: their gradients must not reach it
    bad = dict(t, dy=t["dy"].copy())
    bad["dy"][0, :10] = np.nan
    layer = _layer(cfg, bad)
    layer.forward()
    layer.backward()
    assert nerr(layer.grads()["dx"][:, 32:], g["dx"][:, 32:]) < 1e-5


def test_fp32_sort_tables_too_large_for_the_in_block_scan():
    """The fp64 router's scan and scatter over a count table of 32-token blocks: 259 blocks of 64 experts, past what one block scans."""
    run_case(_cfg(dtype="f32", B=82, T=101, d_model=16, nheads=1, d_head=8, E=64, k=2), seed=139)


def test_bf16_two_token_sets_with_sort_tables_too_large_for_the_in_block_scan():
    """533 blocks of 126 expert sets on one side and 22 on the other: both are summed in a launch of their own."""
    run_case(_cfg(B=34, T=501, T_q=20, d_model=64, nheads=1, d_head=32, E=9, k=4), seed=149)


@pytest.mark.parametrize("over, atomic", [
    (dict(dtype="f32", B=16, T=256, d_model=412, nheads=2, d_head=76, E=5, k=3), ("db_S", "db_D")),   # several chunks, their partial sums in order
    (dict(B=4, T=700, T_q=350, d_model=1024, nheads=4, d_head=128, E=5, k=3), ("db_S", "db_D")),      # two token sets, all weight gradients in one launch
    (dict(B=9, T=300, d_model=1024, nheads=4, d_head=128, E=5, k=3), ()),
    (dict(B=9, T=300, d_model=1024, nheads=4, d_head=128, E=5, k=3, qk_experts=1), ()),
    (dict(dtype="f32", B=2, T=100, d_model=412, nheads=2, d_head=76, E=5, k=3, T_q=60), ()),        # at most 256 tokens
])
def test_gradients_repeat_bit_for_bit(over, atomic):
    """What the header promises to repeat; `atomic` are the ones it does not."""
    cfg = _cfg(**over)
    layer = _layer(cfg, make_inputs(cfg, seed=151))
    layer.forward()
    y = layer.outputs()
    layer.backward()
    first = layer.grads()
    for _ in range(3):
        layer.forward()
        layer.backward()
        assert np.array_equal(layer.outputs(), y)
        for n, v in layer.grads().items():
            if v is not None and n not in atomic:
                assert np.array_equal(v, first[n]), n


@pytest.mark.parametrize("over", [dict(T=1161), dict(T=1160, T_q=1000), dict(T=1161, qk_experts=1),
                                  dict(B=6, T=1000, T_q=961, qk_experts=1)])
def test_gated_forms_are_taken(over):
    """The shapes that the parity test of the gated concatenation relies on do run it, in both passes."""
    cfg = _cfg(**dict(dict(B=5, d_model=2048, nheads=2, d_head=64, E=3, k=2), **over))
    steps = _steps(_layer(cfg, make_inputs(cfg, seed=157)))
    assert "bwd.dx_gemm" in steps and not steps & {"fwd.y_sum", "fwd.y_zero"}, steps


def test_fp32_more_sequences_and_heads_than_one_grid_dimension_holds():
    """65535 sequences of one token with 260 heads: 17 million (sequence, head) pairs of 256 threads pass 2^32.  With a single key the
    read-out is the value row, and queries and keys get no gradient."""
    import torch
    cfg = _cfg(dtype="f32", B=65535, T=1, d_model=4, nheads=260, d_head=4, E=1, k=1)
    layer = _layer(cfg, make_inputs(cfg, seed=163), dense=True)
    layer.forward()
    layer.backward()
    V, ctx = (torch.empty((65535, 260, 4), device=layer.dev) for _ in range(2))
    from paper_2312_07987_amd import binding
    binding.switchhead_get_intermediates(layer.shape, layer.ws, None, None, V, ctx, None)
    assert bool((ctx - V).abs().max() <= 1e-6 * V.abs().max())
    assert float(layer.dW["W_Q"].abs().max()) < 1e-3 and float(layer.dW["W_K"].abs().max()) < 1e-3
    want = torch.einsum("nhd,nm->hdm", V.double(), layer.dy[:, 0].double())
    assert float((layer.dW["W_O"][:, 0].double() - want).abs().max()) < 1e-4 * float(want.abs().max())
