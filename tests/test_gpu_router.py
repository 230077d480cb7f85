"""The two-stage router of bf16 storage and the sorts behind it at the sizes where they change form: columns per router that are a
multiple of four, even or odd (how the router's rows are laid out in LDS) and on both sides of 12, 16 and 20; more than eight
experts (selection by passes); features that fill no K step, one trip or several; 8-byte rows of x; tokens that fill no
tile of 32; count tables past what one block scans, and past what a
wave sums in one step.  Indices, permutation and offsets are the float64 oracle's exactly; gates are
sigmoids of logits summed in fp32 over 64 features at a time (2e-5 bounds that many times over at these sizes)."""
import numpy as np
import pytest

from oracle import switchhead_oracle as orc
from paper_2312_07987_amd.inputs import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over, shared, ties", [
    (dict(T=1, d_model=4, nheads=1, E=1, k=1), False, False),
    (dict(T=33, d_model=68, nheads=3, E=3, k=1), False, True),
    (dict(T=77, d_model=412, nheads=2, E=5, k=3), False, True),
    (dict(T=300, d_model=1024, nheads=4, E=5, k=3), False, True),
    (dict(T=300, d_model=1020, nheads=4, E=5, k=3), True, False),
    (dict(T=95, d_model=1088, nheads=4, E=8, k=2), False, True),
    (dict(T=64, d_model=2100, nheads=2, E=7, k=5), False, True),
    (dict(T=130, d_model=512, nheads=2, E=9, k=4), False, True),
    (dict(T=96, d_model=260, nheads=1, E=31, k=8), False, True),
    (dict(T=70, d_model=1500, nheads=2, E=16, k=3), False, True),            # the second stage's 16 and 32 columns
    (dict(T=50, d_model=2052, nheads=1, E=17, k=8), False, True),
    (dict(T=40, d_model=520, nheads=1, E=32, k=8), True, False),
    (dict(T=513, T_q=65, d_model=1024, nheads=4, E=5, k=3), False, True),
    (dict(T=100, T_q=1, d_model=412, nheads=2, E=5, k=3), True, False),
    (dict(B=5, T=8000, d_model=16, nheads=1, E=9, k=4), False, False),
    (dict(B=3, T=3000, d_model=64, nheads=4, E=4, k=2), False, True),        # more than two tiles for each CU
    (dict(B=3, T=3000, d_model=20, nheads=4, E=4, k=2), True, False),
    (dict(B=3, T=2740, T_q=2733, d_model=36, nheads=2, E=5, k=3), False, False),
    (dict(T=100, d_model=4, nheads=3, E=9, k=4), False, True),               # more counts than partial sums of the heads
    (dict(B=3, T=43, d_model=16, nheads=2, E=9, k=4), False, True),          # short tables of 126 sets: summed in a launch of their own
    (dict(B=40, T=104, d_model=16, nheads=3, E=9, k=4), False, True),
    (dict(B=41, T=102, d_model=16, nheads=3, E=9, k=4), True, False),
    (dict(B=64, T=128, d_model=16, nheads=1, E=8, k=4), False, True),        # 256 blocks of 70 sets: the last size that a block scans
    (dict(B=11, T=745, d_model=16, nheads=1, E=8, k=4), True, False),        # and the next, 257
    (dict(B=9, T=3072, d_model=16, nheads=3, E=2, k=1), False, True),        # four trips of 1296 blocks: scanned by every one
    (dict(B=10, T=2940, d_model=16, nheads=3, E=2, k=1), False, True),       # ... of 1380: not
])
def test_routing_tables(over, shared, ties):
    from paper_2312_07987_amd.runner import DeviceLayer
    cfg = dict(name="router", dtype="bf16", B=2, d_head=4, causal=1, bias0=0.5)
    cfg.update(over)
    print("case", cfg, shared, ties, flush=True)
    t = make_inputs(cfg, seed=31 + cfg["d_model"], shared_router=shared)
    if ties:   # the first head's last expert repeats its first one's column
        for W in ("W_S", "W_D"):
            if t[W] is not None:
                t[W] = t[W].copy()
                t[W][:, cfg["E"] - 1] = t[W][:, 0]
        for b in ("b_S", "b_D"):
            if t[b] is not None:
                t[b] = t[b].copy()
                t[b][cfg["E"] - 1] = t[b][0]
    layer = DeviceLayer(cfg, t)
    layer.forward()
    r = layer.routing()
    T, Tq, k = cfg["T"], cfg.get("T_q") or cfg["T"], cfg["k"]
    x = t["x"].astype(np.float64)
    for side, W, b in (("S", t["W_S"], t["b_S"]), ("D", t["W_S"] if shared else t["W_D"], t["b_S"] if shared else t["b_D"])):
        rows = x if side == "S" else x[:, T - Tq:]
        idx, gate = orc.select_topk(orc.router_logits(rows.reshape(-1, cfg["d_model"]), W, b), cfg["nheads"], k)[:2]
        packed = side == "D" and Tq != T
        got = r["idx_D"] if packed else r["idx"]["SD".index(side)]
        assert np.array_equal(got, idx), side
        got = r["gate_D"] if packed else r["gate"]["SD".index(side)]
        assert np.max(np.abs(got - gate)) < 2e-5, side
        perm = r["perm_D"] if packed else r["perm"]["SD".index(side)]
        for h in range(cfg["nheads"]):
            want = orc.routing_tables(idx[h], cfg["E"])
            assert np.array_equal(perm[h], want[0]), (side, h)
            assert np.array_equal(r["offsets"]["SD".index(side)][h], want[1]), (side, h)
    assert np.isfinite(layer.outputs()).all()


def _first_of_the_largest(z, nheads, k):
    """k passes of "largest remaining logit, the lowest index on ties", where nothing is larger than a NaN that a pass begins with."""
    N, E = z.shape[0], z.shape[1] // nheads
    idx = np.zeros((nheads, N, k), np.int32)
    for h in range(nheads):
        for n in range(N):
            left = list(range(E))
            for j in range(k):
                best = left[0]
                for e in left[1:]:
                    if z[n, h * E + e] > z[n, h * E + best]:
                        best = e
                left.remove(best)
                idx[h, n, j] = best
    return idx


@pytest.mark.parametrize("E, k, columns, bias", [
    (3, 1, (1,), {}),                                    # 1, NaN, 2: every expert goes before one other
    (5, 1, (1,), {}),
    (8, 2, (1, 4), {}),
    (4, 2, (), {1: np.nan}),
    (5, 3, (), {0: np.inf, 3: np.inf, 4: -np.inf}),      # equal infinities
    (9, 2, (0, 5), {}),
    (12, 3, (), {2: np.nan, 7: np.inf}),
])
def test_logits_that_are_not_finite(E, k, columns, bias):
    """NaNs in a router's columns or bias, in tokens, infinities, logits that only fp32 cannot hold: every choice is still one of the
    experts, that of the serial rule, and the permutation is one."""
    from paper_2312_07987_amd.runner import DeviceLayer
    cfg = dict(name="router", dtype="bf16", B=1, T=75, d_model=68, nheads=3 if E < 9 else 2, d_head=8, E=E, k=k, causal=1, bias0=0.0)
    print("case", cfg, columns, bias, flush=True)
    H = cfg["nheads"]
    t = make_inputs(cfg, seed=47 + E)
    t["x"], t["W_S"] = t["x"].copy(), t["W_S"].copy()
    for c in columns:
        t["W_S"][9, E + c] = np.nan
    t["b_S"] = np.zeros(H * E, np.float32)
    for c, v in bias.items():
        t["b_S"][E + c] = v
    t["x"][0, 40] = np.nan
    t["x"][0, 41, ::2] = np.inf
    t["x"][0, 42] *= np.float32(2.0 ** 126)   # the sum of its squares is past the largest fp32
    layer = DeviceLayer(cfg, t)
    layer.forward()
    r = layer.routing()
    with np.errstate(all="ignore"):
        for side, W, b in ((0, "W_S", "b_S"), (1, "W_D", "b_D")):
            want = _first_of_the_largest(orc.router_logits(t["x"][0].astype(np.float64), t[W], t[b]), H, k)
            assert np.array_equal(r["idx"][side], want), side
            for h in range(H):
                perm, offsets = orc.routing_tables(want[h], E)[:2]
                assert np.array_equal(r["perm"][side][h], perm) and np.array_equal(r["offsets"][side][h], offsets), (side, h)
