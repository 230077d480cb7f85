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
])
def test_fp32_tiles(over, shared):
    run_case(_cfg(dtype="f32", **over), shared=shared, seed=211)
