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
