"""The work that users of the layer have it do, as cases that can be timed: training steps
(forward + backward), evaluation and prompt forwards and single-query decoding, in both storage types,
with the options of the layer that the paper's models use.

A case is a dict: the fields of the layer's shape (B, T, d_model, nheads, d_head, E, k, causal, dtype,
qk_experts, rope, T_q), `shared` (one router for both sides), `dense` (no routers, E = k = 1), `bias0`
(logit bias on expert 0 of every head), and
`call`: "train" (forward, then backward), "forward", or "forward_static" (the library's built-in workspace).
"""
import torch

from paper_2312_07987_amd import binding
from paper_2312_07987_amd.flops import layer_flops

# (d_model, nheads, d_head, E, k) of the layers that the package's workloads, tests and benchmark run
LAYER_47M = (412, 2, 76, 5, 3)
LAYER_47M_WIDE = (412, 3, 112, 5, 3)      # MAC-matched head shape
LAYER_47M_ROPE = (412, 2, 64, 5, 3)
LAYER_262M = (1024, 4, 128, 5, 3)
LAYER_262M_E8 = (1024, 4, 128, 8, 2)
LAYER_262M_ROPE = (1024, 4, 100, 4, 2)
DENSE_47M = (412, 10, 48, 1, 1)
DENSE_262M = (1024, 20, 80, 1, 1)
DENSE_262M_WIDE = (1024, 4, 256, 1, 1)

# a drawn case stays below the largest listed call of its storage type
MAX_TOKENS = 32768
MAX_FLOPS = 7e11
MAX_F32_TOKENS = 4096


def _case(layer, B, T, call, dtype="bf16", **options):
    d_model, nheads, d_head, E, k = layer
    case = dict(B=B, T=T, d_model=d_model, nheads=nheads, d_head=d_head, E=E, k=k, causal=True, dtype=dtype,
                qk_experts=False, rope=False, T_q=0, shared=False, dense=False, bias0=0.0, call=call)
    case.update(options)
    return case


def listed():
    named = {
        # a unit test or a toy model in fp32: nothing but launches and latency
        "tiny_f32_train": _case((64, 2, 32, 4, 2), 2, 64, "train", dtype="f32"),
        # training the 47M model's layer in fp32, a quarter of its batch
        "47m_f32_train": _case(LAYER_47M, 16, 256, "train", dtype="f32"),
        # one short prompt through the 262M model's layer, from a serving loop that allocates nothing
        "prompt_forward": _case(LAYER_262M, 1, 100, "forward_static"),
        # the next token of eight running sequences over a cached context
        "decode_forward": _case(LAYER_262M, 8, 1000, "forward", T_q=1),
        # a training step of the 47M model's layer
        "47m_train": _case(LAYER_47M, 64, 256, "train"),
        # a training step of the 262M-scale layer: the benchmark's default workload
        "262m_train": _case(LAYER_262M, 32, 512, "train"),
        # long sequences, more experts: the attention-heavy training step
        "long_train": _case(LAYER_262M_E8, 4, 4096, "train"),
        # evaluation with a skewed routing (one expert takes nearly every token)
        "skewed_forward": _case(LAYER_262M, 32, 512, "forward", bias0=3.0),
        # a fine-tuning step on a few sequences of a length that fits no tile
        "ragged_train": _case(LAYER_262M, 9, 701, "train"),
        # Transformer-XL training: a context of twice the chunk
        "context_train": _case(LAYER_262M, 32, 1024, "train", T_q=512),
        # every projection a mixture of experts
        "all_experts_train": _case(LAYER_262M, 32, 512, "train", qk_experts=True),
        # the rotary 244M-scale layer with one selection for both sides
        "rope_shared_train": _case(LAYER_262M_ROPE, 4, 1024, "train", rope=True, shared=True),
    }
    return [dict(case, name=name) for name, case in named.items()]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    while True:
        kind = rng.choice(("f32", "prompt", "decode", "forward", "train", "train", "train", "context"))
        if kind == "f32":
            layer = rng.choice(((64, 2, 32, 4, 2), LAYER_47M, LAYER_47M_ROPE))
            T = _log_int(rng, 33, 512)
            case = _case(layer, max(1, _log_int(rng, 64, MAX_F32_TOKENS) // T), T, rng.choice(("train", "train", "forward")),
                         dtype="f32")
        elif kind == "prompt":
            case = _case(LAYER_262M, 1, _log_int(rng, 16, 128), "forward_static")
        elif kind == "decode":
            T = _log_int(rng, 128, 4096)
            case = _case(rng.choice((LAYER_47M, LAYER_262M, LAYER_262M_E8)), max(1, _log_int(rng, 256, 16384) // T), T, "forward",
                         T_q=rng.choice((1, 1, 4)))
        else:
            layer = rng.choice((LAYER_47M, LAYER_47M_WIDE, LAYER_262M, LAYER_262M, LAYER_262M, LAYER_262M_E8, LAYER_262M_ROPE,
                                DENSE_47M, DENSE_262M, DENSE_262M_WIDE))
            T = _log_int(rng, 100, 4096)
            case = _case(layer, max(1, _log_int(rng, 500, 20000) // T), T, "forward" if kind == "forward" else "train")
            if kind == "context":
                case["T_q"] = max(1, T // 2)
            if layer[3] == 1:
                case["dense"] = True
            else:
                option = rng.choice(("none", "none", "none", "shared", "skewed", "all_experts"))
                if option == "shared":
                    case["shared"] = True
                elif option == "skewed":
                    case["bias0"] = 3.0
                elif option == "all_experts":
                    case["qk_experts"] = True
            case["rope"] = rng.random() < 0.2
            case["causal"] = rng.random() < 0.85
        if case["B"] * case["T"] <= MAX_TOKENS and work(case)["flops"] <= MAX_FLOPS:
            return case


def _shape(case):
    return binding.make_shape(case["B"], case["T"], case["d_model"], case["nheads"], case["d_head"], case["E"], case["k"],
                              case["causal"], case["dtype"], case["qk_experts"], case["rope"], case["T_q"])


def prepare(case, seed):
    """x, dy and the weights as the package's own synthetic inputs have them (x, dy ~ N(0, 1), weights scaled by the
    square root of what they reduce over), the outputs' buffers and the workspace."""
    B, T, dm, H, dh, E = (case[n] for n in ("B", "T", "d_model", "nheads", "d_head", "E"))
    Tq = case["T_q"] or T
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, std):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)

    state = {"call": case["call"], "shape": _shape(case)}
    qk = (H, E, dm, dh) if case["qk_experts"] else (H, dm, dh)
    state["x"] = normal((B, T, dm), 1.0)
    weights = {"W_Q": normal(qk, dm ** -0.5), "W_K": normal(qk, dm ** -0.5), "W_V": normal((H, E, dm, dh), dm ** -0.5),
               "W_O": normal((H, E, dh, dm), dh ** -0.5), "W_S": None, "W_D": None}
    if not case["dense"]:
        weights["W_S"] = normal((dm, H * E), dm ** -0.5)
        if not case["shared"]:
            weights["W_D"] = normal((dm, H * E), dm ** -0.5)
    state["weights"] = list(weights.values())
    bias = {"b_S": None, "b_D": None}
    if case["bias0"]:
        for name, router in (("b_S", "W_S"), ("b_D", "W_D")):
            if weights[router] is not None:
                bias[name] = torch.zeros(H * E, device="cuda")
                bias[name][::E] = case["bias0"]
    state["bias"] = list(bias.values())
    state["y"] = torch.empty((B, Tq, dm), dtype=dtype, device="cuda")
    state["outputs"] = {"y": state["y"]}
    if case["call"] != "forward_static":
        state["workspace"] = torch.empty(binding.switchhead_workspace_bytes(state["shape"]), dtype=torch.uint8, device="cuda")
    if case["call"] == "train":
        state["dy"] = normal((B, Tq, dm), 1.0)
        state["dx"] = torch.empty_like(state["x"])
        grads = {"d" + n: None if w is None else torch.empty(w.shape, dtype=torch.float32, device="cuda")
                 for n, w in {**weights, **bias}.items()}
        state["grads"] = list(grads.values())
        state["outputs"].update({"dx": state["dx"], **{n: g for n, g in grads.items() if g is not None}})
    return state


def run(state):
    shape, x, weights, bias, y = state["shape"], state["x"], state["weights"], state["bias"], state["y"]
    if state["call"] == "forward_static":
        binding.switchhead_forward_static(shape, x, *weights, *bias, y)
    else:
        binding.switchhead_forward(shape, x, *weights, *bias, y, state["workspace"])
    if state["call"] == "train":
        binding.switchhead_backward(shape, x, *weights, state["dy"], state["workspace"], state["dx"], *state["grads"])
    return state["outputs"]


def work(case):
    """flops: the selected experts' products, the routers and the visible half of the attention (the package's own work model).
    bytes: every input read once, every output written once; a training step reads x and the weights once for both passes."""
    B, T, dm, H, dh, E = (case[n] for n in ("B", "T", "d_model", "nheads", "d_head", "E"))
    Tq = case["T_q"] or T
    size = 2 if case["dtype"] == "bf16" else 4
    flops = layer_flops(B, T, dm, H, dh, E, case["k"], causal=case["causal"], shared=case["shared"], dense=case["dense"],
                        qk_experts=case["qk_experts"], T_q=case["T_q"])
    weights = H * dm * dh * (2 * (E if case["qk_experts"] else 1) + 2 * E)
    if not case["dense"]:
        weights += dm * H * E * (1 if case["shared"] else 2)
    nbytes = size * (B * T * dm + B * Tq * dm + weights)
    if case["call"] == "train":
        nbytes += size * (B * T * dm + B * Tq * dm) + 4 * weights
    return {"bytes": nbytes, "flops": flops["fwd_bwd" if case["call"] == "train" else "fwd"]}


def tolerance(case):
    """Four times what was measured: fp32 storage against the float64 oracle is off by up to 1.0e-6 (weight gradients over
    4096 tokens); bf16 storage on the matrix-core kernels against the plain fp32-arithmetic kernels by up to 4.2e-3."""
    return {"rel": 4e-6 if case["dtype"] == "f32" else 1.6e-2}
