"""What the speed of this framework is measured on: passes through the MoE FFN layer's public entry points.

Two paths:
  train   a training step of the layer: index build, forward, backward, with the routing choice and the gates
          in hand, into buffers that the training program keeps (what bench.py's step does);
  infer   a serving pass: router logits -> routing choice and gates, index build, forward.

A case is a dict of plain values: path, T tokens, d_model, d_ff, E experts, top-k, dtype, activation and the
routing recipe (see paper_2411_01288_amd/workloads.py; "infer" draws logits and lets the library route).
"""
import math

import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate

ACTIVATIONS = {"gelu": B.ACT_GELU_TANH, "relu": B.ACT_RELU, "silu": B.ACT_SILU}


def _case(name, path, T, d, f, E, k, dtype, routing, activation="gelu"):
    return {"name": name, "path": path, "T": T, "d_model": d, "d_ff": f, "E": E, "k": k, "dtype": dtype,
            "routing": routing, "activation": activation}


def listed():
    return [
        # the smallest training step: the fp32 configuration for precision checks (launches and host time count)
        _case("train-f32-tiny", "train", 256, 64, 256, 4, 1, "f32", "uniform_top1"),
        # fp32 sizes that are no multiple of anything, few experts, ReLU
        _case("train-f32-odd", "train", 1001, 90, 362, 5, 2, "f32", "topk", "relu"),
        # fp32 training at the size of a small vision model's layer (4 images of 32x32 patches)
        _case("train-f32-mid", "train", 4096, 384, 1536, 8, 2, "f32", "topk"),
        # ragged bf16 sizes: odd token count, feature sizes that are no multiple of a tile, skewed top-3, SiLU
        _case("train-bf16-ragged", "train", 3001, 320, 448, 17, 3, "bf16", "zipf", "silu"),
        # the small vision layer in bf16
        _case("train-bf16-small", "train", 4096, 384, 1536, 8, 2, "bf16", "topk"),
        # ordinary training steps: 32 images under Zipf-skewed routing; 64 images with half of the tokens on one
        # expert and four empty ones; fp16
        _case("train-bf16-zipf", "train", 32768, 768, 3072, 16, 2, "bf16", "zipf"),
        _case("train-f16-medium", "train", 16384, 1024, 4096, 32, 2, "f16", "bias"),
        _case("train-bf16-forced", "train", 65536, 1024, 4096, 32, 1, "bf16", "forced"),
        # the largest training step (the headline configuration)
        _case("train-bf16-large", "train", 131072, 2048, 8192, 64, 2, "bf16", "bias"),
        # serving: decode steps of a small and of a large layer, prefill of a middling one
        _case("infer-bf16-decode-small", "infer", 16, 768, 3072, 16, 2, "bf16", "bias"),
        _case("infer-bf16-decode-large", "infer", 64, 2048, 8192, 64, 2, "bf16", "bias"),
        _case("infer-bf16-prefill", "infer", 8192, 1024, 4096, 32, 2, "bf16", "bias"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# The most a drawn case may hold: the largest listed case's arithmetic and activations; fp32 training stays at
# the sizes of precision checks and small models (an eighth of a TFLOP).
_MOST_FLOPS = {"bf16": 12.0 * 131072 * 2 * 2048 * 8192, "f16": 12.0 * 131072 * 2 * 2048 * 8192, "f32": 1.25e11}
_MOST_ACT = 131072 * 2 * 8192
_MOST_WEIGHTS = 64 * 2048 * 8192


def draw(rng):
    while True:
        dtype = rng.choice(("bf16", "bf16", "bf16", "f16", "f32"))
        path = rng.choice(("train", "train", "infer"))
        if dtype == "f32":
            T = _log_int(rng, 1 if path == "infer" else 64, 8192)
            d = _log_int(rng, 16, 512)
            f = _log_int(rng, 32, 2048)
            E = _log_int(rng, 1, 16)
        else:
            T = _log_int(rng, 1, 16384) if path == "infer" else _log_int(rng, 256, 131072)
            d = 64 * _log_int(rng, 1, 32)
            f = 4 * d if rng.random() < 0.5 else 64 * _log_int(rng, 1, 128)
            E = _log_int(rng, 1, 64)
        k = min(E, rng.choice((1, 1, 2, 2, 2, 3, 4, 8)))
        routing = rng.choice(("topk", "bias", "zipf")) if path == "train" else "bias"
        activation = rng.choice(("gelu", "gelu", "silu", "relu"))
        if (12.0 * T * k * d * f <= _MOST_FLOPS[dtype] and T * k * f <= _MOST_ACT and E * d * f <= _MOST_WEIGHTS
                and f <= 8192):
            c = _case("", path, T, d, f, E, k, dtype, routing, activation)
            del c["name"]
            return c


def prepare(case, seed):
    dev = torch.device("cuda:0")
    w = MoEWorkload("case", case["T"], case["d_model"], case["d_ff"], case["E"], case["k"], case["dtype"],
                    case["routing"], int(seed))
    data = generate(w, dev)
    shape = B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype, ACTIVATIONS[case["activation"]])
    s = {"path": case["path"], "shape": shape, "data": data,
         "idx": B.alloc_idx(shape, dev),
         "scratch": torch.empty(max(B.index_scratch_bytes(shape), 256), dtype=torch.uint8, device=dev),
         "ws": B.alloc_workspace(shape, dev)}
    if case["path"] == "infer":
        # router logits: the recipe of the "bias" routing, some experts preferred by all tokens
        gen = torch.Generator(device=dev)
        gen.manual_seed(int(seed) + 1)
        beta = 0.5 * torch.randn((1, w.E), generator=gen, device=dev)
        s["logits"] = torch.randn((w.T, w.E), generator=gen, device=dev) + beta
        del data["dY"]
    else:
        E, d, f = w.E, w.d_model, w.d_ff
        f32 = dict(dtype=torch.float32, device=dev)
        s["y"] = torch.empty_like(data["x"])
        s["out"] = {"dx": torch.empty_like(data["x"]), "dW1": torch.empty((E, d, f), **f32),
                    "db1": torch.empty((E, f), **f32), "dW2": torch.empty((E, f, d), **f32),
                    "db2": torch.empty((E, d), **f32), "dgate": torch.empty((w.T, w.k), **f32)}
    return s


def run(state):
    shape, data, idx, ws = state["shape"], state["data"], state["idx"], state["ws"]
    if state["path"] == "infer":
        topk_idx, gate = B.hexa_moe_route(shape, state["logits"])
        B.hexa_moe_index(shape, topk_idx, idx, state["scratch"])
        y = B.hexa_moe_fwd(shape, data["x"], topk_idx, gate, data["W1"], data["b1"], data["W2"], data["b2"],
                           idx, ws)
        return {"y": y, "topk_idx": topk_idx, "gate": gate}
    topk_idx, gate = data["topk_idx"], data["gate"]
    B.hexa_moe_index(shape, topk_idx, idx, state["scratch"])
    y = B.hexa_moe_fwd(shape, data["x"], topk_idx, gate, data["W1"], data["b1"], data["W2"], data["b2"], idx,
                       ws, state["y"])
    grads = B.hexa_moe_bwd(shape, data["dY"], data["x"], topk_idx, gate, data["W1"], data["W2"], idx, ws,
                           out=state["out"])
    return {"y": y, "perm": idx["perm"], "offsets": idx["offsets"], **grads}


def work(case):
    T, d, f, E, k = (case[n] for n in ("T", "d_model", "d_ff", "E", "k"))
    es = 4 if case["dtype"] == "f32" else 2
    A = T * k
    # experts that some token chooses, on average
    used = E * (1.0 - (1.0 - k / E) ** T)
    weights = used * (2 * d * f + d + f) * es
    if case["path"] == "infer":
        # logits, x, the used experts' weights in; choice, gates, y out; two contractions
        return {"bytes": T * E * 4 + 2 * T * d * es + weights + A * 8, "flops": 4.0 * A * d * f}
    # x, dY, weights, choice and gates in; y, dx, the index (perm), dgate and all experts' fp32 gradients out; six contractions
    return {"bytes": 4 * T * d * es + weights + A * 16 + E * (2 * d * f + d + f) * 4.0, "flops": 12.0 * A * d * f}


def tolerance(case):
    # Relative 2-norm error of the worst output.  Against the layer in fp64 on the same inputs the worst output
    # of the listed cases (dx) is off by 8.2e-7 in fp32 and 3.7e-3 in bf16 (two roundings of intermediates to
    # 2^-9 and one of the result), an eighth of that in fp16; stated is about four times as much.
    return {"rel": {"f32": 4e-6, "bf16": 1.5e-2, "f16": 2e-3}[case["dtype"]]}
