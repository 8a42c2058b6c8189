"""The work that the library's speed is judged by: its public entry points as a user's program calls
them, over the range of sizes, types and options in use.

listed() names twelve cases, draw() gives further ones of the same ranges, prepare() makes what a
program has in hand before the call, run() is one call, work() the bytes and operations it cannot do
without, tolerance() how far another correct implementation at the same precision may be off.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_01884_amd import binding as ff

EPS = 1e-5

# Ranges of the drawn cases.  A drawn case stays below the largest listed one in both of these.
MOST_MATRIX_FLOPS = 1.0e12       # bf16; fp32 runs on matrix units a sixteenth as fast
MOST_F32_FLOPS = 1.3e11
MOST_BYTES = 5.0e8


def listed():
    def linear(name, dtype, M, K, N, affine=True):
        return {"name": name, "kind": "linear", "dtype": dtype, "M": M, "K": K, "N": N, "affine": affine}

    return [
        # a small layer in full precision: latency, launches and host work
        linear("linear_f32_256x512x512", "f32", 256, 512, 512),
        # full precision at the size of a model's layer
        linear("linear_f32_4096", "f32", 4096, 4096, 4096),
        # one decode step of a small batch: the weights are read once, almost nothing else
        linear("linear_decode_16x8192x8192", "bf16", 16, 8192, 8192),
        # a decode step of a larger batch, or a short prompt: still bound by the weights
        linear("linear_batch_96x8192x8192", "bf16", 96, 8192, 8192),
        # a layer of a training step or of a prompt's prefill
        linear("linear_4096", "bf16", 4096, 4096, 4096),
        # many short rows: the epilogue weighs as much as the product
        linear("linear_65536x1024x1024", "bf16", 65536, 1024, 1024),
        # wide rows, the largest
        linear("linear_8192x4096x16384", "bf16", 8192, 4096, 16384),
        # sizes that no tile divides
        linear("linear_3001x2056x5000", "bf16", 3001, 2056, 5000),
        # linear, subtract, row mean, GELU, residual add
        {"name": "rowmean_4096", "kind": "rowmean", "dtype": "bf16", "M": 4096, "K": 4096, "N": 4096},
        # the loss of a classifier batch
        {"name": "xent_f32_32768x4096", "kind": "xent", "dtype": "f32", "B": 32768, "C": 4096},
        # the loss over a vocabulary of odd length, in half precision
        {"name": "xent_bf16_4096x50257", "kind": "xent", "dtype": "bf16", "B": 4096, "C": 50257},
        # selection of the profiling metrics of eight tasks, duplicates dropped
        {"name": "metrics_8x10x300", "kind": "metrics", "n": 8, "V": 10, "J": 300, "tau": 0.999},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, step):
    """A size in [lo, hi]: half the time of the round kind (a multiple of 256), else a multiple of `step`."""
    v = _log(rng, lo, hi)
    if hi >= 512 and rng.random() < 0.5:
        return min(hi, max(256, v // 256 * 256))
    return min(hi // step * step, max(step, v // step * step))


def draw(rng):
    kind = rng.choice(["decode", "batch", "layer", "layer", "layer", "f32", "f32", "rowmean", "xent", "xent", "metrics"])
    while True:
        if kind in ("decode", "batch", "layer", "f32"):
            dtype, step = ("f32", 4) if kind == "f32" else ("bf16", 8)
            if kind == "decode":
                M, K, N = _log(rng, 1, 32), _size(rng, 512, 16384, step), _size(rng, 512, 16384, step)
            elif kind == "batch":
                M, K, N = _log(rng, 33, 512), _size(rng, 512, 16384, step), _size(rng, 512, 16384, step)
            elif kind == "layer":
                M, K, N = _size(rng, 512, 65536, 1), _size(rng, 256, 8192, step), _size(rng, 256, 16384, step)
            else:
                M, K, N = _size(rng, 16, 8192, 1), _size(rng, 128, 4096, step), _size(rng, 128, 8192, step)
            case = {"kind": "linear", "dtype": dtype, "M": M, "K": K, "N": N, "affine": rng.random() < 0.8}
        elif kind == "rowmean":
            dtype, step = rng.choice([("bf16", 8), ("bf16", 8), ("f32", 4)])
            case = {"kind": "rowmean", "dtype": dtype, "M": _size(rng, 64, 16384, 1), "K": _size(rng, 256, 8192, step),
                    "N": _size(rng, 256, 16384, step)}
        elif kind == "xent":
            case = {"kind": "xent", "dtype": rng.choice(["f32", "bf16"]), "B": _size(rng, 256, 65536, 1),
                    "C": _size(rng, 16, 131072, 1)}
        else:
            case = {"kind": "metrics", "n": rng.randint(1, 12), "V": rng.randint(8, 64), "J": rng.randint(64, 1024),
                    "tau": rng.choice([0.0, 0.999])}
        w = work(case)
        flops = MOST_F32_FLOPS if case.get("dtype") == "f32" else MOST_MATRIX_FLOPS
        if w["bytes"] <= MOST_BYTES and w["flops"] <= flops:
            return case


def _element(case):
    return (torch.float32, 4) if case["dtype"] == "f32" else (torch.bfloat16, 2)


def prepare(case, seed):
    """Inputs as a model gives them: activations of unit variance, weights of variance 1/K, small biases,
    a scale around one; scores of unit variance with one class index a row; counters of any magnitude that
    follow the run time more or less."""
    if case["kind"] == "metrics":
        return _prepare_metrics(case, seed)
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g, dtype=torch.float32, device="cuda")

    def uniform(n):
        return torch.rand(n, generator=g, dtype=torch.float32, device="cuda") * 0.2 - 0.1

    dtype, _ = _element(case)
    if case["kind"] == "xent":
        return {"kind": "xent", "logits": normal(case["B"], case["C"]).to(dtype),
                "targets": torch.randint(0, case["C"], (case["B"],), generator=g, dtype=torch.int64, device="cuda")}
    M, K, N = case["M"], case["K"], case["N"]
    state = {"kind": case["kind"], "X": normal(M, K).to(dtype), "W": (normal(N, K) * float(K) ** -0.5).to(dtype),
             "b": uniform(N).to(dtype)}
    if case["kind"] == "rowmean":
        state["s"] = uniform(N).to(dtype)
    else:
        state["gamma"] = (1.0 + 0.1 * normal(N)).to(dtype) if case["affine"] else None
        state["beta"] = (0.1 * normal(N)).to(dtype) if case["affine"] else None
    return state


def _prepare_metrics(case, seed):
    n, V, J = case["n"], case["V"], case["J"]
    rng = np.random.default_rng(seed)
    runtime = np.exp(0.5 * rng.standard_normal((n, V)))
    z = (runtime - runtime.mean(axis=1, keepdims=True)) / runtime.std(axis=1, keepdims=True)
    follows = np.clip(rng.uniform(-1, 1, J) + 0.5 * rng.standard_normal((n, J)), -1, 1)
    values = follows[:, None, :] * z[:, :, None] + np.sqrt(1 - follows ** 2)[:, None, :] * rng.standard_normal((n, V, J))
    scale = 10.0 ** rng.uniform(0, 9, J)
    values = scale * (values + rng.uniform(0, 4, J))
    values[:, :, 16::17] = scale[16::17]                 # counters that never move
    values[:, :, 19::19] = values[:, :, 18:J - 1:19]     # counters that are another one under a second name
    return {"kind": "metrics", "tau": case["tau"], "values": torch.from_numpy(np.ascontiguousarray(values)).cuda(),
            "runtime": torch.from_numpy(runtime).cuda()}


def run(state):
    kind = state["kind"]
    if kind == "linear":
        return ff.ff_fused_linear_gelu_ln(state["X"], state["W"], state["b"], state["gamma"], state["beta"], EPS)
    if kind == "rowmean":
        return ff.ff_fused_linear_sub_rowmean_gelu_residual(state["X"], state["W"], state["b"], state["s"])
    if kind == "xent":
        mean, rows = ff.ff_cross_entropy_mean(state["logits"], state["targets"], with_rows=True)
        return {"mean": mean, "rows": rows}
    got = ff.ff_metric_selection(state["values"], state["runtime"], collinear_tau=state["tau"])
    selected = np.zeros(got["score"].shape, dtype=np.int64)
    selected[got["selected"]] = 1
    return {"r": got["r"], "score": got["score"], "threshold": got["threshold"],
            "top": np.array([m for row in got["top"] for m in row], dtype=np.int64), "selected": selected}


def work(case):
    """Inputs read once and outputs written once; products only, where there is a product."""
    kind = case["kind"]
    if kind == "metrics":
        n, V, J = case["n"], case["V"], case["J"]
        flops = 2.0 * n * V * J * (J / 2 if case["tau"] > 0 else 3)
        return {"bytes": 8.0 * (n * V * (J + 1) + n * J + J), "flops": flops}
    _, e = _element(case)
    if kind == "xent":
        return {"bytes": float(case["B"]) * (case["C"] * e + 8 + 4) + 4, "flops": 0.0}
    M, K, N = case["M"], case["K"], case["N"]
    if kind == "rowmean":
        return {"bytes": float(e) * (N * K + 2 * M * K + 2 * N), "flops": 0.0}
    vectors = 3 if case["affine"] else 1
    return {"bytes": float(e) * (M * K + N * K + M * N + vectors * N), "flops": 2.0 * M * K * N}


def tolerance(case):
    """About four times what the results of the listed cases differ by, at the most, from the same formula
    evaluated in 64 bits and rounded once to the type of the result: measured, 6.1e-5 and one unit in the
    last place (7.8e-3) in bf16; 1.5e-6 and 1.7e-5 in fp32; 4.5e-8 and 1.1e-7 for the losses, whose own
    rounding is as large (hence ten times); 2.6e-16 and 1e-15 for the correlations, where sums in another
    order differ by more on longer columns."""
    if case["kind"] == "metrics":
        return {"rel": 2e-15, "max": 2e-14}
    if case["kind"] == "xent":
        return {"rel": 5e-7, "max": 2e-6}
    return {"rel": 6e-6, "max": 7e-5} if case["dtype"] == "f32" else {"rel": 2.5e-4, "max": 3.2e-2}
