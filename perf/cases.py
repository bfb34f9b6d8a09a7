"""The work this framework is used for, as cases that can be timed and compared.

A case is one operator DAG with one executor.  `prepare` does what a program that serves
the model does once: it describes the DAG, binds it to device buffers (`Session`), puts
weights and inputs into them and captures the executor.  `run` is one inference as such a
program issues it: `Session.replay`, which launches the captured graph and waits for it,
after which the outputs can be read from the session's buffers.

Weights and inputs are drawn on the GPU from the seed, with the deviations the models have
in earnest: convolutions sqrt(2 / fan-in) so that activations of the deep networks stay at
order one, transformer weights 0.02, inputs N(0, 1), small non-zero biases.
"""
import math
from unittest import mock

import torch

from paper_2312_10351_amd import binding as B
from paper_2312_10351_amd.runtime import Session
from workloads import (Builder, Workload, bert_base_like, googlenet_like, inception_block, inception_v3_like,
                       nasnet_like, random_small_dag, random_wide_dag)


def listed():
    return [
        # The smallest DAG anybody runs: one four-branch block in fp32.  Launch latency counts.
        {"name": "block_f32", "model": "block", "dtype": "f32", "batch": 1, "mode": "fused"},
        # The headline network, one image at a time.
        {"name": "googlenet_f16", "model": "googlenet", "dtype": "f16", "batch": 1, "mode": "fused"},
        # The same network through the multi-stream graph, the executor of the paper.
        {"name": "googlenet_f16_streams", "model": "googlenet", "dtype": "f16", "batch": 1, "mode": "streams"},
        # The same network for users who keep fp32.
        {"name": "googlenet_f32", "model": "googlenet", "dtype": "f32", "batch": 1, "mode": "fused"},
        # A deeper image network: asymmetric filters, 17 x 17 and 35 x 35 images.
        {"name": "inception_f16", "model": "inception", "dtype": "f16", "batch": 1, "mode": "fused"},
        # ... serving a batch of images (throughput).
        {"name": "inception_f16_b16", "model": "inception", "dtype": "f16", "batch": 16, "mode": "fused"},
        # A transformer encoder at its ordinary length,
        {"name": "bert_s128", "model": "bert", "dtype": "f16", "seq": 128, "layers": 12, "hidden": 768, "mode": "fused"},
        # ... at the length a sentence happens to have (no multiple of any vector or tile),
        {"name": "bert_s77", "model": "bert", "dtype": "f16", "seq": 77, "layers": 12, "hidden": 768, "mode": "fused"},
        # ... and at the longest input such a model takes.
        {"name": "bert_s512", "model": "bert", "dtype": "f16", "seq": 512, "layers": 12, "hidden": 768, "mode": "fused"},
        # An irregular cell network: many small operators per level.
        {"name": "nasnet_f16", "model": "nasnet", "dtype": "f16", "batch": 1, "cells": 6, "width": 32, "hw": 28, "mode": "fused"},
        # Irregular wiring with tiny operators: what is left is the cost of the executor.
        {"name": "small_dag_f16", "model": "small_dag", "dtype": "f16", "n_ops": 60, "wiring": 7, "mode": "fused"},
        # The heaviest workload: 400 operators, large GEMMs beside streaming operators.
        {"name": "wide_dag_f16", "model": "wide_dag", "dtype": "f16", "n_ops": 400, "wiring": 231210355, "mode": "fused"},
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    model = rng.choice(("block", "googlenet", "inception", "bert", "bert", "nasnet", "small_dag", "wide_dag"))
    if model == "bert":
        return {"model": model, "dtype": "f16", "seq": _spread(rng, 16, 512), "layers": rng.randint(2, 12),
                "hidden": 64 * rng.randint(4, 12), "mode": rng.choice(("fused", "fused", "sequential"))}
    if model == "small_dag":
        return {"model": model, "dtype": rng.choice(("f16", "f32")), "n_ops": _spread(rng, 20, 200),
                "wiring": rng.randint(1, 1 << 20), "mode": rng.choice(("fused", "fused", "sequential"))}
    if model == "wide_dag":
        return {"model": model, "dtype": "f16", "n_ops": _spread(rng, 20, 300), "wiring": rng.randint(1, 1 << 20), "mode": "fused"}
    case = {"model": model, "dtype": rng.choice(("f16", "f16", "f32")), "mode": rng.choice(("fused", "fused", "sequential", "streams"))}
    most = {"block": 32, "googlenet": 16, "inception": 16, "nasnet": 4}[model]
    case["batch"] = _spread(rng, 2, most if case["dtype"] == "f16" else max(2, most // 8))
    if model == "nasnet":
        case.update(cells=rng.randint(2, 8), width=4 * _spread(rng, 3, 16), hw=_spread(rng, 10, 40))
    return case


def _structure(case):
    """The case's DAG.  Its tensors are placeholders without storage: `prepare` draws the
    real ones on the GPU."""
    import numpy as np

    def build(self, seed, random_bias=False, w_std=0.02, he_init=False):
        zero = np.zeros((), dtype=np.float32 if self.dtype == "f32" else np.float16)
        blank = lambda shape: np.broadcast_to(zero, shape)
        lead = lambda s: ((self.batch,) + s) if (self.batch > 1 and len(s) == 3) else s
        weights = {}
        for op in self.ops:
            p = op.params
            if op.type == "conv2d":
                weights[op.id] = {"w": blank((p["cout"], p["cin"], p["kh"], p["kw"])), "b": blank((p["cout"],))}
            elif op.type == "gemm":
                weights[op.id] = {"w": blank((p["k"], p["n"])), "b": blank((p["n"],))}
        return Workload(self.name, self.dtype, self.ops, [blank(lead(s)) for s in self.ext_shapes], weights, seed, self.batch)

    model, dtype = case["model"], case["dtype"]
    with mock.patch.object(Builder, "build", build):
        if model == "bert":
            return bert_base_like(dtype=dtype, layers=case["layers"], seq=case["seq"], hidden=case["hidden"],
                                  heads=case["hidden"] // 64, ffn=4 * case["hidden"])
        if model == "small_dag":
            return random_small_dag(case["wiring"], dtype=dtype, n_ops=case["n_ops"])
        if model == "wide_dag":
            return random_wide_dag(case["wiring"], dtype=dtype, n_ops=case["n_ops"])
        if model == "nasnet":
            return nasnet_like(dtype=dtype, cells=case["cells"], width=case["width"], hw=case["hw"], batch=case["batch"])
        return {"block": inception_block, "googlenet": googlenet_like, "inception": inception_v3_like}[model](dtype=dtype, batch=case["batch"])


class _Served:
    """A captured model: the session, its executor and the outputs its user reads."""

    def __init__(self, session, exe, outputs):
        self.session, self.exe, self.outputs = session, exe, outputs

    def __del__(self):
        self.session.close()


def _read_outputs(case, wl, session):
    """What a user reads after a pass: every sink of the DAG (logits, the results of a random
    DAG) and, for the networks, the features of every block: concatenated and pooled feature
    maps of the image networks, hidden states of the transformer."""
    ids = set(wl.sinks())
    if not case["model"].endswith("_dag"):
        ids.update(op.id for op in wl.ops if op.type in ("concat", "gavgpool", "layernorm"))
    ids = sorted(ids)
    return [session.out_dev[v] for v in ids[::-(-len(ids) // 32)]]      # at most 32, spread over the DAG


def prepare(case, seed):
    wl = _structure(case)
    s = Session(wl, zero_copy_concat=True)
    gen = torch.Generator(device=s.device).manual_seed(seed)
    for slot, t in enumerate(s.ext_dev):
        t.normal_(generator=gen)
        if slot in s.ext_pad:                      # channels appended for alignment hold zeros
            t[..., wl.ext_inputs[slot].shape[-3]:] = 0
    std = {"bert": 0.02, "wide_dag": 0.02, "small_dag": 0.1}.get(case["model"])
    for v, w in s.w_dev.items():
        op = wl.ops[v]
        fan_in = math.prod(wl.weights[v]["w"].shape[1:]) if op.type == "conv2d" else op.params["k"]
        w.normal_(0.0, std or math.sqrt(2.0 / fan_in), generator=gen)
        if op.type == "conv2d":
            w[..., op.params["cin"]:] = 0
        s.b_dev[v].normal_(0.0, 0.02, generator=gen)
    torch.cuda.synchronize()
    exe = s.capture({"fused": B.FUSED, "streams": B.PARALLEL, "sequential": B.SEQUENTIAL}[case["mode"]])
    return _Served(s, exe, _read_outputs(case, wl, s))


def run(state):
    state.session.replay(state.exe)
    return state.outputs


def work(case):
    """Inputs and weights read once, every operator's result written once (each is an output
    the session hands out); multiply-adds of the contractions."""
    wl = _structure(case)
    es = 4 if wl.dtype == "f32" else 2
    nbytes = sum(a.size for a in wl.ext_inputs) * es
    flops = 0
    for op in wl.ops:
        images = wl.batch if len(op.out_shape) == 3 else 1
        nbytes += math.prod(op.out_shape) * images * es
        p = op.params
        if op.id in wl.weights:
            w = wl.weights[op.id]["w"]
            nbytes += w.size * es + 4 * wl.weights[op.id]["b"].size
            flops += 2 * w.size * (op.out_shape[1] * op.out_shape[2] * images if op.type == "conv2d" else p["m"])
        elif op.type == "bgemm":
            flops += 2 * p["heads"] * p["seq"] * p["seq"] * p["dhead"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what other executors of the same DAG show, which add the same products in
    another order (wavefronts per tile, tile shapes): 8e-7 in fp32, 1.3e-3 in fp16 (one fp16
    rounding per operator, carried through the DAG); largest single difference 5e-6 and 9e-3."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 6e-3, "max": 4e-2}
