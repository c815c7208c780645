"""Serving calls of the merged multi-task model as its users make them, for timing.

A case names a model of mt_synth (its shapes and task table), a precision, an entry point and the size of the call.  What a
server has in hand before a call is prepared once: the loaded model (kept per process, as a server keeps it), the requests' ids and
masks on the device, and the buffers that receive the logits.  One pass is one call of the entry point.

Weights are random (matrices N(0, 0.02), biases and LayerNorm offsets N(0, 0.02), gains 1 + N(0, 0.02)), the same for every seed:
a checkpoint.  Ids are uniform over the vocabulary, lengths uniform between a fraction of the padded length and all of it.
"""
from __future__ import annotations

import math
from dataclasses import replace

import numpy as np
import torch

from mt_synth.spec import get_config, task_tensors, trunk_tensors
from paper_2107_05377_amd import binding as mt

PRECISION = {"bf16": mt.MT_BF16, "fp8_ffn": mt.MT_FP8_FFN, "fp8_layer": mt.MT_FP8_LAYER, "fp32": mt.MT_FP32_CHECK}

# What a server creates each model for: (most sequences of a call, longest padded length).
BOUNDS = {
    ("latency", "bf16"): [(8, 64)],
    ("base", "bf16"): [(256, 128), (16, 512)],
    ("base", "fp8_ffn"): [(256, 128)],
    ("base", "fp8_layer"): [(256, 128)],
    ("base", "fp32"): [(16, 128)],
    ("hetero", "bf16"): [(256, 128)],
    ("large", "bf16"): [(128, 256)],
    ("industrial", "bf16"): [(512, 32)],
    ("assistant", "bf16"): [(64, 32)],
}


def _case(name, model, precision, call, requests, batch, seq, segments=False, profiles=0):
    """requests: request batches of the call; batch: sequences of each ("requests": of the largest); seq: padded length;
    segments: sentence pairs with segment ids; profiles: ("routed") number of different task sets that sequences ask for."""
    return {"name": name, "model": model, "precision": precision, "call": call, "requests": requests, "batch": batch, "seq": seq,
            "segments": segments, "profiles": profiles}


def listed():
    return [
        # an interactive service: one short utterance at a time, and the few that arrive together
        _case("latency_b1", "latency", "bf16", "forward", 1, 1, 64),
        _case("latency_b8", "latency", "bf16", "forward", 1, 8, 64),
        # one request batch of eight classification tasks; eight of them in one call, the throughput organisation
        _case("base_b32", "base", "bf16", "forward", 1, 32, 128),
        _case("base_8x32", "base", "bf16", "multi", 8, 32, 128),
        # sentence pairs up to the model's longest input, a few at a time, an odd number of them
        _case("base_pairs_b7_s509", "base", "bf16", "forward", 1, 7, 509, segments=True),
        # the reduced precision variant at the throughput organisation
        _case("base_fp8_8x32", "base", "fp8_layer", "multi", 8, 32, 128),
        # validation of a checkpoint in float32
        _case("base_fp32_b8", "base", "fp32", "forward", 1, 8, 128),
        # tasks that fork at different depths
        _case("hetero_4x64", "hetero", "bf16", "multi", 4, 64, 128),
        # the wide, deep model on a full batch: the largest call
        _case("large_b128", "large", "bf16", "forward", 1, 128, 256),
        # 21 tasks over short utterances, requests of 1 to 16 sequences that a dispatcher has put together
        _case("industrial_32_ragged", "industrial", "bf16", "requests", 32, 16, 32),
        # the same tasks with three of them labelling every token, one request batch
        _case("assistant_tokens_b16", "assistant", "bf16", "tokens", 1, 16, 32),
        # every sequence asks for some of the tasks only
        _case("base_routed_b32", "base", "bf16", "routed", 1, 32, 128, profiles=3),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, even over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["latency", "base", "base", "multi", "pairs", "fp8", "fp32", "hetero", "large", "industrial", "assistant", "routed"])
    if kind == "latency":
        c = _case("", "latency", "bf16", "forward", 1, rng.randint(1, 8), rng.randint(9, 64))
    elif kind == "base":
        c = _case("", "base", "bf16", "forward", 1, _log(rng, 1, 256), _log(rng, 17, 128), segments=rng.random() < 0.3)
    elif kind == "multi":
        c = _case("", "base", "bf16", "multi", rng.randint(2, 8), _log(rng, 4, 32), rng.randint(33, 128))
    elif kind == "pairs":
        c = _case("", "base", "bf16", "forward", 1, rng.randint(1, 16), rng.randint(129, 512), segments=True)
    elif kind == "fp8":
        c = _case("", "base", rng.choice(["fp8_ffn", "fp8_layer"]), "multi", rng.randint(1, 8), _log(rng, 4, 32), rng.randint(33, 128))
    elif kind == "fp32":
        c = _case("", "base", "fp32", "forward", 1, rng.randint(1, 16), rng.randint(17, 128))
    elif kind == "hetero":
        c = _case("", "hetero", "bf16", "multi", rng.randint(1, 4), _log(rng, 8, 64), rng.randint(33, 128))
    elif kind == "large":
        c = _case("", "large", "bf16", "forward", 1, _log(rng, 8, 128), rng.randint(65, 256))
    elif kind == "industrial":
        c = _case("", "industrial", "bf16", "requests", _log(rng, 2, 32), rng.randint(2, 16), rng.randint(9, 32))
    elif kind == "assistant":
        c = _case("", "assistant", "bf16", "tokens", 1, _log(rng, 1, 64), rng.randint(9, 32))
    else:
        c = _case("", "base", "bf16", "routed", 1, _log(rng, 4, 64), rng.randint(33, 128), profiles=rng.randint(2, 6))
    del c["name"]
    return c


def _sizes(case):
    """Sequences of each request: ragged calls bring 1 .. batch of them."""
    if case["call"] != "requests":
        return [case["batch"]] * case["requests"]
    return [1 + (7 * r + case["batch"] - 1) % case["batch"] for r in range(case["requests"])]


def _len_lo(case):
    return max(1, case["seq"] // (4 if case["model"] == "large" else 8))


# ---- the loaded models, kept as a server keeps them
_models = {}


def _fill(flat, tensors, gen):
    at = 0
    for name, shape in tensors:
        n = math.prod(shape)
        v = flat[at:at + n].normal_(0.0, 0.02, generator=gen)
        if name.endswith("_g"):
            v.add_(1.0)
        at += n


def _load(model, spec):
    gen = torch.Generator(device="cuda").manual_seed(spec.weights_seed)
    for scope in range(-1, spec.n_tasks):
        tensors = trunk_tensors(spec) if scope < 0 else task_tensors(spec, scope)
        flat = torch.empty(sum(math.prod(s) for _, s in tensors), dtype=torch.float32, device="cuda")
        _fill(flat, tensors, gen)
        model.load_params(scope, flat.cpu().numpy(), len(tensors))


def _model(case):
    """The handle that serves this case: of those created for its model, the one with the shortest padded length that fits."""
    total = sum(_sizes(case))
    max_batch, max_seq = next(b for b in BOUNDS[case["model"], case["precision"]] if case["seq"] <= b[1] and total <= b[0])
    key = case["model"], case["precision"], max_batch, max_seq
    if key not in _models:
        spec = replace(get_config(case["model"]), batch=max_batch, seq=max_seq)
        m = mt.Model(mt.make_config(spec, precision=PRECISION[case["precision"]]))
        _load(m, spec)
        _models[key] = m
    return _models[key]


def prepare(case, seed):
    spec = get_config(case["model"])
    model = _model(case)
    rng = np.random.default_rng(seed)
    lo, S = _len_lo(case), case["seq"]
    state = {"call": case["call"], "model": model, "requests": [], "outs": [], "segments": None}
    for b in _sizes(case):
        lengths = rng.integers(lo, S + 1, b)
        ids = rng.integers(0, spec.vocab, (b, S), dtype=np.int32)
        mask = (np.arange(S)[None, :] < lengths[:, None]).astype(np.int32)
        state["requests"].append((torch.from_numpy(ids).cuda(), torch.from_numpy(mask).cuda()))
        state["outs"].append(torch.zeros((b, model.n_logits), dtype=torch.float32, device="cuda"))
        if case["segments"]:              # the second sentence starts somewhere inside the first half of the real tokens
            second = (np.arange(S)[None, :] >= (lengths * rng.uniform(0.2, 0.6, b))[:, None]).astype(np.int32)
            state["segments"] = torch.from_numpy(second).cuda()
    if case["call"] == "tokens":
        state["tokens"] = torch.zeros((case["batch"], S, model.n_token_logits), dtype=torch.float32, device="cuda")
    if case["call"] == "routed":
        state["route"] = _profiles(case, spec)[rng.integers(0, case["profiles"], case["batch"])]
    return state


def _profiles(case, spec):
    """Task sets [profiles][n_tasks]: profile p asks for about half of the tasks, each task is asked for by some."""
    p, t = np.meshgrid(np.arange(case["profiles"]), np.arange(spec.n_tasks), indexing="ij")
    return ((t + p) % 2 == 0) | (t % case["profiles"] == p)


def run(state):
    model, outs = state["model"], state["outs"]
    if state["call"] == "multi":
        return model.forward_multi(state["requests"], outs=outs)
    if state["call"] == "requests":
        return model.forward_requests(state["requests"], outs=outs)
    ids, mask = state["requests"][0]
    if state["call"] == "tokens":
        return model.forward_tokens(ids, mask, out=outs[0], out_tokens=state["tokens"])
    if state["call"] == "routed":
        return model.forward_routed(ids, mask, state["route"], outs[0])
    return model.forward(ids, mask, out=outs[0], type_ids=state["segments"])


def work(case):
    """Padding needs no work; of a sequence task's last layer only the first token's output is read, so its keys and values
    are folded into the query side (rows x heads scores and sums instead of two projections)."""
    spec = get_config(case["model"])
    H, F, A, n_seq = spec.hidden, spec.ffn, spec.heads, sum(_sizes(case))
    lo, hi = _len_lo(case), case["seq"]
    rows = n_seq * (lo + hi) / 2.0
    squares = n_seq * sum(n * n for n in range(lo, hi + 1)) / (hi - lo + 1.0)
    per_row, per_square = 2.0 * (4 * H * H + 2 * H * F), 4.0 * H
    full, first = per_row * rows + per_square * squares, 2.0 * n_seq * (4 * H * H + 2 * H * F) + 4.0 * rows * H * A
    flops = spec.n_trunk_layers * full
    share = 1.0
    for t in range(spec.n_tasks):
        task = spec.tasks[t]
        if case["call"] == "routed":
            share = float(_profiles(case, spec)[:, t].mean())
        if task.token_level:
            flops += share * (task.n_layers * full + 2.0 * rows * H * task.n_classes)
        else:
            flops += share * (max(task.n_layers - 1, 0) * full + (first if task.n_layers else 0.0) + 2.0 * n_seq * (H * H + H * task.n_classes))
    # every weight once (of the embedding tables the rows that are read), the ids and masks, the logits
    layers = spec.n_trunk_layers + sum(t.n_layers for t in spec.tasks)
    act = 4 if case["precision"] == "fp32" else 2
    matrix = {"fp32": 4.0, "bf16": 2.0, "fp8_ffn": (2.0 * 4 * H + 1.0 * 2 * F) / (4 * H + 2 * F), "fp8_layer": 1.0}[case["precision"]]
    bytes_ = layers * (4 * H * H + 2 * H * F) * matrix + sum(0 if t.token_level else H * H * act for t in spec.tasks)
    bytes_ += (rows + min(rows, hi)) * H * act + 2 * n_seq * hi * 4 + n_seq * spec.n_logits * 4
    if case["call"] == "tokens":
        bytes_ += n_seq * hi * spec.n_token_logits * 4
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """bfloat16 operands carry 2^-9 each through ten to twenty layers (6e-3 against float32 at ten layers, so 8e-3 between two
    implementations), E4M3 operands 2^-4 (4e-2 against unrounded activations); float32 is float32."""
    return {"bf16": {"rel": 1e-2}, "fp8_ffn": {"rel": 6e-2}, "fp8_layer": {"rel": 6e-2}, "fp32": {"rel": 1e-5}}[case["precision"]]
