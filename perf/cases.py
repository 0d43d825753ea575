"""The calls that performance work on this library is measured on.

Every case is one pass through the public Python entry points, with the inputs, packed routers and frozen calls that a
program holding a model would have in hand.  The sizes are those of the paper's models (8B: d = 4096, 32 or 36 layers,
checkpoints every 4), of the hidden-size sweep and of Table 2's widths, and ragged ones between them.

    decode       one step of a running batch: all checkpoints' rows of a few tokens (static buffers, frozen call)
    prompt       one request's prompt through all checkpoints, then the rows its LM head consumes
    checkpoint   a layer-skipping loop's call: ONE checkpoint on the rows that still run (static buffers, frozen call)
    prefill      a batch of prompts through all checkpoints
    labels       calibration: similarity labels of a batch of texts against the last layer's states
"""
from __future__ import annotations

import math

import torch

from paper_2603_21365_amd import tide_route as tr

EPS = 1e-6
THETA = 0.5
TAU = 0.98                                  # the paper's calibration threshold
SIZES = (768, 1024, 2048, 2560, 3072, 4096, 5120, 8192)          # the hidden-size sweep
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
CODE = {"f32": tr.F32, "f16": tr.F16, "bf16": tr.BF16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def _case(name, path, dtype, C, T, d, b=128, raw=False):
    return {"name": name, "path": path, "dtype": dtype, "C": C, "T": T, "d": d, "b": b, "raw": raw}


def listed():
    return [
        # a single user's generation: one token through the routers of an 8B model
        _case("decode_f16_T1", "decode", "f16", 8, 1, 4096),
        # continuous batching: 48 sequences decode together
        _case("decode_bf16_T48", "decode", "bf16", 8, 48, 4096),
        # the same call by a program that keeps its router weights in fp32 and never packs them
        _case("decode_raw_f16_T4", "decode", "f16", 8, 4, 4096, raw=True),
        # the 322 prompt tokens of the paper's evaluation, 8B model, and the projection of the exiting rows
        _case("prompt_bf16_T322", "prompt", "bf16", 8, 322, 4096),
        # true layer skipping: the rows still running after a few checkpoints of a batched prefill
        _case("checkpoint_bf16_T3000", "checkpoint", "bf16", 1, 3000, 4096),
        # the benchmark's step: raw fp32 router weights, 4096 tokens, 8B model
        _case("prefill_raw_bf16", "prefill", "bf16", 8, 4096, 4096, raw=True),
        # the 36-layer model's batch of 8 x 2048 tokens: the largest call
        _case("prefill_bf16_36l", "prefill", "bf16", 9, 16384, 4096),
        # Table 2's narrow router on a small model, ragged batch
        _case("prefill_f16_b64", "prefill", "f16", 8, 6001, 2048, b=64),
        # a model that runs in fp32, ragged batch
        _case("prefill_f32_d2560", "prefill", "f32", 10, 3001, 2560),
        # Table 2's wide router on the 8B model
        _case("prefill_bf16_b256", "prefill", "bf16", 8, 4096, 4096, b=256),
        # a 48-layer model whose hidden size is no multiple of 128: the generic fallback
        _case("prefill_bf16_d1600", "prefill", "bf16", 12, 4000, 1600),
        # calibration on eight texts of 170 tokens
        _case("labels_bf16_T1360", "labels", "bf16", 8, 1360, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _bytes_of_rows(c):
    return c["C"] * c["T"] * c["d"] * BYTES[c["dtype"]]


def draw(rng):
    path = rng.choice(("decode", "prompt", "checkpoint", "prefill", "prefill", "labels"))
    c = {"path": path, "dtype": rng.choice(("bf16", "bf16", "f16", "f32")), "C": rng.randint(4, 10), "T": 0, "d": rng.choice(SIZES),
         "b": 128, "raw": False}
    if path == "decode":
        c["T"], c["raw"] = _log_int(rng, 1, 64), rng.random() < 0.3
    elif path == "prompt":
        c["T"], c["b"] = _log_int(rng, 65, 1000), rng.choice((64, 128, 128, 256))
    elif path == "checkpoint":
        c["T"], c["C"] = _log_int(rng, 64, 16384), 1
    elif path == "prefill":
        c["T"], c["b"], c["raw"] = _log_int(rng, 1000, 16384), rng.choice((64, 128, 128, 256)), rng.random() < 0.25
    else:
        c["T"] = _log_int(rng, 340, 5440)
    odd = path != "labels" and rng.random() < 0.2
    if odd:                                         # hidden sizes that are no multiple of 128
        c["d"], c["b"] = 128 * rng.randint(6, 36) + 8 * rng.randint(1, 15), 128
    # no dearer than the largest listed case, whose 1.2 GB of rows move at the copy rate; these are slower per byte
    most = (0.55e9 if c["dtype"] == "f32" else 1.1e9) / (2 if c["b"] == 256 or odd else 1)
    while _bytes_of_rows(c) > most:
        c["T"] = c["T"] * 7 // 10
    return c


def _inputs(case, seed):
    """Hidden states that drift towards the last layer's (noise falling from 1.0 to 0.05 over the checkpoints, eight
    outlier channels), random routers of the usual scales, and biases that let about 30 % of the rows fire."""
    C, T, d, b, dev = case["C"], case["T"], case["d"], case["b"], "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1000003 + 17)
    r = lambda *s: torch.randn(s, generator=g, device=dev)
    final = r(T, d)
    scale = torch.ones(d, device=dev)
    scale[torch.randperm(d, generator=g, device=dev)[:8]] = 20.0
    hidden = torch.empty((C, T, d), dtype=TORCH[case["dtype"]], device=dev)
    for c in range(C):
        sigma = 1.0 - 0.95 * c / (C - 1) if C > 1 else 0.5
        hidden[c] = (final + sigma * r(T, d)) * scale
    final = (final * scale).to(hidden.dtype)
    x = {"hidden": hidden, "final": final, "gamma": 1.0 + 0.1 * r(C, d), "W1": r(C, d, b) / math.sqrt(d), "b1": 0.1 * r(C, b),
         "w2": r(C, b) / math.sqrt(b), "norm": 1.0 + 0.1 * r(d), "ids": [4 * c + 3 for c in range(C)], "layers": 4 * C}
    x["b2"] = [-0.21 * s - 0.3 for s in x["w2"].sum(1).tolist()]        # the mean of SiLU on unit normals is 0.21
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    state = {"case": case, "x": x}
    if case["path"] == "labels":
        for name in ("gamma", "W1", "b1", "w2"):
            x.pop(name)
        return state
    if not case["raw"]:
        x["packed"] = tr.router_pack(CODE[case["dtype"]], x.pop("gamma"), x.pop("W1"))
    if case["path"] != "prompt":
        x.pop("final")
    tail = (x["b1"], x["w2"], x["b2"], THETA, x["ids"], 0, x["layers"])
    if case["path"] in ("decode", "checkpoint", "prompt"):              # static buffers: the calls are frozen once
        if case["raw"]:
            state["select"] = tr.prepare_select_exit(x["hidden"], x["gamma"], EPS, x["W1"], *tail)
        else:
            state["select"] = tr.prepare_select_exit_packed(x["hidden"], x["packed"], EPS, *tail, d=case["d"])
        if case["path"] == "prompt":
            state["project"] = tr.prepare_exit_project(x["hidden"], x["final"], state["select"].outputs[0], x["ids"], x["norm"], EPS)
    else:
        state["tail"] = tail
    return state


def run(state):
    case, x = state["case"], state["x"]
    if case["path"] == "labels":
        return tr.cosine_labels(x["hidden"], x["final"], TAU)
    if "select" in state:
        out = state["select"]()
        return (*out, state["project"]()) if "project" in state else out
    if case["raw"]:
        return tr.select_exit(x["hidden"], x["gamma"], EPS, x["W1"], *state["tail"])
    return tr.select_exit_packed(x["hidden"], x["packed"], EPS, *state["tail"], d=case["d"])


def work(case):
    C, T, d, b, e = case["C"], case["T"], case["d"], case["b"], BYTES[case["dtype"]]
    rows = C * T * d * e
    if case["path"] == "labels":
        return {"bytes": rows + T * d * e + 5 * C * T, "flops": 4 * C * T * d}
    weights = C * d * (b + 1) * 4 if case["raw"] else C * d * b * e
    size = {"bytes": rows + weights + 8 * T + 4 * C * T, "flops": 2 * C * T * d * b}
    if case["path"] == "prompt":
        size["bytes"] += 2 * T * d * e
    return size


def tolerance(case):
    """About four times the difference to 64-bit results that was measured over these ranges."""
    if case["path"] == "labels":                    # fp32 sums: 8e-8; a label flips where a similarity lies within that of tau
        return {"rel": 4e-7, "max": 2e-6, "differ": 1e-3}
    if case["raw"] and case["T"] <= 8:              # fp32 weights, products and sums: 1.5e-7
        return {"rel": 6e-7, "max": 2e-6, "differ": 0.0}
    if case["dtype"] == "f32":                      # two bf16 terms per value: 4.4e-6
        return {"rel": 1.8e-5, "max": 1e-4, "differ": 2e-4}
    if case["dtype"] == "f16":                      # the folded router weights are rounded to the storage type: 2.1e-4
        return {"rel": 8.5e-4, "max": 4e-3, "differ": 1.5e-3}
    return {"rel": 6.5e-3, "max": 3e-2, "differ": 1e-2}                 # likewise: 1.6e-3


def exact(case, seed):
    x = _inputs(case, seed)
    C, T = case["C"], case["T"]
    step = 4096
    if case["path"] == "labels":
        sim = torch.empty((C, T), dtype=torch.float64, device="cuda")
        for c in range(C):
            for t in range(0, T, step):
                h, f = x["hidden"][c, t:t + step].double(), x["final"][t:t + step].double()
                sim[c, t:t + step] = (h * f).sum(1) / (h.square().sum(1) * f.square().sum(1)).sqrt()
        return sim, (sim > TAU).to(torch.uint8)
    z = torch.empty((C, T), dtype=torch.float64, device="cuda")
    for c in range(C):
        w = x["gamma"][c].double()[:, None] * x["W1"][c].double()
        b2 = float(torch.tensor(x["b2"][c], dtype=torch.float32))
        for t in range(0, T, step):
            h = x["hidden"][c, t:t + step].double()
            a = (h @ w) / (h.square().mean(1, keepdim=True) + EPS).sqrt() + x["b1"][c].double()
            z[c, t:t + step] = (a * torch.sigmoid(a)) @ x["w2"][c].double() + b2
    fired = z > math.log(THETA / (1 - THETA))
    exits = torch.full((T,), x["layers"], dtype=torch.int32, device="cuda")
    mask = torch.zeros(T, dtype=torch.int32, device="cuda")
    for c in range(C - 1, -1, -1):
        exits = torch.where(fired[c], torch.full_like(exits, x["ids"][c]), exits)
        mask |= fired[c].to(torch.int32) << c
    if case["path"] != "prompt":
        return exits, z, mask
    return exits, z, mask, None                     # the projected rows follow the exit layers, ties and all
