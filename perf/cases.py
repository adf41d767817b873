"""Timing cases of the block-sparse attention library: what its users run, over the range they run it on.

A case is one use of the public entry points:
  mode "infer"  one forward pass (`bigbird_attn_fwd`, or the callable of `prepare_attn_fwd` where a
                serving loop keeps its buffers: `prepared`);
  mode "train"  forward and backward of one layer and step (`bigbird_attn_fwd` / `bigbird_attn_bwd`,
                their dropout forms when `p_drop` > 0), fresh outputs on every call.
Shapes come from the workload table in `bigbird_inputs.py`, `bench.py` and the tests: the ITC pattern
(g, w, r) = (2, 3, 3) at 512 .. 16384 positions, the ETC construction (leading global tokens, no random
blocks), key-padded batches with lengths that end anywhere, bf16 and fp32, attention dropout 0.1.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2007_14062_amd as bb

BLOCK = 64          # block length
DIM = 64            # head width
SCALE = 0.125       # 1 / sqrt(DIM)
P_DROP = 0.1
MIN_FILL = 0.25     # shortest sequence of a key-padded batch, as a share of n


def _case(mode, B, H, n, dtype="bf16", global_tokens=0, w=3, padded=False, skip=False, p_drop=0.0, prepared=False):
    """global_tokens 0: the ITC pattern, else that many leading global tokens and no random blocks."""
    return {"mode": mode, "B": B, "H": H, "n": n, "dtype": dtype, "global_tokens": global_tokens, "w": w,
            "padded": padded, "skip": skip, "p_drop": p_drop, "prepared": prepared}


def listed():
    return [
        # one short request in a serving loop: latency and launches
        dict(_case("infer", 1, 12, 1024, prepared=True), name="infer_short"),
        # the fp32 workload of the table, as a plain call
        dict(_case("infer", 1, 2, 1024, dtype="f32"), name="infer_fp32_short"),
        # the base model's layer at its full length (the benchmark's headline shape)
        dict(_case("infer", 4, 12, 4096, prepared=True), name="infer_base"),
        # a batch of documents of different lengths, padded to the longest
        dict(_case("infer", 8, 12, 4096, padded=True), name="infer_padded"),
        # the same by a caller that never reads padded rows
        dict(_case("infer", 8, 12, 4096, padded=True, skip=True), name="infer_padded_skip"),
        # long documents, the largest forward sequence of the table
        dict(_case("infer", 1, 16, 16384, prepared=True), name="infer_long"),
        # ETC question answering: 230 global tokens, the last global block partly filled
        dict(_case("infer", 4, 12, 4096, global_tokens=230), name="infer_etc"),
        # one step at a short, odd length (17 blocks), as in fine-tuning on short texts
        dict(_case("train", 1, 12, 1088), name="train_short"),
        # training step of the table
        dict(_case("train", 2, 12, 4096), name="train_base"),
        # pre-training as the paper's table states it: dropout on, here on padded documents (48 blocks)
        dict(_case("train", 4, 12, 3072, padded=True, skip=True, p_drop=P_DROP), name="train_dropout_padded"),
        # the longest sequence the backward takes
        dict(_case("train", 1, 16, 16384), name="train_long"),
        # fp32 step: gradients to check a model against
        dict(_case("train", 1, 2, 1024, dtype="f32"), name="train_fp32"),
    ]


def _log_blocks(rng, lo, hi):
    """A sequence length: lo .. hi blocks, spread over the logarithm."""
    return BLOCK * min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng: random.Random):
    most = {k: max(work(c)[k] for c in listed()) for k in ("bytes", "flops")}
    while True:
        if rng.random() < 0.15:
            c = _case(rng.choice(("infer", "train")), 1, rng.choice((2, 4, 8, 12)), _log_blocks(rng, 8, 32), dtype="f32",
                      padded=rng.random() < 0.3)
        else:
            mode = rng.choice(("infer", "train"))
            padded = rng.random() < 0.4
            etc = rng.random() < 0.25
            c = _case(mode, rng.choice((1, 1, 2, 3, 4, 6, 8)), rng.choice((8, 10, 12, 12, 16)),
                      _log_blocks(rng, 16 if etc else 8, 256),
                      global_tokens=rng.randrange(64, 431) if etc else 0, w=rng.choice((3, 3, 7)) if etc else 3,
                      padded=padded, skip=padded and rng.random() < 0.5,
                      p_drop=P_DROP if mode == "train" and rng.random() < 0.4 else 0.0,
                      prepared=mode == "infer" and rng.random() < 0.5)
        if all(work(c)[k] <= most[k] for k in most):
            return c


def _pattern(case):
    """(g, r, global_mode) of the case."""
    if case["global_tokens"]:
        return -(-case["global_tokens"] // BLOCK), 0, bb.BB_GLOBAL_LEADING
    return 2, 3, bb.BB_GLOBAL_FIRST_LAST


def _fills(case):
    """Mean valid share of each sequence: even steps from MIN_FILL to 1, so that a batch of every seed holds
    short and long sequences (one sequence alone is about half full)."""
    B = case["B"]
    return [MIN_FILL + (1 - MIN_FILL) * (i + 0.5) / B for i in range(B)] if case["padded"] else [1.0] * B


def _lengths(case, rng):
    """Valid positions of each sequence, anywhere in its step of `_fills`, in shuffled order."""
    step = (1 - MIN_FILL) / case["B"]
    n = case["n"]
    out = [max(1, min(n, round(n * (f + step * (rng.random() - 0.5))))) for f in _fills(case)]
    rng.shuffle(out)
    return out


def prepare(case, seed):
    dev = torch.device("cuda:0")
    B, H, n = case["B"], case["H"], case["n"]
    g, r, mode = _pattern(case)
    rng = random.Random(seed)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    Q, K, V = (torch.randn((B, H, n, DIM), generator=gen, device=dev).to(dtype) for _ in range(3))
    rand_idx = bb.bigbird_make_rand_idx(H, n, BLOCK, g, case["w"], r, seed & 0xFFFFFFFF, mode)
    mask = None
    if case["padded"] or case["global_tokens"] % BLOCK:
        mask = torch.ones((B, n), dtype=torch.uint8)
        if case["global_tokens"]:
            mask[:, case["global_tokens"]:g * BLOCK] = 0  # unused slots of the last global block
        if case["padded"]:
            for i, length in enumerate(_lengths(case, rng)):
                mask[i, length:] = 0
        mask = mask.to(dev)
    args = {"g": g, "w": case["w"], "scale": SCALE, "key_padding_mask": mask,
            "global_mode": mode | (bb.BB_SKIP_PADDED_QUERY_BLOCKS if case["skip"] else 0)}
    state = {"mode": case["mode"], "qkv": (Q, K, V), "rand_idx": torch.from_numpy(rand_idx).to(dev), "args": args,
             "drop": {"p_drop": case["p_drop"], "seed": seed} if case["p_drop"] else None}
    if case["mode"] == "train":
        state["dO"] = torch.randn((B, H, n, DIM), generator=gen, device=dev).to(dtype)
    elif case["prepared"]:
        O = torch.empty_like(Q)
        LSE = torch.empty((B, H, n), dtype=torch.float32, device=dev)
        ws = torch.empty(max(256, bb.bigbird_attn_workspace_bytes(B, H, n, DIM, BLOCK, g, case["w"], r)),
                         dtype=torch.uint8, device=dev)
        state["out"], state["workspace"] = (O, LSE), ws
        state["call"] = bb.prepare_attn_fwd(Q, K, V, state["rand_idx"], O, LSE, ws, **args)
    return state


def run(state):
    Q, K, V = state["qkv"]
    ridx, args, drop = state["rand_idx"], state["args"], state["drop"]
    if state["mode"] == "infer":
        if "call" in state:
            state["call"]()
            return state["out"]
        return bb.bigbird_attn_fwd(Q, K, V, ridx, **args)
    if drop is None:
        O, LSE = bb.bigbird_attn_fwd(Q, K, V, ridx, **args)
        return (O, LSE) + tuple(bb.bigbird_attn_bwd(Q, K, V, O, LSE, state["dO"], ridx, **args))
    O, LSE = bb.bigbird_attn_fwd_dropout(Q, K, V, ridx, **drop, **args)
    return (O, LSE) + tuple(bb.bigbird_attn_bwd_dropout(Q, K, V, O, LSE, state["dO"], ridx, **drop, **args))


def work(case):
    """Two matrix products of the forward (and five of the backward) per block pair of the pattern that holds a
    valid key; Q, K, V (dO) read once, O, LSE (and the fp32 gradients) written once."""
    B, H, n = case["B"], case["H"], case["n"]
    g, r, _ = _pattern(case)
    nb, w = n // BLOCK, case["w"]
    lead = g if case["global_tokens"] else 1
    pairs = 0.0
    for f in _fills(case):
        v = math.ceil(f * nb)                      # key blocks with a valid position
        g_v = lead + (g - lead if v == nb else 0)  # global ones among them
        r_v = r * v / nb                           # random ones of a row
        row_pairs = (g_v if case["skip"] else g) * v + (v - g_v) * (g_v + w + r_v) - (w * w - 1) // 2
        if not case["skip"]:
            row_pairs += (nb - v) * (g_v + r_v)    # rows of padded queries: computed all the same
        pairs += H * row_pairs
    el = 2 if case["dtype"] == "bf16" else 4
    rows = B * H * n
    fill = sum(_fills(case)) / B
    nbytes = rows * DIM * el * (2 + 2 * fill) + rows * 4
    if case["mode"] == "train":
        nbytes += rows * DIM * (el + 3 * 4)
    return {"bytes": int(nbytes), "flops": int(pairs * BLOCK * BLOCK * DIM * (14 if case["mode"] == "train" else 4))}


def tolerance(case):
    """Four times the largest error seen against fp64 dense attention (rel, and max against max(rms, value)):
    fp32 6e-7 and 6e-6; bf16, whose probabilities and outputs are rounded to 2^-9, 2.3e-3 and 2.4e-2."""
    if case["dtype"] == "f32":
        return {"rel": 2.5e-6, "max": 2.5e-5}
    return {"rel": 1e-2, "max": 1e-1}
