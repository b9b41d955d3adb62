"""Timed workloads of the packed-attention path, through the public entry points of `binding`.

Three kinds of pass:
  step    : position ids -> boundaries -> forward -> backward, what one attention layer of a training step
            does (optionally preceded by the device collator and the rotary embedding of Q and K and followed
            by the inverse rotation of their gradients, as an online minibatch is trained on);
  forward : position ids -> boundaries -> forward, as an evaluation or a prefill runs it;
  inputs  : collator -> boundaries -> rotary embedding of Q and K, what happens before attention.

A case fixes the multiset of example lengths of every row (drawn from its length law with its own
`lengths_seed`), so that its work is known; the order of the rows and of the examples in them, and every
tensor, come from the seed given to `prepare`.
"""
import functools
import math
import random

import numpy as np
import torch

from paper_2407_09105_amd import binding
from paper_2407_09105_amd import workloads as wl

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

# ---- the cases --------------------------------------------------------------------------------------


def _case(kind, rows, tokens, hq, hkv, d, dtype, law, lengths_seed=1, grads="same", examples=0):
    """law: "uniform lo hi", "lognormal median sigma lo hi", "longtail median sigma share lo hi" or
    "whole" (one example per row).  examples > 0: the stream is one row of that many whole examples,
    collated on the device from a padded batch (tokens is then ignored); the step also rotates Q and K."""
    return {"kind": kind, "rows": rows, "tokens": tokens, "hq": hq, "hkv": hkv, "d": d, "dtype": dtype, "law": law,
            "lengths_seed": lengths_seed, "grads": grads, "examples": examples}


def listed():
    cases = {
        # the smallest call: 16 tokens in fp32, what a first check of an integration runs (latency and launches)
        "fp32_16_tokens": _case("step", 1, 16, 2, 2, 16, "f32", "uniform 1 7"),
        # a layer re-run in fp32 to check a 16-bit model's numbers and gradients: about a thousand tokens, few heads
        "fp32_check_1x1000": _case("step", 1, 1000, 8, 2, 64, "f32", "lognormal 128 1.0 8 1000"),
        # online minibatch of 4 examples of a few hundred tokens, collated on the fly, with rotary embedding
        "minibatch_of_4": _case("step", 1, 0, 32, 8, 128, "bf16", "lognormal 256 0.8 16 2048", examples=4),
        # one packed row of 8192 tokens, as many KV heads as query heads
        "row_1x8192": _case("step", 1, 8192, 32, 32, 128, "bf16", "lognormal 256 1.0 16 4096", wl.SEED_BASE + 2),
        # fixed-length packing, four rows of 4096 tokens, grouped heads
        "gqa_4x4096": _case("step", 4, 4096, 32, 8, 128, "bf16", "lognormal 512 0.8 32 4096", wl.SEED_BASE + 3),
        # a thousand examples of 8..128 tokens: bound by memory, full of boundaries
        "short_8x8192": _case("step", 8, 8192, 32, 32, 128, "bf16", "uniform 8 128", wl.SEED_BASE + 4),
        # examples of up to a whole row among many short ones, five query heads to a KV head: the largest step
        "longtail_2x16384": _case("step", 2, 16384, 40, 8, 128, "bf16", "longtail 300 1.2 0.1 4096 16384", wl.SEED_BASE + 5),
        # fp16, one KV head for all query heads, head dim 64, rows one token short of a power of two
        "f16_mqa_3x2047": _case("step", 3, 2047, 16, 1, 64, "f16", "lognormal 400 0.8 16 2047"),
        # head dim 80 (no power of two), odd rows, gradients handed on in fp32
        "d80_fp32_grads_2x3001": _case("step", 2, 3001, 32, 32, 80, "bf16", "lognormal 100 1.0 8 3001", grads="f32"),
        # head dim 256
        "d256_1x8192": _case("step", 1, 8192, 16, 16, 256, "bf16", "lognormal 400 1.0 16 4096"),
        # forward only over one long example (evaluation, prefill)
        "forward_1x16384": _case("forward", 1, 16384, 32, 8, 128, "bf16", "whole"),
        # what precedes attention: a thousand examples collated into one row, their boundaries, Q and K rotated
        "inputs_1024_examples": _case("inputs", 1, 0, 32, 8, 128, "bf16", "uniform 8 128", examples=1024),
    }
    return [{"name": name, **case} for name, case in cases.items()]


# head layouts (query heads, KV heads, head_dim) of decoder layers with a few billion parameters
HEADS = [(32, 32, 128), (32, 8, 128), (40, 8, 128), (36, 4, 128), (32, 32, 64), (16, 1, 64), (32, 32, 80), (24, 8, 96),
         (16, 16, 256)]
LAWS = ["uniform 8 128", "lognormal 100 1.0 8 4096", "lognormal 256 1.0 16 4096", "lognormal 512 0.8 32 4096",
        "longtail 300 1.2 0.1 4096 16384", "whole"]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = work(next(c for c in listed() if c["name"] == "longtail_2x16384"))
    while True:
        seed = rng.randrange(1, 1 << 20)
        what = rng.choice(["row", "row", "row", "row", "minibatch", "forward", "inputs", "fp32"])
        hq, hkv, d = rng.choice(HEADS)
        dtype = rng.choice(["bf16", "bf16", "f16"])
        rows = rng.choice([1, 1, 2, 3, 4, 8])
        tokens = max(64, _log_uniform(rng, 512, 65536) // rows)
        if rng.random() < 0.5:
            tokens = min(16384, (tokens + 255) // 256 * 256)
        else:
            tokens = min(16383, tokens)
        if what == "row":
            c = _case("step", rows, tokens, hq, hkv, d, dtype, rng.choice(LAWS), seed, rng.choice(["same", "same", "f32"]))
        elif what == "forward":
            c = _case("forward", rows, tokens, hq, hkv, d, dtype, rng.choice(LAWS), seed)
        elif what == "minibatch":
            c = _case("step", 1, 0, hq, hkv, d, dtype, rng.choice(LAWS[1:4]), seed, examples=rng.choice([1, 2, 3, 4, 8, 16]))
        elif what == "inputs":
            c = _case("inputs", 1, 0, hq, hkv, d, dtype, rng.choice(LAWS[:4]), seed, examples=_log_uniform(rng, 16, 1024))
        else:
            heads = rng.choice([2, 4, 8])
            c = _case("step", rng.choice([1, 2]), _log_uniform(rng, 16, 1024), heads, heads // rng.choice([1, 2]), rng.choice([16, 32, 64]),
                      "f32", "lognormal 100 1.0 4 1024", seed)
        w = work(c)
        if w["bytes"] <= most["bytes"] * 4 and w["flops"] <= 0.9 * most["flops"] and sum(sum(r) for r in lengths(c)) <= 65536:
            return c


# ---- inputs -----------------------------------------------------------------------------------------


def _law(case):
    name, *args = case["law"].split()
    return name, tuple(float(a) for a in args)


@functools.lru_cache(maxsize=64)
def _lengths(law, args, rows, tokens, examples, seed):
    rng = np.random.default_rng(seed)
    integer = lambda a: tuple(int(x) if float(x).is_integer() else x for x in a)  # noqa: E731
    if law == "whole":
        return tuple((tokens,) for _ in range(rows))
    if examples:  # that many whole examples in one row, whatever they add up to
        cfg = wl.Config(0, "drawn", 1, 1 << 20, 1, 1, 8, "bf16", law, integer(args))
        return (tuple(wl.draw_lengths(cfg, rng)[0][:examples]),)
    cfg = wl.Config(0, "drawn", rows, tokens, 1, 1, 8, "bf16", law, integer(args))
    return tuple(tuple(row) for row in wl.draw_lengths(cfg, rng))


def lengths(case):
    """Example lengths per row, in the order they were drawn."""
    law, args = _law(case)
    return _lengths(law, args, case["rows"], case["tokens"], case["examples"], case["lengths_seed"])


def prepare(case, seed):
    rng = random.Random(seed)
    rows = [list(row) for row in lengths(case)]
    rng.shuffle(rows)
    for row in rows:
        rng.shuffle(row)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    n = sum(sum(row) for row in rows)
    normal = lambda heads: torch.randn((n, heads, case["d"]), generator=gen, device=DEV, dtype=torch.float32).to(dt)  # noqa: E731
    state = {"case": case, "n_examples": sum(len(row) for row in rows), "n_tokens": n,
             "q": normal(case["hq"]), "k": normal(case["hkv"])}
    if case["kind"] != "inputs":
        state["v"] = normal(case["hkv"])
    if case["kind"] == "step":
        state["do"] = normal(case["hq"])
        state["grad_dtype"] = torch.float32 if case["grads"] == "f32" else dt
    if case["examples"]:
        row = rows[0]
        state["ids"] = torch.randint(1, 32000, (len(row), max(row)), generator=gen, device=DEV, dtype=torch.int64)
        state["lengths"] = torch.tensor(row, dtype=torch.int32, device=DEV)
    else:
        state["position_ids"] = torch.from_numpy(wl.position_ids_from_lengths(rows)).to(DEV)
    return state


# ---- one pass ---------------------------------------------------------------------------------------


def run(state):
    case = state["case"]
    q, k = state["q"], state["k"]
    rotate = case["examples"] > 0
    if rotate:
        batch = binding.collate_padding_free(state["ids"], state["lengths"], state["n_tokens"])
        pos = batch["position_ids"]
    else:
        pos = state["position_ids"]
    seg = binding.pack_to_cu_seqlens(pos)
    if rotate:
        ids = pos.view(-1)
        q, k = binding.rope_apply(q, ids), binding.rope_apply(k, ids)
    if case["kind"] == "inputs":
        return {**batch, "cu_seqlens": seg.cu_seqlens_capacity[: state["n_examples"] + 1], "seg_id": seg.seg_id,
                "seg_start": seg.seg_start, "seg_end": seg.seg_end, "q": q, "k": k}
    o, lse = binding.varlen_attn_fwd(q, k, state["v"], seg)
    if case["kind"] == "forward":
        return {"o": o, "lse": lse}
    dq, dk, dv = binding.varlen_attn_bwd(state["do"], q, k, state["v"], o, lse, seg, grad_dtype=state["grad_dtype"])
    if rotate:
        binding.rope_apply(dq, ids, inverse=True, out=dq)
        binding.rope_apply(dk, ids, inverse=True, out=dk)
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


# ---- what a pass cannot do without, and how exact it is ----------------------------------------------


def work(case):
    """Bytes: every input of the pass read once, every output written once.  Flops: the unmasked
    (query, key) pairs, 4 d per pair and query head forward, 10 d backward."""
    flat = [L for row in lengths(case) for L in row]
    n, pairs = sum(flat), sum(L * (L + 1) // 2 for L in flat)
    hq, hkv, d, e = case["hq"], case["hkv"], case["d"], 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "inputs":  # ids in; ids, labels, position ids, boundaries out; Q and K in and out
        return {"bytes": n * (4 * 8 + 3 * 4) + 2 * n * e * d * (hq + hkv), "flops": 0}
    bytes_ = n * (8 + e * d * (2 * hq + 2 * hkv) + 4 * hq)  # position ids, Q, K, V, O, LSE
    if case["kind"] == "forward":
        return {"bytes": bytes_, "flops": 4 * d * hq * pairs}
    eg = 4 if case["grads"] == "f32" or case["dtype"] == "f32" else 2
    bytes_ += n * (e * d * hq + eg * d * (hq + 2 * hkv))    # dO, dQ, dK, dV
    return {"bytes": bytes_, "flops": 14 * d * hq * pairs}


def tolerance(case):
    """About four times the distance from a float64 evaluation of the same inputs (largest seen over the listed cases
    and a dozen drawn ones: fp32 6e-7 / 1.3e-5, bf16 2.4e-3 / 4e-2, fp16 4e-4 / 1.3e-2; a bf16 output averaged over
    16384 keys 0.12)."""
    if case["dtype"] == "f32":
        return {"rel": 2.5e-6, "max": 5e-5}
    if case["dtype"] == "f16":
        return {"rel": 1.6e-3, "max": 0.05}
    return {"rel": 1e-2, "max": 0.4 if case["law"] == "whole" else 0.16}
