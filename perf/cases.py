"""Performance cases: packed causal attention over slices and units, as a training or prefill program runs it.

A case is one attention layer over one pack.  `prepare` makes what the program holds before the call (tensors, tables,
workspace), `run` makes the calls of one pass:

  train      forward, then backward, each over its whole unit list in one fused launch per kernel;
  units      the same, one launch per scheduling unit in list order (a pipeline runtime that gets one unit at a time);
  forward    the fused forward alone (evaluation, recomputation of a layer);
  backward   the fused backward alone, from the o and lse of a forward pass made in `prepare`;
  slice      the forward of one unit, the last slice of a long sample, against that sample's earlier keys and values
             (prefill by slices).

Values have the distributions of the repository's workloads: q, k, v ~ 0.5 N(0,1), dO ~ 0.1 N(0,1).
"""
import math

import numpy as np
import torch

from paper_2509_26246_amd import binding as B
from paper_2509_26246_amd import harness as H

MODES = ("train", "units", "forward", "backward", "slice")


def _case(name, mode, dtype, tokens, hq, hkv, d, mix, slice_size, fwd_units, bwd_units, mix_seed=1):
    return {"name": name, "mode": mode, "dtype": dtype, "tokens": tokens, "hq": hq, "hkv": hkv, "d": d, "mix": mix,
            "mix_seed": mix_seed, "slice_size": slice_size, "fwd_units": fwd_units, "bwd_units": bwd_units}


def listed():
    return [
        # the repository's tiny pack in full precision: bound by launches and latency
        _case("tiny_f32", "train", "f32", 876, 2, 2, 64, "tiny", 64, 4, 4),
        # the tiny length mix with one GPU's share of grouped-query heads: the smallest bf16 training call
        _case("tiny_bf16", "train", "bf16", 876, 8, 1, 128, "tiny", 256, 1, 1),
        # full precision at the size of a validation step (gradient checks against the bf16 mode)
        _case("valid_f32_4k", "train", "f32", 4096, 8, 2, 128, "lognormal", 1024, 2, 4),
        # instruction-tuning data: a pack of many short ragged samples
        _case("short_16k", "train", "bf16", 16384, 32, 8, 128, "short", 4096, 4, 4),
        # an 8B-shaped layer's 32K pack, fused and by units (the repository's benchmark workload)
        _case("gqa_32k", "train", "bf16", 32768, 32, 8, 128, "lognormal", 4096, 8, 20, 2),
        _case("gqa_32k_units", "units", "bf16", 32768, 32, 8, 128, "lognormal", 4096, 8, 20, 2),
        # as many key/value heads as query heads (7B- and 13B-shaped layers)
        _case("mha_16k", "train", "bf16", 16384, 32, 32, 128, "lognormal", 4096, 4, 8, 1),
        # head dim 64
        _case("d64_32k", "train", "bf16", 32768, 32, 8, 64, "lognormal", 4096, 8, 8, 3),
        # one GPU's tensor-parallel share of a 70B-shaped layer: long-tailed 128K pack, and its units with a tail sample
        _case("tp_128k", "train", "bf16", 131072, 8, 1, 128, "pareto", 8192, 8, 16, 1),
        _case("tp_tail_units", "units", "bf16", 65536, 8, 1, 128, "tail", 8192, 4, 8, 1),
        # prefill by slices: 1024 new rows against a 32K prefix
        _case("slice_prefill", "slice", "bf16", 32768, 8, 1, 128, "one", 1024, 32, 32),
        # one long-context sample
        _case("long_64k", "train", "bf16", 65536, 8, 1, 128, "one", 8192, 8, 8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.2:
        hq, hkv = rng.choice([(2, 2), (8, 2), (4, 1), (3, 1)])
        return _unnamed("train", "f32", _log(rng, 200, 4096), hq, hkv, rng.choice([32, 64, 128]), rng.choice(["short", "lognormal", "one"]),
                        rng)
    hq, hkv = rng.choice([(32, 8), (8, 1), (32, 32), (16, 4), (40, 40), (5, 5), (3, 1), (12, 2)])
    d = rng.choice([64, 128, 128])
    mode = rng.choice(["train", "train", "units", "forward", "backward", "slice"])
    mix = "one" if mode == "slice" else rng.choice(["short", "lognormal", "lognormal", "pareto", "tail", "one"])
    while True:
        c = _unnamed(mode, "bf16", _log(rng, 500, 65536), hq, hkv, d, mix, rng)
        if c["tokens"] * hq <= 32768 * 32 and _pairs(c) * hq * d <= 65536 * 65537 // 2 * 8 * 128:
            return c


def _unnamed(mode, dtype, tokens, hq, hkv, d, mix, rng):
    slice_size = min(tokens, max(rng.randint(200, 8192), tokens // 32))
    c = _case("", mode, dtype, tokens, hq, hkv, d, mix, slice_size, max(1, min(8, tokens // 4096)), max(1, min(20, tokens // 2048)),
              rng.randint(1, 1 << 20))
    del c["name"]
    return c


def _lengths(case):
    """Sample lengths of the pack: drawn until the tokens are used up, the last one cut to fit."""
    r, left, mix = np.random.default_rng(case["mix_seed"]), case["tokens"], case["mix"]
    if mix == "tiny":
        return [37, 128, 200, 511]
    if mix == "one":
        return [left]
    out = []
    if mix == "tail":                                   # half of the pack is one sample
        out.append(left // 2)
        left -= left // 2
    while left > 0:
        if mix == "short":
            n = int(r.integers(32, 513))
        elif mix == "lognormal":
            n = int(np.clip(np.exp(7.0 + 1.2 * r.standard_normal()), 64, 32768))
        else:                                           # pareto, tail
            n = int(np.clip(256 * (1.0 - r.random()) ** (-1 / 1.1), 256, 131072))
        out.append(min(n, left))
        left -= out[-1]
    return out


def _pairs(case):
    """Visible (query, key) pairs the pass covers."""
    if case["mode"] == "slice":
        first = (case["tokens"] - 1) // case["slice_size"] * case["slice_size"]
        rows = case["tokens"] - first
        return rows * first + rows * (rows + 1) // 2
    return sum(n * (n + 1) // 2 for n in _lengths(case))


def _tables(case):
    cu, sl = B.build_slices(_lengths(case), case["slice_size"])
    if case["mode"] == "slice":                         # one unit per slice, in order
        fwd = bwd = (np.arange(len(sl) + 1), np.arange(len(sl)))
    else:
        fwd = B.build_units(cu, sl, "PREFIX_FILL", m=case["fwd_units"], w_quad=2, w_lin=0)
        bwd = B.build_units(cu, sl, "PREFIX_FILL", m=case["bwd_units"], w_quad=5, w_lin=0, backward=True)
    return B.tables_create(cu, sl, *fwd, *bwd)


def prepare(case, seed):
    T, hq, hkv, d = case["tokens"], case["hq"], case["hkv"], case["d"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(h, factor):
        return torch.randn((T, h, d), generator=gen, device="cuda", dtype=torch.float32).mul_(factor).to(dt)

    q, k, v, dO = normal(hq, 0.5), normal(hkv, 0.5), normal(hkv, 0.5), normal(hq, 0.1)
    tables = _tables(case)
    zeros = lambda shape, t=dt: torch.zeros(shape, dtype=t, device="cuda")
    ws = torch.empty(max(B.bwd_workspace_bytes(tables, hq, hkv, d), 256), dtype=torch.uint8, device="cuda")
    problem = H.Problem(tables, hq, hkv, d, B.BF16 if dt == torch.bfloat16 else B.F32, d ** -0.5, q, k, v, dO, zeros((T, hq, d)),
                        zeros((hq, T), torch.float32), zeros((T, hq, d)), zeros((T, hkv, d)), zeros((T, hkv, d)), ws)
    if case["mode"] == "backward":
        problem.forward()
    return {"mode": case["mode"], "problem": problem}


def run(state):
    p, mode = state["problem"], state["mode"]
    if mode == "slice":
        p.forward(unit_lo=p.tables.n_fwd_units - 1, unit_hi=p.tables.n_fwd_units)
        return {"o": p.o, "lse": p.lse}
    flags = B.FLAG_PER_UNIT_LAUNCH if mode == "units" else 0
    if mode != "backward":
        p.forward(flags=flags)
    if mode == "forward":
        return {"o": p.o, "lse": p.lse}
    p.backward(flags=flags)
    return {"o": p.o, "lse": p.lse, "dQ": p.dQ, "dK": p.dK, "dV": p.dV}


def work(case):
    T, hq, hkv, d, mode = case["tokens"], case["hq"], case["hkv"], case["d"], case["mode"]
    e = 2 if case["dtype"] == "bf16" else 4
    rows = T - (T - 1) // case["slice_size"] * case["slice_size"] if mode == "slice" else T
    q_like, kv_like, lse = rows * hq * d * e, T * hkv * d * e, 4 * rows * hq
    fwd_bytes = 2 * q_like + 2 * kv_like + lse          # q, k, v in; o, lse out
    bwd_bytes = 4 * q_like + 4 * kv_like + lse          # q, k, v, o, dO, lse in; dQ, dK, dV out
    product = 2 * d * hq * _pairs(case)                 # one tile product over the visible pairs; 2 forward, 5 backward
    forward, backward = mode != "backward", mode in ("train", "units", "backward")
    return {"bytes": forward * fwd_bytes + backward * bwd_bytes, "flops": (2 * forward + 5 * backward) * product}


def tolerance(case):
    # four times the largest relative error of any output against the same pass in 64 bits: 2.5e-3 (dQ, dK) in bf16,
    # 1.8e-6 (dK) in 32 bits, where a sum runs over up to 4096 x 4 terms
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 7e-6}
