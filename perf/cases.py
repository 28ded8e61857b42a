"""The work a decoder gives this library, as measurable cases.

Five kinds of pass, all through `paper_2105_04779_amd.el_attn`:

  step       one decode step: cross-attention of `beam` queries per sentence over an encoder output, or (beam 1) of one
             query per history over the previous layer's outputs
  layers     one token through a decoder: twelve attention layers, weights of their own each, on one encoder output
  segments   one decoder-only step: attention over the shared prefix and over each beam's own continuation, joined
             under one softmax
  gather     beam re-order: every surviving beam takes over its parent's history

Inputs are drawn on the device from the seed alone: hidden states and queries N(0, 1), weights N(0, 1/d_m), biases
N(0, 0.02^2).  Lengths are an even spread over [len_lo, len_hi] in random order, so a case has the same amount of work
for every seed.
"""
import math

import torch

from paper_2105_04779_amd import el_attn

_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_BYTES = {"f32": 4, "f16": 2, "bf16": 2}
_HEADS = {64: 4, 128: 2, 256: 4, 512: 8, 768: 12, 1024: 16}


def _step(dtype, d_m, B, beam, n, len_lo=None, out="f32", layers=1):
    return {"kind": "step" if layers == 1 else "layers", "dtype": dtype, "d_m": d_m, "heads": _HEADS[d_m], "B": B, "beam": beam,
            "n": n, "len_lo": n if len_lo is None else len_lo, "out": out, "layers": layers}


def _segments(dtype, d_m, B, beam, n, len_lo, suffix):
    return {"kind": "segments", "dtype": dtype, "d_m": d_m, "heads": _HEADS[d_m], "B": B, "beam": beam, "n": n,
            "len_lo": len_lo, "suffix": suffix, "out": "f32"}


def _gather(dtype, d_m, B, group, n, len_lo):
    return {"kind": "gather", "dtype": dtype, "d_m": d_m, "B": B, "group": group, "n": n, "len_lo": len_lo}


def listed():
    cases = {
        # the fp32 configuration of the benchmark: the smallest call, launches and latency alone
        "tiny_f32": _step("f32", 64, 2, 2, 32),
        # Transformer-base width in fp32: a model that is run at full precision
        "base_f32": _step("f32", 512, 16, 4, 300, 150),
        # one sentence, beam 4, BART-large width: interactive use, an odd length
        "one_sentence_bf16": _step("bf16", 1024, 1, 4, 613),
        # the same user's whole token: twelve decoder layers on one encoder output, results in the storage type
        "twelve_layers_b4_bf16": _step("bf16", 1024, 4, 4, 410, 205, out="bf16", layers=12),
        # Transformer-base batch decode in fp16
        "base_beam_f16": _step("f16", 512, 64, 4, 512, 256),
        # the benchmark's default: BART-large batch decode, beam 4
        "large_beam_bf16": _step("bf16", 1024, 64, 4, 1024, 512),
        # base-size models (12 heads), a beam of five and lengths that fit no tile
        "w768_beam5_bf16": _step("bf16", 768, 48, 5, 777, 301),
        # the largest batch: 320 sentences, beam 4, BART-large width
        "large_b320_bf16": _step("bf16", 1024, 320, 4, 1024, 512),
        # per-beam self-attention histories early and late in a generation (GPT-2-medium width; GPT-2-small width)
        "history_1024_bf16": _step("bf16", 1024, 512, 1, 1024),
        "history_w768_f16": _step("f16", 768, 160, 1, 211),
        # decoder-only generation: shared prompt and 37 tokens of each beam's own
        "prefix_suffix_bf16": _segments("bf16", 1024, 32, 4, 512, 256, 37),
        # beam re-order of histories of mixed length between two steps
        "reorder_bf16": _gather("bf16", 1024, 512, 4, 1024, 512),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "history", "f32", "layers", "segments", "gather"])
    d_m, dtype, out = rng.choice([512, 768, 1024]), rng.choice(["f16", "bf16"]), rng.choice(["f32", "storage"])
    out = dtype if out == "storage" else "f32"
    if kind == "f32":
        d_m = rng.choice([64, 128, 256, 512])
        n = _log_int(rng, 16, 300)
        return _step("f32", d_m, rng.randint(1, 16), rng.randint(1, 4), n, rng.randint((n + 1) // 2, n))
    if kind == "step":
        n, beam, B = _log_int(rng, 16, 1024), rng.randint(1, 8), _log_int(rng, 1, 320)
        B = min(B, max(1, 320 * 4 * 1024 // (beam * max(n, 256))))    # never beyond the largest listed batch
        return _step(dtype, d_m, B, beam, n, rng.randint((n + 1) // 2, n), out)
    if kind == "history":
        return _step(dtype, d_m, _log_int(rng, 8, 512), 1, _log_int(rng, 16, 1024), None, out)
    if kind == "layers":
        n = _log_int(rng, 32, 1024)
        return _step(dtype, d_m, rng.randint(1, 8), rng.randint(1, 6), n, rng.randint((n + 1) // 2, n), out, layers=12)
    if kind == "segments":
        n, beam = _log_int(rng, 64, 768), rng.randint(2, 6)
        return _segments(dtype, d_m, _log_int(rng, 1, 64), beam, n, rng.randint((n + 1) // 2, n), _log_int(rng, 1, 256))
    n, group = _log_int(rng, 32, 1024), rng.randint(2, 8)
    return _gather(dtype, d_m, group * _log_int(rng, 2, 512 // group), group, n, rng.randint((n + 1) // 2, n))


def _lengths_sorted(case):
    """Evenly spread over [len_lo, n], both ends included (a single element has the full length)."""
    B, lo, n = case["B"], case["len_lo"], case["n"]
    return [n - (n - lo) * k // max(1, B - 1) for k in range(B)]


def _sum_len(case):
    return sum(_lengths_sorted(case))


def _randn(g, shape, dtype, scale=1.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=_TORCH[dtype])
    return x if scale == 1.0 else x.mul_(scale)


def _weights(g, case):
    d_m, dt = case["d_m"], case["dtype"]
    W = {k: _randn(g, (d_m, d_m), dt, d_m ** -0.5) for k in ("Wq", "Wk", "Wv", "Wo")}
    W.update({k: _randn(g, (d_m,), dt, 0.02) for k in ("bq", "bk", "bv", "bo")})
    return W


def _layer(g, case, max_batch, max_beam, max_n):
    return el_attn.ElAttention(_weights(g, case), heads=case["heads"], d_k=case["d_m"] // case["heads"], dtype=case["dtype"],
                               max_batch=max_batch, max_beam=max_beam, max_n=max_n, out_dtype=case["out"])


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    gc = torch.Generator().manual_seed(seed)
    B, n, d_m, dt = case["B"], case["n"], case["d_m"], case["dtype"]
    lens = torch.tensor(_lengths_sorted(case), dtype=torch.int32)[torch.randperm(B, generator=gc)]
    s = {"kind": case["kind"], "H": _randn(g, (B, n, d_m), dt), "lengths": lens.cuda()}
    if case["kind"] == "gather":
        parent = torch.arange(B) // case["group"] * case["group"]         # a parent among the beams of the same sentence
        s["index"] = (parent + torch.randint(case["group"], (B,), generator=gc)).to(torch.int32).cuda()
        s["H_dst"] = torch.zeros_like(s["H"])
        s["lengths_dst"] = torch.zeros_like(s["lengths"])
        return s
    x = case["beam"]
    if case["kind"] == "segments":
        s["layer"] = _layer(g, case, B * x, x, max(n, case["suffix"]))
        s["H_own"] = _randn(g, (B * x, case["suffix"], d_m), dt)
        s["lengths_own"] = torch.full((B * x,), case["suffix"], dtype=torch.int32, device="cuda")
        s["Q"] = _randn(g, (B, x, d_m), dt)
        s["Q_own"] = s["Q"].view(B * x, 1, d_m)
        return s
    s["layers"] = [_layer(g, case, B, x, n) for _ in range(case["layers"])]
    s["Q"] = [_randn(g, (B, x, d_m), dt) for _ in s["layers"]]
    s["out"] = [torch.empty((B, x, d_m), dtype=_TORCH[case["out"]], device="cuda") for _ in s["layers"]]
    return s


def run(state):
    kind = state["kind"]
    if kind == "gather":
        return el_attn.gather_batch(state["H"], state["lengths"], state["index"], H_dst=state["H_dst"],
                                    lengths_dst=state["lengths_dst"])
    if kind == "segments":
        layer, Q = state["layer"], state["Q"]
        shared = layer.decode_segment(state["H"], state["lengths"], Q)
        own = layer.decode_segment(state["H_own"], state["lengths_own"], state["Q_own"])
        return layer.merge_segments([shared, own], Q.shape[0], Q.shape[1]), shared, own
    H, lengths = state["H"], state["lengths"]
    return [layer.decode_step(H, lengths, q, out=o) for layer, q, o in zip(state["layers"], state["Q"], state["out"])]


def _attention_flops(sum_len, rows, beam, heads, d_m):
    """Algorithm 3's routine: four products of the projections per query row, two over every valid position."""
    return 8.0 * rows * d_m * d_m + 4.0 * heads * beam * sum_len * d_m


def work(case):
    d_m, e, total = case["d_m"], _BYTES[case["dtype"]], _sum_len(case)
    if case["kind"] == "gather":
        # parents are drawn among the beams of one sentence: on average every source row is read and written once
        return {"bytes": 2.0 * total * d_m * e, "flops": 0.0}
    rows, x, h = case["B"] * case["beam"], case["beam"], case["heads"]
    weights = (4.0 * d_m * d_m + 4.0 * d_m) * e
    if case["kind"] == "segments":
        own = rows * case["suffix"]
        seg = rows * (d_m + h) * 4.0                                      # head outputs and statistics of a segment, fp32
        return {"bytes": weights + (total + own + rows) * d_m * e + 2 * seg + rows * d_m * 4.0,
                "flops": _attention_flops(total, rows, x, h, d_m) + _attention_flops(own, rows, 1, h, d_m)}
    L = case["layers"]
    return {"bytes": total * d_m * e + L * (weights + rows * d_m * (e + _BYTES[case["out"]])),
            "flops": L * _attention_flops(total, rows, x, h, d_m)}


def tolerance(case):
    # About four times what an fp64 evaluation of the same inputs differs by: fp32 3e-7 to 7.4e-7; 16-bit storage 3.8e-4
    # to 4.4e-4 with fp32 results (intermediates are rounded to fp16 once each); 1.7e-3 where the result itself is bf16.
    if case["kind"] == "gather":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-6}
    return {"rel": 7e-3 if case["out"] == "bf16" else 2e-3}
