"""Workloads of the library for timing: what a program that quantizes a model has it do, through the
public entry points of `paper_2305_12356_amd.binding`, on the synthetic inputs of `mofq_inputs`.

A case is a dict of plain values with an "op":

  select      one layer (mofq_select_layer): weight-only by tensor error, or with tokens > 0 by layer output
  model       the linear layers of decoder blocks in one call (mofq_select_layers, a second stream given)
  model_wa    the same with activations, W8A8 (mofq_select_layers_wa)
  units       one layer, format per scale unit (mofq_select_units)
  quantize    one tensor in one format (mofq_quantize)
  calibrate   calibration batches folded into one magnitude, then the select of an unseen batch with it
"""
from __future__ import annotations

import math

import torch

import mofq_inputs as mi
from paper_2305_12356_amd import binding as mq

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
GRANS = {"tensor": mq.PER_TENSOR, "channel": mq.PER_CHANNEL, "group": mq.PER_GROUP}
PAIRS = {4: [mq.INT4, mq.FP4_E2M1], 8: [mq.INT8, mq.FP8_E4M3]}
METRICS = {"tensor": mq.ERR_TENSOR, "output": mq.ERR_LAYER_OUTPUT, "output_fp8_unit": mq.ERR_LAYER_OUTPUT_FP8_UNIT,
           "output_w_only": mq.ERR_LAYER_OUTPUT_W_ONLY}


def _case(op, **kw):
    c = dict(op=op, dtype="f16", bits=4, gran="channel", group=0, scale_f16=False, n_clip=1, tokens=0, metric="tensor",
             blocks=0, hidden=0, ffn=0, rows=0, cols=0)
    c.update(kw)
    return c


def listed():
    cases = [
        # one small fp32 weight, absmax scales: launch latency and host time of a single-layer call
        _case("select", name="absmax_f32_1024", dtype="f32", rows=1024, cols=1024),
        # an activation of a few tokens quantized on the fly, per tensor (decode)
        _case("quantize", name="act_e4m3_16tok", dtype="bf16", bits=8, gran="tensor", rows=16, cols=4096),
        # static calibration of one layer's input over four batches, then the select of an unseen one
        _case("calibrate", name="calibrate_2048tok", dtype="bf16", bits=8, gran="tensor", rows=2048, cols=4096, blocks=4),
        # a large fp32 matrix with absmax scales (no search): bound by memory
        _case("select", name="absmax_f32_16384", dtype="f32", rows=16384, cols=16384),
        # 8-bit weight-only search on a ragged bf16 layer
        _case("select", name="search8_ragged", dtype="bf16", bits=8, rows=3001, cols=5000, n_clip=50),
        # 4-bit weight-only search on a ragged bf16 layer, one call for the layer
        _case("select", name="search4_ragged", dtype="bf16", rows=1237, cols=5000, n_clip=100),
        # 4-bit weight-only select of decoder blocks: per-channel scales, 100 clip ratios
        _case("model", name="search4_7b_8blocks", blocks=8, hidden=4096, ffn=11008, n_clip=100),
        _case("model", name="search4_65b_2blocks", blocks=2, hidden=8192, ffn=22016, n_clip=100),
        # the same with fp16 scales per group of 128, 50 clip ratios
        _case("model", name="group128_7b_block", blocks=1, hidden=4096, ffn=11008, gran="group", group=128, scale_f16=True,
              n_clip=50),
        # W8A8 select of decoder blocks by layer output, 2048 tokens, low-bit matrix cores
        _case("model_wa", name="w8a8_7b_2blocks", dtype="bf16", bits=8, gran="tensor", blocks=2, hidden=4096, ffn=11008,
              tokens=2048, metric="output_fp8_unit"),
        # W8A8 select of one ragged layer with the exact E4M3 product
        _case("select", name="w8a8_exact_ragged", dtype="bf16", bits=8, gran="tensor", rows=3000, cols=5056, tokens=777,
              metric="output"),
        # weight-only select by layer output (16-bit input), one MLP projection
        _case("select", name="w4a16_output_gate", dtype="bf16", rows=11008, cols=4096, tokens=2048, metric="output_w_only"),
    ]
    return cases


def _log(rng, lo, hi):
    """Log-uniform integer in [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, m):
    """Log-uniform multiple of m in [lo, hi]."""
    return max(m, _log(rng, lo, hi) // m * m)


def draw(rng):
    kind = rng.choice(["absmax", "act", "calibrate", "search8", "search4", "search4_model", "group", "wa", "wa_model", "w4a16"])
    if kind == "absmax":
        cols = _mult(rng, 256, 16384, 8)
        rows = _log(rng, 64, 16384)
        return _case("select", dtype=rng.choice(["f32", "f32", "f16", "bf16"]), bits=rng.choice([4, 4, 8]), rows=rows, cols=cols)
    if kind == "act":
        return _case("quantize", dtype=rng.choice(["bf16", "f16"]), bits=8, gran="tensor", rows=_log(rng, 1, 4096),
                     cols=_mult(rng, 1024, 11008, 8))
    if kind == "calibrate":
        return _case("calibrate", dtype="bf16", bits=8, gran="tensor", rows=_log(rng, 64, 4096), cols=_mult(rng, 1024, 11008, 8),
                     blocks=rng.randint(1, 8))
    if kind == "search8":
        return _case("select", dtype=rng.choice(["bf16", "f16", "f32"]), bits=8, rows=_log(rng, 128, 4096),
                     cols=_mult(rng, 512, 11008, 8), n_clip=rng.randint(10, 100))
    if kind == "search4":
        return _case("select", dtype=rng.choice(["f16", "bf16", "f16", "bf16", "f32"]), rows=_log(rng, 128, 11008),
                     cols=_mult(rng, 512, 22016, 8), n_clip=rng.randint(10, 128), scale_f16=rng.random() < 0.3)
    if kind == "search4_model":
        hidden = _mult(rng, 1024, 8192, 64)
        return _case("model", dtype=rng.choice(["f16", "bf16"]), blocks=rng.randint(1, 2), hidden=hidden,
                     ffn=int(hidden * rng.uniform(2.5, 3.0)) // 32 * 32 if hidden < 8192 else 22016, n_clip=rng.randint(20, 128))
    if kind == "group":
        g = rng.choice([128, 128, 64, 32, 256])
        op = rng.choice(["units", "select", "model"])
        if op == "model":
            hidden = 256 * rng.randint(4, 14)
            return _case("model", dtype=rng.choice(["f16", "bf16"]), gran="group", group=g, scale_f16=True, blocks=1, hidden=hidden,
                         ffn=int(hidden * rng.uniform(2.5, 3.0)) // 256 * 256, n_clip=rng.randint(10, 64))
        return _case(op, dtype=rng.choice(["f16", "bf16", "f32"]), gran="group", group=g, scale_f16=rng.random() < 0.7,
                     rows=_log(rng, 64, 8192), cols=256 * rng.randint(2, 43), n_clip=rng.randint(10, 64))
    if kind == "wa":
        return _case("select", dtype="bf16", bits=8, gran=rng.choice(["tensor", "tensor", "channel"]), rows=_log(rng, 512, 11008),
                     cols=_mult(rng, 512, 11008, 64), tokens=_log(rng, 64, 2048), metric=rng.choice(["output", "output_fp8_unit"]))
    if kind == "wa_model":
        hidden = _mult(rng, 1024, 4096, 64)
        return _case("model_wa", dtype="bf16", bits=8, gran="tensor", blocks=rng.randint(1, 2), hidden=hidden,
                     ffn=int(hidden * rng.uniform(2.5, 2.6875)) // 64 * 64, tokens=_log(rng, 128, 2048),
                     metric=rng.choice(["output", "output_fp8_unit"]))
    return _case("select", dtype="bf16", rows=_log(rng, 512, 11008), cols=_mult(rng, 512, 8192, 64), tokens=_log(rng, 64, 2048),
                 metric="output_w_only", n_clip=rng.choice([1, 1, 20]))


def _shapes(c):
    """[rows, cols] of the case's weights and, per weight, the index of the activation it shares."""
    if c["op"] not in ("model", "model_wa"):
        return [(c["rows"], c["cols"])], [0]
    h, f = c["hidden"], c["ffn"]
    # q, k, v share the block's input; o; gate and up share the MLP's input; down
    shapes = [(h, h), (h, h), (h, h), (h, h), (f, h), (f, h), (h, f)] * c["blocks"]
    act = [4 * b + a for b in range(c["blocks"]) for a in (0, 0, 0, 1, 2, 2, 3)]
    return shapes, act


def _cfg(c):
    return mq.Cfg(GRANS[c["gran"]], mi.clip_ratios(c["n_clip"]), c["group"], c["scale_f16"])


def _round(n, m):
    return (n + m - 1) // m * m


def _outputs(shapes, bits, cfg):
    """Buffers for the quantized tensors side by side (a program that keeps a whole quantized model),
    every tensor's part 16-byte aligned; returns the parts and the buffers."""
    nb = [r * k // 2 if bits == 4 else r * k for r, k in shapes]
    nu = [mq.num_units(r, k, cfg.gran, cfg.group_size) for r, k in shapes]
    whole = {"codes": torch.zeros(sum(_round(n, 16) for n in nb), dtype=torch.uint8, device=DEV),
             "scales": torch.zeros(sum(_round(n, 8) for n in nu), dtype=torch.float16 if cfg.scale_f16 else torch.float32, device=DEV),
             "clip_idx": torch.zeros(sum(_round(n, 8) for n in nu), dtype=torch.int32, device=DEV),
             "unit_err": torch.zeros(sum(_round(n, 8) for n in nu), dtype=torch.float64, device=DEV)}
    parts, b, u = [], 0, 0
    for cb, cu in zip(nb, nu):
        parts.append(mq.QBuffers(whole["codes"][b:b + cb], whole["scales"][u:u + cu], whole["clip_idx"][u:u + cu],
                                 whole["unit_err"][u:u + cu]))
        b, u = b + _round(cb, 16), u + _round(cu, 8)
    return parts, whole


def _results(n):
    """Result records, and their fields as tensors: the choice, and the errors with the reference energy."""
    r = mq.alloc_result(DEV, n)
    return r, {"choice": r.view(torch.int32)[:, :2], "errors": r.view(torch.float64)[:, 1:]}


def _bytes(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c, op = case, case["op"]
    cfg, cands, dtype = _cfg(c), PAIRS[c["bits"]], DTYPES[c["dtype"]]
    seed = int(seed) * 4096
    s = {"op": op, "cfg": cfg, "cands": cands, "metric": METRICS[c["metric"]]}
    if op == "quantize":
        s["x"] = mi.activations(c["rows"], c["cols"], seed=seed, dtype=dtype, device=DEV)
        (s["to"],), s["out"] = _outputs([(c["rows"], c["cols"])], c["bits"], cfg)
        s["err"] = torch.zeros(1, dtype=torch.float64, device=DEV)
        s["out"]["tensor_err"] = s["err"]
        s["ws"] = _bytes(mq.workspace_bytes(s["x"], None, 1, mq.ERR_TENSOR, cfg))
        return s
    if op == "calibrate":
        batches = mi.activation_batches(c["blocks"] + 1, c["rows"], c["cols"], seed=seed, dtype=dtype, device=DEV)
        s["seen"], s["x"] = batches[:-1], batches[-1]
        (s["to"],), s["out"] = _outputs([(c["rows"], c["cols"])], c["bits"], cfg)
        s["absmax"] = torch.zeros(1, dtype=torch.float32, device=DEV)
        s["result"], fields = _results(1)
        s["out"].update(fields, absmax=s["absmax"])
        s["ws"] = _bytes(mq.workspace_bytes(s["x"], None, 2, mq.ERR_TENSOR, cfg))
        return s
    shapes, act = _shapes(c)
    # layers differ in how heavy their tails are, so that both outcomes of the select occur
    ws = [mi.llama_like_weight(r, k, seed=seed + i, dtype=dtype, device=DEV, outlier_frac=mi.layer_outlier_frac(1, i // 7, i % 7))
          for i, (r, k) in enumerate(shapes)]
    to, s["out"] = _outputs(shapes, c["bits"], cfg)
    s["result"], fields = _results(len(shapes))
    s["out"].update(fields)
    xs = {}
    for i, a in enumerate(act):
        if c["tokens"] and a not in xs:
            xs[a] = mi.activations(c["tokens"], shapes[i][1], seed=seed + 2048 + a, device=DEV)
    s["w"], s["x"], s["to"] = ws[0], xs.get(0), to[0]
    if op == "model":
        s["batch"] = mq.LayerBatch(ws, to)
        s["side"] = torch.cuda.Stream()
        s["ws"] = _bytes(s["batch"].workspace_bytes(len(cands), cfg))
    elif op == "units":
        s["unit_format"] = torch.zeros(to[0].scales.numel(), dtype=torch.uint8, device=DEV)
        s["mixed"] = torch.zeros(1, dtype=torch.float64, device=DEV)
        s["out"].update(unit_format=s["unit_format"], mixed_err=s["mixed"])
        s["ws"] = _bytes(mq.select_units_workspace_bytes(ws[0], len(cands), cfg))
    else:
        x_to = None
        if c["tokens"] and c["metric"] != "output_w_only":
            xcfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
            x_to, x_out = _outputs([(c["tokens"], k) for _, k in shapes], c["bits"], xcfg)
            s["out"].update({"x_" + k: v for k, v in x_out.items()})
        s["x_to"] = x_to[0] if x_to else None
        if op == "model_wa":
            s["batch"] = mq.WaLayerBatch(ws, [xs[a] for a in act], to, x_to)
            s["ws"] = _bytes(s["batch"].workspace_bytes(len(cands), s["metric"], cfg))
        else:
            s["ws"] = _bytes(mq.workspace_bytes(ws[0], s["x"], len(cands), s["metric"], cfg))
    return s


def run(state):
    s, op = state, state["op"]
    if op == "select":
        mq.select_layer(s["w"], s["x"], s["cands"], s["metric"], s["cfg"], s["to"], s["x_to"], s["result"], s["ws"])
    elif op == "model":
        mq.select_layers(s["batch"], s["cands"], s["cfg"], s["result"], s["ws"], side_stream=s["side"])
    elif op == "model_wa":
        mq.select_layers_wa(s["batch"], s["cands"], s["metric"], s["cfg"], s["result"], s["ws"])
    elif op == "units":
        mq.select_units(s["w"], s["cands"], s["cfg"], s["to"], s["unit_format"], s["result"], s["mixed"], s["ws"])
    elif op == "quantize":
        mq.quantize(s["x"], mq.FP8_E4M3, s["cfg"], s["to"], s["err"], s["ws"])
    else:
        s["absmax"].zero_()
        for x in s["seen"]:
            mq.calibrate_absmax(x, s["absmax"], s["ws"])
        mq.select_calibrated(s["x"], s["cands"], s["absmax"], s["to"], s["result"], s["ws"])
    return s["out"]


def work(case):
    c = case
    shapes, act = _shapes(c)
    size = 4 if c["dtype"] == "f32" else 2
    n_bytes, flops = 0, 0
    for r, k in shapes:
        units = mq.num_units(r, k, GRANS[c["gran"]], c["group"])
        n_bytes += r * k * size + r * k * c["bits"] // 8 + units * ((2 if c["scale_f16"] else 4) + 4 + 8)
        # one scoring of each of the two formats: scale, round, clamp, residual (2), square and add (2)
        flops += 14 * r * k
        if c["tokens"]:
            # the reference product and the two quantized ones
            flops += 3 * 2 * c["tokens"] * r * k
            if c["metric"] != "output_w_only":
                n_bytes += c["tokens"] * k            # the activation's codes, written for every layer
    if c["tokens"]:
        n_bytes += sum(2 * c["tokens"] * k for k in {a: shapes[i][1] for i, a in enumerate(act)}.values())
    if c["op"] == "calibrate":
        n_bytes += c["blocks"] * c["rows"] * c["cols"] * size
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # codes, scales, indices and choices are exact everywhere; tensor errors are fp64 sums, layer-output
    # errors sums of squares of fp32-accumulated matrix products
    return {"rel": 1e-5 if case["tokens"] else 1e-9}
