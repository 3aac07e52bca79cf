#!/usr/bin/env python3
"""Benchmark of the MoFQ quantize-and-score / format-select hot path on one MI355X.

Headline workload (`config.workload`): the LLaMA-7B-shaped weight set, fp16, 32 blocks x 7
linears = 224 tensors, 4-bit weight-only, per-channel scales searched over 100 clip ratios
in [0.5, 1], INT4 vs FP4-E2M1, per-layer select and emit of the codes.  A step is one pass
of the whole path (scale search + select + emit) over all 224 tensors, which are resident in
HBM before the timed region starts.

Prints ONE JSON line: the elements x candidates scored per second (and the full-model select
time), the roofline of the dominant kernel measured with HIP events inside the timed region,
the device ceilings measured in the same run (`ceilings`: copy, vector FMA, matrix cores),
the CPU oracle timed on a bounded sample of the same workload (1 thread and all threads),
and, under `secondary`, the other configurations of the same path, each timed the same way:
the memory-bound single-candidate case, the group-wise search, W8A8 by layer-output error
(exact and with the fp8 matrix cores), the weight-only layer-output select, and the
65B-shaped set.

`--workload NAME` runs one of them alone (its own JSON line, same keys).
`--full-parity` is not a benchmark: it holds every linear of a block range to the oracle
(all rows: format choice, both error sums, codes, scales, clip indices) and prints a summary.
"""
from __future__ import annotations

import argparse
import json
import os
import subprocess
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

N_CLIP = 100
N_CLIP_GROUP = 50
GROUP = 128
TOKENS = 2048
N_FMT = 2
HBM_PEAK_GBPS = 8000.0
# Published dense matrix-core peaks (TFLOP/s or TOP/s) per operand type.
MFMA_PEAK = {"bf16": 2500.0, "int8": 5000.0, "fp8": 5000.0}
# Work of the EXHAUSTIVE scale search per element, candidate and format: scale (1 multiply),
# round (1), clamp/saturate (1), residual x - g*s (2), error accumulation d*d + acc (2).  The
# per-channel search does not execute it (it builds a histogram of each row's bit patterns and
# reads every candidate's level counts and sums from its prefixes), so this prices an
# equivalent rate, reported under its own key, never as a utilisation.
FLOPS_PER_ELEM_CAND_FMT = 7
TAIL_SPREAD = False   # set from --tail-spread

# Counter-derived facts about the search kernels, measured by rocprofv3 runs of this command (not in the run that
# prints them): where they come from is printed beside them.  sweep_hist_kernel, 4096-column rows: a launch of 8192
# rows and more also writes the rows' codes (0.5 byte per element).
SEARCH_KERNEL_COUNTERS = {
    "from": "profiles/w_only_hist_kernel_counters.txt, profiles/w_only_7b_k100_hbm_traffic.txt",
    "read_per_input_byte": 374276.0 / (46592 * 4096 * 2 / 1024),     # FETCH_SIZE, scaled by a plain copy
    "write_bytes_per_row": 896.0 * 1024 / 4096,                      # WRITE_SIZE: records alone
    "write_bytes_per_row_with_codes": 104104.0 * 1024 / 46592,
    "rows_with_codes": 8192,
    "valu_instr_per_wave": 904.0,                                    # SQ_INSTS_VALU / SQ_WAVES, 4096-column instance
}
# sweep_group_bits_kernel, fp16 groups of 128, 50 ratios: a wave takes four groups (a mean over this recipe: how many gaps
# of the coarse search are looked at depends on the data)
GROUP_KERNEL_COUNTERS = {"from": "profiles/w4_group128_7b_k50_kernel_stats.txt", "valu_instr_per_wave": 1356.0}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=8)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--model", default="7b", choices=["7b", "65b"],
                    help="65b: 560 linears, 129.5 GB of fp16 weights resident in HBM")
    ap.add_argument("--workload", default="all",
                    choices=["all", "w4_channel", "w4_group128", "w8a8", "w4a16_output", "k1_hbm", "fp4_variants",
                             "w4_units", "ceilings"])
    ap.add_argument("--exact-e4m3", action="store_true",
                    help="w8a8: E4M3 product from the grid values on the bf16 matrix cores (MOFQ_ERR_LAYER_OUTPUT) "
                         "instead of the E4M3 codes on the fp8 matrix cores (MOFQ_ERR_LAYER_OUTPUT_FP8_UNIT)")
    ap.add_argument("--fp8-unit", action="store_true", help="w8a8: the default (kept for older command lines)")
    ap.add_argument("--blocks", type=int, default=0, help="debug: use only the first N blocks")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-65b", action="store_true", help="all: leave the 65B-shaped set out of `secondary`")
    ap.add_argument("--single-stream", action="store_true",
                    help="w4_channel: no second stream (kernels run one at a time; for counter runs)")
    ap.add_argument("--tail-spread", action="store_true",
                    help="model-shaped sets with a per-layer share of heavy-tail entries (both outcomes of the "
                         "4-bit select occur) instead of 0.05 %% in every layer")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run one plain 1 GiB device copy (reference for rocprofv3 byte counters)")
    ap.add_argument("--full-parity", action="store_true",
                    help="hold every linear of --block-list to the oracle on all rows and print a summary")
    ap.add_argument("--block-list", default="0", help="full-parity: blocks, e.g. 0,39,79 or 0:11")
    ap.add_argument("--head", default=None, help="commit to record in the output where no git checkout is at hand")
    return ap.parse_args()


HEAD_OVERRIDE = None


def git_head():
    if HEAD_OVERRIDE:
        return HEAD_OVERRIDE
    try:
        return subprocess.run(["git", "rev-parse", "--short", "HEAD"], cwd=ROOT, capture_output=True,
                              text=True, timeout=5).stdout.strip() or None
    except Exception:
        return None


# ---- device ceilings ----------------------------------------------------------------

def measure_ceilings(dev):
    """Stream copy, vector FMA and matrix-core loop rates of this device, with the library's
    micro-kernels, HIP events around each launch, best of three."""
    import torch
    from paper_2305_12356_amd import binding as mq

    stream = torch.cuda.current_stream()
    buf = torch.empty(2 << 30, dtype=torch.uint8, device=dev)      # copy: 1 GiB -> 1 GiB
    buf.zero_()

    def rate(kind, iters):
        best = 0.0
        for rep in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            work = mq.device_ceiling(kind, buf, iters, stream)
            e1.record(stream)
            torch.cuda.synchronize()
            if rep:                                             # the first launch warms up
                best = max(best, work / (e0.elapsed_time(e1) * 1e-3))
        return best

    out = {
        "copy_GBps": rate(mq.CEILING_COPY, 4) / 1e9,
        "read_GBps": rate(mq.CEILING_READ, 4) / 1e9,
        "valu_fma_f32_TFLOPs": rate(mq.CEILING_FMA_F32, 20000) / 1e12,
        "valu_fma_f64_TFLOPs": rate(mq.CEILING_FMA_F64, 10000) / 1e12,
        "mfma_bf16_TFLOPs": rate(mq.CEILING_MFMA_BF16, 4000) / 1e12,
        "mfma_int8_TOPs": rate(mq.CEILING_MFMA_INT8, 4000) / 1e12,
        "mfma_fp8_TFLOPs": rate(mq.CEILING_MFMA_FP8, 4000) / 1e12,
    }
    # one fused multiply-add instruction of a wave = 128 flop: the issue rate behind the FMA figure
    out["valu_wave_instr_per_s"] = out["valu_fma_f32_TFLOPs"] * 1e12 / 128.0
    out["note"] = ("measured in this run with the library's micro-kernels (HIP events, best of 3): 1 GiB device copy "
                   "(read + write bytes), 2 GiB read-only pass, register-only fused multiply-add loops (one plain instruction per wave and "
                   "operation: the packed fp32 form behind the published 157.3 TFLOP/s is not used), register-only "
                   "32x32 matrix-instruction loops")
    del buf
    return out


# ---- CPU oracle beside it -------------------------------------------------------------

def cpu_baseline(weights, outs, clip, cands):
    """Time the oracle (as it stands) on a bounded sample of the same tensors, with all host
    threads and with one, and check the library's results on those rows against it."""
    import numpy as np
    import mofq_inputs as mi
    from oracle import mofq_oracle as orc
    from tests.gpu_util import compare_quantized, scales_to_f32

    # rows of block 0: q (4096 cols), gate (4096 cols), down (11008 cols)
    plan = [(0, 4096), (4, 3072), (6, 2048)]     # about 11 s of oracle time on 16 host threads
    threads = orc.max_threads()
    total_ec, total_t, checked, band = 0, 0.0, 0, 0
    desc = []
    for idx, n_rows in plan:
        w_dev, out, res = weights[idx], outs[idx][0], outs[idx][1]
        n_rows = min(n_rows, w_dev.shape[0])
        cols = w_dev.shape[1]
        w32 = mi.to_f32_numpy(w_dev[:n_rows])
        t0 = time.perf_counter()
        ref = [orc.quantize(w32, f, orc.PER_CHANNEL, clip, want_table=True, threads=threads)
               for f in cands]
        total_t += time.perf_counter() - t0
        total_ec += n_rows * cols * N_CLIP * N_FMT
        desc.append(f"{n_rows}x{cols}")
        best = res.best
        codes = out.codes[: n_rows * cols // 2].cpu().numpy()
        un = np.empty(n_rows * cols, dtype=np.uint8)
        un[0::2] = codes & 0xF
        un[1::2] = codes >> 4
        band += compare_quantized(w32, cands[best], orc.PER_CHANNEL, 0, False, clip, ref[best],
                                  un.reshape(n_rows, cols), scales_to_f32(out.scales[:n_rows]),
                                  out.clip_idx[:n_rows].cpu().numpy(),
                                  out.unit_err[:n_rows].cpu().numpy())
        checked += n_rows
    # one thread: the first 320 rows of q
    one_rows = 320
    w32 = mi.to_f32_numpy(weights[0][:one_rows])
    t0 = time.perf_counter()
    for f in cands:
        orc.quantize(w32, f, orc.PER_CHANNEL, clip, threads=1)
    one_t = time.perf_counter() - t0
    one_rate = one_rows * w32.shape[1] * N_CLIP * N_FMT / one_t
    return {
        "value": total_ec / total_t, "unit": "elem*cand/s", "cores": threads, "kind": "oracle",
        "sample": "first rows of block 0 q/gate/down (" + ", ".join(desc) +
                  "), both formats x 100 clip ratios, full oracle search",
        "seconds": round(total_t, 3),
        "rows_checked_bit_exact": checked, "near_tie_rows": band,
        "one_thread": {"value": one_rate, "unit": "elem*cand/s", "cores": 1, "seconds": round(one_t, 3),
                       "sample": f"first {one_rows} rows of block 0 q, both formats x 100 clip ratios"},
    }


# ---- weight-only, tensor error: per channel and per group ------------------------------------

def make_weights(shapes, dev, dtype=None):
    import torch
    import mofq_inputs as mi
    return [mi.model_weight(1, b, mi.LINEAR_NAMES.index(name), o, n, dtype=dtype or torch.float16, device=dev,
                            tail_spread=TAIL_SPREAD)
            for b, name, o, n in shapes]


def run_w4(args, shapes, dev, weights, group, model, steps, warmup, ceilings=None, want_cpu=False):
    import torch
    import mofq_inputs as mi
    from paper_2305_12356_amd import binding as mq

    n_clip = N_CLIP_GROUP if group else N_CLIP
    clip = mi.clip_ratios(n_clip)
    cands = [mq.INT4, mq.FP4_E2M1]
    cfg = mq.Cfg(mq.PER_GROUP, clip, GROUP, True) if group else mq.Cfg(mq.PER_CHANNEL, clip)
    qouts = [mq.alloc_qbuffers(o, n, 4, cfg, dev) for _, _, o, n in shapes]
    results = mq.alloc_result(dev, len(shapes))
    # one call for the whole model (mofq_select_layers): the per-tensor reduce / select /
    # per-unit outputs of up to 12 tensors share a launch, and so do the searches of those of
    # them that have one row length
    batch = mq.LayerBatch(weights, qouts)
    ws = torch.empty(batch.workspace_bytes(len(cands), cfg), dtype=torch.uint8, device=dev)
    n_elems = sum(o * n for _, _, o, n in shapes)
    stream = torch.cuda.current_stream()
    # default priority: select + code emission beside the next batch's searches
    side = None if args.single_stream else torch.cuda.Stream()

    # the events the library records around each search launch, created (and recorded once,
    # so that they exist) before the timed region
    ev_pool = []
    for _ in range(steps):
        e0 = [torch.cuda.Event(enable_timing=True) for _ in weights]
        e1 = [torch.cuda.Event(enable_timing=True) for _ in weights]
        for e in e0 + e1:
            e.record()
        ev_pool.append((e0, e1))

    def step(events=None):
        e0 = e1 = None
        if events is not None:
            e0, e1 = ev_pool.pop()
            events.extend((i, a, b) for i, (a, b) in enumerate(zip(e0, e1)))
        mq.select_layers(batch, cands, cfg, results, ws, stream, e0, e1, side_stream=side)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    events = []
    t0 = time.perf_counter()
    for _ in range(steps):
        step(events)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0

    ms_per_step = elapsed / steps * 1e3
    elem_cand = n_elems * n_clip * N_FMT
    value = elem_cand / (elapsed / steps)

    # ---- dominant kernel: the search launches over the most common row length -----------
    # Duration from the HIP events the library recorded around each launch: the begin event of a
    # launch's first tensor, the end event of its last.
    first = batch.search_groups(cands)
    last = {f: i for i, f in enumerate(first)}
    by_cols = {}
    for step_i in range(steps):
        ev = events[step_i * len(shapes):(step_i + 1) * len(shapes)]
        for f, l in last.items():
            members = [i for i in range(f, l + 1) if first[i] == f]
            elems = sum(shapes[i][2] * shapes[i][3] for i in members)
            rows = sum(shapes[i][2] for i in members)
            by_cols.setdefault(shapes[f][3], []).append((elems, ev[f][1].elapsed_time(ev[l][2]) * 1e-3, rows))
    dom_cols = max(by_cols, key=lambda c: sum(e for e, _, _ in by_cols[c]))
    dom = by_cols[dom_cols]
    dom_elems = sum(e for e, _, _ in dom)
    dom_time = sum(t for _, t, _ in dom)
    dom_rows = sum(r for _, _, r in dom)
    alg_bytes_per_launch = dom_elems * 2 / len(dom)               # 2 bytes per element, read once
    achieved = dom_elems * 2 / dom_time / 1e9
    search_time = sum(t for v in by_cols.values() for _, t, _ in v) / steps
    roofline = {
        "bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
        "frac": achieved / HBM_PEAK_GBPS, "traffic": None,
        "kernel": (f"sweep_group_bits_kernel<F16, INT4, FP4_E2M1, {GROUP}, 32-bit words> on {dom_cols}-column rows" if group else
                   f"sweep_hist_kernel<F16, INT4, FP4_E2M1> instance for {dom_cols}-column rows"),
        "limited_by": "vector instruction issue, not bytes: " +
                      (f"per group a table of its bit patterns, then 7 or 8 boundary look-ups for each of the {n_clip} x {N_FMT} candidates that "
                       f"its coarse search of {GROUP // 8} ratios leaves" if group else
                       f"per row a histogram of its bit patterns, then {n_clip} x {N_FMT} candidates x 7 or 8 boundary look-ups"),
        "avg_launch_ms": dom_time / len(dom) * 1e3, "launches": len(dom),
        "algorithmic_bytes_per_launch": alg_bytes_per_launch,
        "algorithmic_bytes_per_elem": 2,
        "search_ms_per_step": search_time * 1e3,
        # what the exhaustive search would need for the same result: an equivalent rate, not a utilisation
        "exhaustive_equivalent": {
            "TFLOPs": dom_elems * n_clip * N_FMT * FLOPS_PER_ELEM_CAND_FMT / dom_time / 1e12,
            "flops_per_elem_cand_fmt": FLOPS_PER_ELEM_CAND_FMT,
            "note": "flop of scoring every element x candidate x format one by one (7 each) over the launch "
                    "time; the kernel reaches the same result with far fewer instructions (a table of the "
                    "row's or group's bit patterns + prefix look-ups), so this is not a fraction of any peak",
        },
    }
    if ceilings:
        roofline["frac_of_measured_read"] = achieved / ceilings["read_GBps"]
    if not group and model == "7b" and dom_cols == 4096:
        c = SEARCH_KERNEL_COUNTERS
        written = sum(r * c["write_bytes_per_row_with_codes" if r >= c["rows_with_codes"] else "write_bytes_per_row"] for _, _, r in dom)
        roofline["traffic"] = alg_bytes_per_launch * c["read_per_input_byte"] + written / len(dom)
        roofline["traffic_from"] = {"file": c["from"], "measured_in_this_run": False,
                                    "how": "rocprofv3 FETCH_SIZE / WRITE_SIZE per row, scaled by a plain copy, "
                                           "times the rows of this run's launches (codes written by most of them included)"}
    if ceilings and model == "7b":
        # what binds the kernel: wave instructions issued per second (4 waves per row or a wave per 4 groups, the
        # instruction count per wave from the counters profile) against the rate of the plain FMA loop of this run
        c = GROUP_KERNEL_COUNTERS if group else SEARCH_KERNEL_COUNTERS
        waves = dom_elems / (4 * GROUP) if group else 4 * dom_rows
        rate = c["valu_instr_per_wave"] * waves / dom_time
        roofline["vector_issue"] = {"wave_instr_per_s": rate, "ceiling_measured": ceilings["valu_wave_instr_per_s"],
                                    "frac": rate / ceilings["valu_wave_instr_per_s"],
                                    "instr_per_wave": c["valu_instr_per_wave"],
                                    "instr_per_wave_from": {"file": c["from"], "measured_in_this_run": False}}

    res = mq.read_results(results)
    fp_pct = 100.0 * sum(1 for r in res if r.best == 1) / len(res)
    out = {
        "metric": f"weight-elems x candidates scored/sec (+ LLaMA-{model.upper()} full-model MoFQ select time)",
        "value": value, "unit": "elem*cand/s",
        "n_gpus": 1, "steps": steps, "warmup": warmup, "ms_per_step": ms_per_step,
        "select_time_s": ms_per_step / 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 decisions, f64 errors", "data": "synthetic",
        "config": {"workload": ("LLaMA-7B-shaped fp16 weight set, "
                                f"{len(shapes)} linears, {n_elems} weights, 4-bit W-only group-wise "
                                "(128 along the input dim, fp16 scales), 50 clip ratios in [0.5,1], "
                                "INT4 vs FP4-E2M1, per-layer select + emit") if group else
                               (("LLaMA-65B-shaped" if model == "65b" else
                                 "LLaMA-7B-shaped") + " fp16 weight set, "
                                f"{len(shapes)} linears, {n_elems} weights, 4-bit W-only per-channel, "
                                "100 clip ratios in [0.5,1], INT4 vs FP4-E2M1, per-layer select + emit"),
                   "n_clip": n_clip, "formats": ["INT4", "FP4_E2M1"], "fp_percent": fp_pct,
                   "weights": ("per-layer share of heavy-tail entries, log-uniform over [1.3e-5, 5e-3] (--tail-spread)"
                               if TAIL_SPREAD else "rows N(0, sigma^2), sigma ~ U(0.01, 0.04), 0.05 % Student-t(3) outliers")},
        "roofline": roofline,
    }
    if want_cpu:
        outs = [(qouts[i], res[i]) for i in range(len(shapes))]
        out["cpu_baseline"] = cpu_baseline(weights, outs, clip, cands)
    return out


# ---- layer-output error: weight-activation and the weight-only variant -------------------------

def run_w8a8(args, shapes, dev, weights, w_only, fp8_unit, steps, warmup, ceilings=None):
    """W8A8: per linear, X [2048, in] bf16 with outlier channels, W bf16; per-tensor
    INT8 vs FP8-E4M3 for both; layer-output error through the matrix cores; select + emit.
    With w_only: the weight-only select by layer-output error (X stays bf16; W per-channel
    absmax scales, INT4 vs FP4-E2M1)."""
    import torch

    import mofq_inputs as mi
    from paper_2305_12356_amd import binding as mq

    metric = mq.ERR_LAYER_OUTPUT_FP8_UNIT if fp8_unit else mq.ERR_LAYER_OUTPUT
    cands = [mq.INT8, mq.FP8_E4M3]
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    bits = 8
    if w_only:
        metric, cands, bits = mq.ERR_LAYER_OUTPUT_W_ONLY, [mq.INT4, mq.FP4_E2M1], 4
        cfg = mq.Cfg(mq.PER_CHANNEL, mi.clip_ratios(1))
    xcfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    results = mq.alloc_result(dev, len(shapes))
    stream = torch.cuda.current_stream()
    if w_only:
        xs = {}
        wouts = {}
        ws_bytes = 0
        for i, (b, name, o, n) in enumerate(shapes):
            if n not in xs:
                xs[n] = mi.activations(TOKENS, n, seed=mi.tensor_seed(3, 0, 0, n), device=dev)
            ws_bytes = max(ws_bytes, mq.workspace_bytes(weights[i], xs[n], len(cands), metric, cfg))
            # one output buffer per distinct weight shape (the codes are not read back here)
            if (o, n) not in wouts:
                wouts[(o, n)] = mq.alloc_qbuffers(o, n, bits, cfg, dev)
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)

        def step(events=None):
            for i, w in enumerate(weights):
                _, _, o, n = shapes[i]
                e0 = e1 = None
                if events is not None:
                    e0 = torch.cuda.Event(enable_timing=True)
                    e1 = torch.cuda.Event(enable_timing=True)
                    events.append((i, e0, e1))
                mq.select_layer(w, xs[n], cands, metric, cfg, wouts[(o, n)], None, results[i], ws, stream, e0, e1)
    else:
        # One activation per role of a decoder block, as in a model: q, k, v read the block's
        # input, o the attention output, gate and up the MLP input, down the MLP's hidden state.
        # Every layer has its own output buffers.
        role = {"q": 0, "k": 0, "v": 0, "o": 1, "gate": 2, "up": 2, "down": 3}
        acts = {}
        x_list = []
        for b, name, o, n in shapes:
            key = (role[name], n)
            if key not in acts:
                acts[key] = mi.activations(TOKENS, n, seed=mi.tensor_seed(3, 0, role[name], 1), device=dev)
            x_list.append(acts[key])
        w_outs = [mq.alloc_qbuffers(o, n, bits, cfg, dev) for _, _, o, n in shapes]
        x_outs = [mq.alloc_qbuffers(TOKENS, n, 8, xcfg, dev) for _, _, o, n in shapes]
        batch = mq.WaLayerBatch(weights, x_list, w_outs, x_outs)
        ws = torch.empty(batch.workspace_bytes(len(cands), metric, cfg), dtype=torch.uint8, device=dev)

        def step(events=None):
            e0 = e1 = None
            if events is not None:
                e0 = [torch.cuda.Event(enable_timing=True) for _ in shapes]
                e1 = [torch.cuda.Event(enable_timing=True) for _ in shapes]
                events.extend((i, e0[i], e1[i]) for i in range(len(shapes)))
            mq.select_layers_wa(batch, cands, metric, cfg, results, ws, stream, e0, e1)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    events = []
    t0 = time.perf_counter()
    for _ in range(steps):
        step(events)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed / steps * 1e3

    # dominant kernel: the fused three-product GEMM; one launch per linear
    mnk = sum(TOKENS * o * n for _, _, o, n in shapes)
    gemm_time = sum(e0.elapsed_time(e1) for _, e0, e1 in events) * 1e-3 / steps
    kinds = ["bf16", "bf16", "bf16"] if w_only else ["bf16", "int8", "fp8" if fp8_unit else "bf16"]
    flops = 2.0 * mnk * len(kinds)
    ideal = sum(2.0 * mnk / (MFMA_PEAK[k] * 1e12) for k in kinds)
    achieved = flops / gemm_time / 1e12
    peak = flops / ideal / 1e12
    res = mq.read_results(results)
    roofline = {
        "bound": "mfma", "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
        "frac": achieved / peak, "traffic": None,
        "kernel": ("wa_gemm_shared_kernel (reference, INT4 and E2M1 products of one linear, which share X)" if w_only else
                   "wa_gemm_kernel (reference, INT8-code and E4M3 products of one linear)"),
        "note": "three products per launch, " + " + ".join(kinds) + "; peak is the rate at which the "
                "three would finish if each ran at the published dense peak of its own type "
                "(bf16 2.5, int8 5.0, fp8 5.0 PFLOP/s)",
        "gemm_ms_per_step": gemm_time * 1e3, "launches": len(events),
        "flops_per_launch_avg": flops / len(shapes),
    }
    if ceilings:
        key = {"bf16": "mfma_bf16_TFLOPs", "int8": "mfma_int8_TOPs", "fp8": "mfma_fp8_TFLOPs"}
        ideal_m = sum(2.0 * mnk / (ceilings[key[k]] * 1e12) for k in kinds)
        roofline["frac_of_measured_mfma"] = ideal_m / gemm_time
    return {
        "metric": ("W4A16" if w_only else "W8A8") + " layer-output MoFQ select time over the LLaMA-7B linear shapes",
        "value": ms_per_step / 1e3, "unit": "s", "n_gpus": 1, "steps": steps,
        "warmup": warmup, "ms_per_step": ms_per_step, "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None,
        "dtype": ("bf16 reference product, 4-bit grid values on the bf16 matrix cores, f64 error sums" if w_only else
                  "bf16 reference product, int8 codes, " +
                  ("fp8 codes on the fp8 matrix cores" if fp8_unit else "e4m3 grid values on the bf16 matrix cores") +
                  ", f64 error sums"),
        "data": "synthetic",
        "config": {"workload": (f"weight-only select by layer-output error: {len(shapes)} linears of the LLaMA-7B shape, "
                                f"X [{TOKENS} x in] bf16 unquantized, W bf16, per-channel absmax scales, "
                                "INT4 vs FP4-E2M1, per-layer select + emit") if w_only else
                               (f"W8A8: {len(shapes)} linears of the LLaMA-7B shape, X [{TOKENS} x in] bf16 "
                                "with 6 outlier channels x60, W bf16, per-tensor INT8 vs FP8-E4M3, "
                                "layer-output error, per-layer select + emit"),
                   "fp8_product": ("E4M3 codes on the fp8 matrix cores, the activation's outlier columns in one K step "
                                   "on the bf16 matrix cores (MOFQ_ERR_LAYER_OUTPUT_FP8_UNIT)") if fp8_unit else
                                  "E4M3 grid values on the bf16 matrix cores (MOFQ_ERR_LAYER_OUTPUT)",
                   "fp_percent": 100.0 * sum(1 for r in res if r.best == 1) / len(res)},
        "roofline": roofline,
    }


def run_k1_hbm(args, dev, steps, warmup, ceilings=None):
    """The single-candidate case at a size that does not fit in the caches: one 16384 x 16384 fp32
    tensor, per-channel absmax scale (one candidate), INT4 vs FP4-E2M1, select + emit."""
    import torch

    import mofq_inputs as mi
    from paper_2305_12356_amd import binding as mq

    n = 16384
    w = mi.config0_weight(seed=0, rows=n, cols=n, device=dev)
    cfg = mq.Cfg(mq.PER_CHANNEL, mi.clip_ratios(1))
    cands = [mq.INT4, mq.FP4_E2M1]
    out = mq.alloc_qbuffers(n, n, 4, cfg, dev)
    res = mq.alloc_result(dev)
    ws = torch.empty(mq.workspace_bytes(w, None, 2, mq.ERR_TENSOR, cfg), dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream()
    for _ in range(warmup):
        mq.select_layer(w, None, cands, mq.ERR_TENSOR, cfg, out, None, res, ws, stream)
    torch.cuda.synchronize()
    events = []
    t0 = time.perf_counter()
    for _ in range(steps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        events.append((e0, e1))
        mq.select_layer(w, None, cands, mq.ERR_TENSOR, cfg, out, None, res, ws, stream, e0, e1)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed / steps * 1e3
    sweep_s = sum(e0.elapsed_time(e1) for e0, e1 in events) * 1e-3 / steps
    alg_bytes = n * n * 4 + n * n // 2      # read once, the codes written by the same kernel
    achieved = alg_bytes / sweep_s / 1e9
    r = mq.read_result(res)
    roofline = {
        "bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBPS,
        # FETCH_SIZE / WRITE_SIZE of this kernel, scaled by a plain copy's
        "traffic": (1048932 + 135129) * 1024.0,
        "traffic_from": {"file": "profiles/k1_hbm_fp32_16384_kernel_stats.txt", "measured_in_this_run": False},
        "kernel": "sweep_channel_single_kernel<F32, INT4, FP4_E2M1, 512 threads, 4 chunks>",
        "note": "algorithmic bytes = 4 B per element read and 0.5 B of codes written, once each, by the scoring kernel; "
                "the select, the per-channel outputs and the rows that change format follow (rest_ms_per_step)",
        "avg_launch_ms": sweep_s * 1e3, "launches": len(events),
        "algorithmic_bytes_per_launch": alg_bytes,
        "rest_ms_per_step": (elapsed / steps - sweep_s) * 1e3,
    }
    if ceilings:
        roofline["frac_of_measured_read"] = n * n * 4 / sweep_s / 1e9 / ceilings["read_GBps"]
    return {
        "metric": "weight-elems x candidates scored/sec (memory-bound case: one scale candidate)",
        "value": n * n * N_FMT / (elapsed / steps), "unit": "elem*cand/s", "n_gpus": 1,
        "steps": steps, "warmup": warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 decisions, f64 errors", "data": "synthetic",
        "config": {"workload": "one 16384 x 16384 fp32 tensor (1 GiB): N(0, 0.02^2), 0.1 % of "
                               "entries x10, per-channel absmax scale, INT4 vs FP4-E2M1, tensor error, select + emit",
                   "best": int(r.best), "err": [float(r.err[0]), float(r.err[1])]},
        "roofline": roofline,
    }


def run_fp4_variants(args, shapes, dev):
    """Section 4.2 in kind, on the synthetic 7B-shaped set: tensor error of the redesigned
    FP4 (Table 1, without NaN/Inf) against the IEEE-aligned FP4, per-channel absmax scales,
    and how many layers prefer each FP4 over INT4."""
    import torch

    import mofq_inputs as mi
    from paper_2305_12356_amd import binding as mq

    cfg = mq.Cfg(mq.PER_CHANNEL, mi.clip_ratios(1))
    sets = {"redesigned": [mq.INT4, mq.FP4_E2M1], "ieee": [mq.INT4, mq.FP4_E2M1_IEEE]}
    results = {k: mq.alloc_result(dev, len(shapes)) for k in sets}
    stream = torch.cuda.current_stream()
    ws = out = None
    t0 = time.perf_counter()
    for i, (b, name, o, n) in enumerate(shapes):
        w = mi.model_weight(1, b, mi.LINEAR_NAMES.index(name), o, n, device=dev, tail_spread=TAIL_SPREAD)
        need = mq.workspace_bytes(w, None, 2, mq.ERR_TENSOR, cfg)
        if ws is None or ws.numel() < need:
            ws = torch.empty(need, dtype=torch.uint8, device=dev)
        out = mq.alloc_qbuffers(o, n, 4, cfg, dev)
        for k, cands in sets.items():
            mq.select_layer(w, None, cands, mq.ERR_TENSOR, cfg, out, None, results[k][i], ws, stream)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    res = {k: mq.read_results(v) for k, v in results.items()}
    e_int = sum(r.err[0] for r in res["redesigned"])
    e_new = sum(r.err[1] for r in res["redesigned"])
    e_ieee = sum(r.err[1] for r in res["ieee"])
    per_layer = [r1.err[1] / r2.err[1] for r1, r2 in zip(res["redesigned"], res["ieee"])]
    return {
        "metric": "tensor error of the redesigned FP4 relative to the IEEE-aligned FP4 (synthetic 7B-shaped weights)",
        "value": e_new / e_ieee, "unit": "ratio", "n_gpus": 1, "steps": 1, "warmup": 0,
        "ms_per_step": elapsed * 1e3, "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 decisions, f64 errors", "data": "synthetic",
        "config": {"workload": f"{len(shapes)} linears of the LLaMA-7B shape, fp16, per-channel absmax scales (one candidate)",
                   "error_reduction_percent": 100.0 * (1.0 - e_new / e_ieee),
                   "per_layer_ratio_min_max": [min(per_layer), max(per_layer)],
                   "int4_error_relative_to_redesigned_fp4": e_int / e_new,
                   "layers_preferring_fp4_over_int4_percent": {
                       k: 100.0 * sum(1 for r in v if r.best == 1) / len(v) for k, v in res.items()}},
    }


def run_w4_units(args, shapes, dev):
    """Per-unit format select (finer than the layer) on the 7B-shaped set, group 128 with
    fp16 scales and 50 clip ratios: time, and the tensor error of the mixed assignment
    against the layer-wise choice."""
    import torch

    import mofq_inputs as mi
    from paper_2305_12356_amd import binding as mq

    clip = mi.clip_ratios(N_CLIP_GROUP)
    cfg = mq.Cfg(mq.PER_GROUP, clip, GROUP, True)
    cands = [mq.INT4, mq.FP4_E2M1]
    weights, outs, tags = [], [], []
    results = mq.alloc_result(dev, len(shapes))
    mixed = torch.zeros(len(shapes), dtype=torch.float64, device=dev)
    ws_bytes = 0
    for b, name, o, n in shapes:
        w = mi.model_weight(1, b, mi.LINEAR_NAMES.index(name), o, n, device=dev, tail_spread=TAIL_SPREAD)
        weights.append(w)
        outs.append(mq.alloc_qbuffers(o, n, 4, cfg, dev))
        tags.append(torch.empty(o * (n // GROUP), dtype=torch.uint8, device=dev))
        ws_bytes = max(ws_bytes, mq.select_units_workspace_bytes(w, 2, cfg))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream()

    def step():
        for i, w in enumerate(weights):
            mq.select_units(w, cands, cfg, outs[i], tags[i], results[i], mixed[i:i + 1], ws, stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    res = mq.read_results(results)
    layer = sum(min(r.err[0], r.err[1]) for r in res)
    mix = float(mixed.sum().item())
    fp_units = sum(int(t.sum().item()) for t in tags)
    n_units = sum(t.numel() for t in tags)
    n_elems = sum(o * n for _, _, o, n in shapes)
    return {
        "metric": "weight-elems x candidates scored/sec, per-unit format select (group 128)",
        "value": n_elems * N_CLIP_GROUP * N_FMT / (elapsed / args.steps), "unit": "elem*cand/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": elapsed / args.steps * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 decisions, f64 errors", "data": "synthetic",
        "config": {"workload": f"{len(shapes)} linears of the LLaMA-7B shape, fp16, group 128, fp16 scales, 50 clip "
                               "ratios, INT4 vs FP4-E2M1 chosen per group",
                   "mixed_error_relative_to_layer_wise": mix / layer,
                   "fp4_units_percent": 100.0 * fp_units / n_units},
    }


# ---- the oracle over whole tensors (not a benchmark) -------------------------------------

def parse_blocks(text, n_blocks):
    out = []
    for part in text.split(","):
        if ":" in part:
            a, b = part.split(":")
            out.extend(range(int(a), int(b)))
        else:
            out.append(int(part))
    assert all(0 <= b < n_blocks for b in out), "block out of range"
    return out


def full_parity(args, dev):
    """Every linear of the listed blocks of the 7B- or 65B-shaped set through
    mofq_select_layers (the launch configuration the benchmark times) and, whole, through
    the oracle: per tensor the format choice, both candidates' error sums, and on ALL rows the
    winner's codes, scales and clip indices (near-tie rule of tests/gpu_util.py)."""
    import numpy as np
    import torch

    import mofq_inputs as mi
    from oracle import mofq_oracle as orc
    from paper_2305_12356_amd import binding as mq
    from tests.gpu_util import compare_quantized, scales_to_f32, unpack_codes

    group = args.workload == "w4_group128"
    n_clip = N_CLIP_GROUP if group else N_CLIP
    clip = mi.clip_ratios(n_clip)
    cands = [mq.INT4, mq.FP4_E2M1]
    cfg = mq.Cfg(mq.PER_GROUP, clip, GROUP, True) if group else mq.Cfg(mq.PER_CHANNEL, clip)
    gran, grp, f16 = (orc.PER_GROUP, GROUP, True) if group else (orc.PER_CHANNEL, 0, False)
    blocks = parse_blocks(args.block_list, mi.LLAMA_SHAPES[args.model]["blocks"])
    all_shapes = mi.model_linear_shapes(args.model)
    # the 7B-shaped set runs whole, as bench.py times it; of the 65B-shaped set only the listed blocks
    shapes = all_shapes if args.model == "7b" else [s for s in all_shapes if s[0] in blocks]
    weights = make_weights(shapes, dev)
    qouts = [mq.alloc_qbuffers(o, n, 4, cfg, dev) for _, _, o, n in shapes]
    results = mq.alloc_result(dev, len(shapes))
    batch = mq.LayerBatch(weights, qouts)
    ws = torch.empty(batch.workspace_bytes(2, cfg), dtype=torch.uint8, device=dev)
    mq.select_layers(batch, cands, cfg, results, ws, torch.cuda.current_stream(), side_stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    res = mq.read_results(results)
    threads = orc.max_threads()
    summary = {"mode": "full-parity", "model": args.model, "tail_spread": TAIL_SPREAD,
               "workload": "w4_group128" if group else "w4_channel",
               "blocks": blocks, "n_clip": n_clip, "tensors_in_the_select_layers_call": len(shapes),
               "tensors_checked": 0, "rows_checked": 0, "elements_checked": 0,
               "choice_mismatches": 0, "error_sum_mismatches_rtol_1e-9": 0, "max_error_sum_rel_diff": 0.0,
               "tensors_with_code_scale_or_index_mismatch": 0, "near_tie_units": 0, "fp_chosen": 0,
               "oracle_seconds": 0.0, "oracle_threads": threads, "head": git_head(), "failures": []}
    for i, (b, name, o, n) in enumerate(shapes):
        if b not in blocks:
            continue
        w32 = mi.to_f32_numpy(weights[i])
        t0 = time.perf_counter()
        ref = orc.select_layer_w_only(w32, cands, gran, clip, grp, f16, want_table=True, threads=threads)
        summary["oracle_seconds"] += time.perf_counter() - t0
        r = res[i]
        summary["tensors_checked"] += 1
        summary["rows_checked"] += o
        summary["elements_checked"] += o * n
        summary["fp_chosen"] += int(ref.best == 1)
        if r.best != ref.best:
            summary["choice_mismatches"] += 1
            summary["failures"].append(f"block {b} {name}: choice {r.best} vs oracle {ref.best}")
        rel = max(abs(r.err[c] - ref.errs[c]) / ref.errs[c] for c in range(2))
        summary["max_error_sum_rel_diff"] = max(summary["max_error_sum_rel_diff"], rel)
        if rel > 1e-9 or abs(r.ref_energy - ref.ref_energy) > 1e-9 * ref.ref_energy:
            summary["error_sum_mismatches_rtol_1e-9"] += 1
            summary["failures"].append(f"block {b} {name}: error sums {list(r.err)[:2]} vs {ref.errs}")
        try:
            win = ref.per_candidate[r.best] if r.best != ref.best else ref.w
            summary["near_tie_units"] += compare_quantized(
                w32, cands[r.best], gran, grp, f16, np.asarray(clip, dtype=np.float32), win,
                unpack_codes(qouts[i].codes, o, n, 4), scales_to_f32(qouts[i].scales),
                qouts[i].clip_idx.cpu().numpy(), qouts[i].unit_err.cpu().numpy())
        except AssertionError as e:
            summary["tensors_with_code_scale_or_index_mismatch"] += 1
            summary["failures"].append(f"block {b} {name}: {e}")
        print(f"[full-parity] block {b} {name} {o}x{n}: best={r.best} oracle={ref.best} "
              f"rel={rel:.2e} oracle_s={summary['oracle_seconds']:.1f}", file=sys.stderr, flush=True)
    summary["oracle_elem_cand_per_s"] = summary["elements_checked"] * n_clip * N_FMT / max(summary["oracle_seconds"], 1e-9)
    summary["ok"] = not summary["failures"]
    print(json.dumps(summary))
    return 0 if summary["ok"] else 1


def full_parity_wa(args, dev):
    """Every linear of the listed blocks of the W8A8 workload, block by block through
    mofq_select_layers_wa as bench.py times it (one call per block here, one activation per role
    of the block: q/k/v, o, gate/up, down) with both forms of the layer-output
    metric and, whole, through the oracle (fp64 matrix products): both candidates' error sums and
    the reference energy to 1e-5, the choice, and the winner's codes and scales of W and X bit for
    bit."""
    import numpy as np
    import torch

    import mofq_inputs as mi
    from oracle import mofq_oracle as orc
    from paper_2305_12356_amd import binding as mq
    from tests.gpu_util import scales_to_f32, unpack_codes

    blocks = parse_blocks(args.block_list, mi.LLAMA_SHAPES["7b"]["blocks"])
    cands = [mq.INT8, mq.FP8_E4M3]
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    xcfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    role = {"q": 0, "k": 0, "v": 0, "o": 1, "gate": 2, "up": 2, "down": 3}
    summary = {"mode": "full-parity", "workload": "w8a8", "tail_spread": TAIL_SPREAD, "blocks": blocks,
               "tokens": TOKENS, "linears_checked": 0,
               "choice_mismatches": 0, "error_sum_mismatches_rtol_1e-5": 0, "max_error_sum_rel_diff_exact": 0.0,
               "max_error_sum_rel_diff_fp8_unit": 0.0, "fp8_unit_layers_beyond_1e-5": 0,
               "code_or_scale_mismatches": 0, "fp_chosen": 0,
               "oracle_seconds": 0.0, "head": git_head(), "failures": []}
    for b in blocks:
        shapes = [s_ for s_ in mi.model_linear_shapes("7b") if s_[0] == b]
        acts, xs, ws_ = {}, [], []
        for _, name, o, n in shapes:
            lin = mi.LINEAR_NAMES.index(name)
            if role[name] not in acts:
                acts[role[name]] = mi.activations(TOKENS, n, seed=mi.tensor_seed(3, b, role[name], 1), device=dev)
            xs.append(acts[role[name]])
            ws_.append(mi.model_weight(3, b, lin, o, n, dtype=torch.bfloat16, device=dev, tail_spread=TAIL_SPREAD))
        got = {}
        for metric, key in ((mq.ERR_LAYER_OUTPUT, "exact"), (mq.ERR_LAYER_OUTPUT_FP8_UNIT, "fp8_unit")):
            w_outs = [mq.alloc_qbuffers(o, n, 8, cfg, dev) for _, _, o, n in shapes]
            x_outs = [mq.alloc_qbuffers(TOKENS, n, 8, xcfg, dev) for _, _, o, n in shapes]
            batch = mq.WaLayerBatch(ws_, xs, w_outs, x_outs)
            res = mq.alloc_result(dev, len(shapes))
            wsp = torch.empty(batch.workspace_bytes(2, metric, cfg), dtype=torch.uint8, device=dev)
            mq.select_layers_wa(batch, cands, metric, cfg, res, wsp)
            torch.cuda.synchronize()
            got[key] = (mq.read_results(res), w_outs, x_outs)
        for i, (_, name, o, n) in enumerate(shapes):
            t0 = time.perf_counter()
            ref = orc.select_layer_wa(mi.to_f32_numpy(xs[i]), mi.to_f32_numpy(ws_[i]), cands, orc.PER_TENSOR)
            summary["oracle_seconds"] += time.perf_counter() - t0
            summary["linears_checked"] += 1
            summary["fp_chosen"] += int(ref.best == 1)
            for key, (rs, w_outs, x_outs) in got.items():
                r = rs[i]
                rel = max(abs(r.err[c] - ref.errs[c]) / ref.errs[c] for c in range(2))
                rel = max(rel, abs(r.ref_energy - ref.ref_energy) / ref.ref_energy)
                summary["max_error_sum_rel_diff_" + key] = max(summary["max_error_sum_rel_diff_" + key], rel)
                if key == "exact" and rel > 1e-5:
                    summary["error_sum_mismatches_rtol_1e-5"] += 1
                    summary["failures"].append(f"block {b} {name} {key}: {list(r.err)[:2]} vs {ref.errs}")
                if key == "fp8_unit":
                    # with the activation's outlier columns split off into an exact K step the fp8 unit's
                    # in-instruction alignment stays far inside the same tolerance
                    summary["fp8_unit_layers_beyond_1e-5"] += int(rel > 1e-5)
                    if rel > 1e-5:
                        summary["error_sum_mismatches_rtol_1e-5"] += 1
                        summary["failures"].append(f"block {b} {name} {key}: {list(r.err)[:2]} vs {ref.errs}")
                if r.best != ref.best:
                    summary["choice_mismatches"] += 1
                    summary["failures"].append(f"block {b} {name} {key}: choice {r.best} vs {ref.best}")
                same = (np.array_equal(unpack_codes(w_outs[i].codes, o, n, 8), ref.w.codes) and
                        np.array_equal(unpack_codes(x_outs[i].codes, TOKENS, n, 8), ref.x.codes) and
                        np.array_equal(scales_to_f32(w_outs[i].scales), ref.w.scale) and
                        np.array_equal(scales_to_f32(x_outs[i].scales), ref.x.scale))
                if not same:
                    summary["code_or_scale_mismatches"] += 1
                    summary["failures"].append(f"block {b} {name} {key}: codes or scales differ")
            print(f"[full-parity] w8a8 block {b} {name} {o}x{n}: oracle best={ref.best} "
                  f"oracle_s={summary['oracle_seconds']:.1f}", file=sys.stderr, flush=True)
        del got
    summary["ok"] = not summary["failures"]
    print(json.dumps(summary))
    return 0 if summary["ok"] else 1


def brief(d):
    """A secondary workload inside the headline line: the figures, not the boilerplate."""
    keep = ("metric", "value", "unit", "ms_per_step", "steps", "warmup",
            "higher_is_better", "dtype", "config", "roofline")
    return {k: d[k] for k in keep if k in d}


def main():
    global HEAD_OVERRIDE, TAIL_SPREAD
    args = parse()
    HEAD_OVERRIDE = args.head
    TAIL_SPREAD = args.tail_spread
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no collectives, no second device); "
              "use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch

    import mofq_inputs as mi

    if not torch.cuda.is_available():
        print("bench.py needs an MI355X (cuda:0)", file=sys.stderr)
        sys.exit(2)
    dev = "cuda:0"
    torch.cuda.set_device(0)

    if args.full_parity:
        sys.exit(full_parity_wa(args, dev) if args.workload == "w8a8" else full_parity(args, dev))

    def note(msg):
        print(f"[bench] {msg}", file=sys.stderr, flush=True)

    shapes = mi.model_linear_shapes(args.model)
    if args.blocks:
        shapes = [s for s in shapes if s[0] < args.blocks]
    wl = args.workload
    if wl == "ceilings":
        print(json.dumps(measure_ceilings(dev)))
        return
    if wl in ("w8a8", "w4a16_output"):
        weights = make_weights(shapes, dev, torch.bfloat16)
        print(json.dumps(run_w8a8(args, shapes, dev, weights, wl == "w4a16_output",
                                  wl == "w8a8" and not args.exact_e4m3, args.steps, args.warmup)))
        return
    if wl == "k1_hbm":
        print(json.dumps(run_k1_hbm(args, dev, args.steps, args.warmup)))
        return
    if wl == "fp4_variants":
        print(json.dumps(run_fp4_variants(args, shapes, dev)))
        return
    if wl == "w4_units":
        print(json.dumps(run_w4_units(args, shapes, dev)))
        return
    if wl in ("w4_channel", "w4_group128"):
        weights = make_weights(shapes, dev)
        out = run_w4(args, shapes, dev, weights, wl == "w4_group128", args.model, args.steps, args.warmup,
                     want_cpu=(wl == "w4_channel" and args.model == "7b" and not args.no_cpu_baseline and not args.blocks))
        if args.copy_calibration:
            src = torch.empty(1 << 30, dtype=torch.uint8, device=dev).fill_(1)
            dst = torch.empty_like(src)
            dst.copy_(src)          # reads 1 GiB, writes 1 GiB
            torch.cuda.synchronize()
        print(json.dumps(out))
        return

    # ---- all: the headline workload, then the others under `secondary` ------------------
    t_start = time.perf_counter()
    note("device ceilings")
    ceilings = measure_ceilings(dev)
    shapes7 = mi.model_linear_shapes("7b")
    if args.blocks:
        shapes7 = [s for s in shapes7 if s[0] < args.blocks]
    note("7B-shaped fp16 weights")
    weights = make_weights(shapes7, dev)
    note("7B-shaped set: per-channel, 100 clip ratios")
    out = run_w4(args, shapes7, dev, weights, False, "7b", args.steps, args.warmup, ceilings,
                 want_cpu=not args.no_cpu_baseline and not args.blocks)
    out["ceilings"] = ceilings
    sec = {}
    few, few_w = max(1, min(args.steps, 3)), max(1, min(args.warmup, 1))
    note("7B-shaped set: group 128, 50 clip ratios")
    sec["w4_group128"] = brief(run_w4(args, shapes7, dev, weights, True, "7b", few, few_w, ceilings))
    del weights
    torch.cuda.empty_cache()
    note("single candidate, fp32, 1 GiB")
    sec["k1_hbm"] = brief(run_k1_hbm(args, dev, few, few_w, ceilings))
    torch.cuda.empty_cache()
    note("bf16 weights for the layer-output workloads")
    weights = make_weights(shapes7, dev, torch.bfloat16)
    note("W8A8, int8 and fp8 matrix cores for the quantized products")
    sec["w8a8"] = brief(run_w8a8(args, shapes7, dev, weights, False, True, few, few_w, ceilings))
    note("W8A8, E4M3 product from grid values on the bf16 matrix cores")
    sec["w8a8_exact_e4m3"] = brief(run_w8a8(args, shapes7, dev, weights, False, False, few, few_w, ceilings))
    note("weight-only select by layer-output error")
    sec["w4a16_output"] = brief(run_w8a8(args, shapes7, dev, weights, True, False, few, few_w, ceilings))
    del weights
    torch.cuda.empty_cache()
    if not args.no_65b and not args.blocks:
        note("65B-shaped set, 129.5 GB resident")
        shapes65 = mi.model_linear_shapes("65b")
        weights = make_weights(shapes65, dev)
        sec["w4_channel_65b"] = brief(run_w4(args, shapes65, dev, weights, False, "65b", 2, 1, ceilings))
        del weights
        torch.cuda.empty_cache()
    out["secondary"] = sec
    out["bench_wall_s"] = round(time.perf_counter() - t_start, 1)
    out["head"] = git_head()
    print(json.dumps(out))


if __name__ == "__main__":
    main()
