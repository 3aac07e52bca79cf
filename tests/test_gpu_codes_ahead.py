"""Codes that the search writes row by row in the row's own better format, and the rows that are done again once the
tensor's choice is known: tensors whose rows disagree, against the CPU oracle (tolerances as in test_gpu_w_only)."""
import numpy as np
import pytest
import torch

import mofq_inputs as mi
from oracle import mofq_oracle as orc
from tests.test_gpu_w_only import check_tensor, mq  # noqa: F401

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
PAIRS = {4: [orc.INT4, orc.FP4_E2M1], 8: [orc.FP8_E4M3, orc.INT8]}


def rows_that_disagree(rows, cols, every, dtype, factor=1.0, heavy=1.0):
    """LLaMA-like rows (floating point wins), every so many of them uniform (integers win), `heavy` times as large."""
    w = mi.llama_like_weight(rows, cols, seed=rows + cols, dtype=torch.float32, device=DEV)
    g = torch.Generator().manual_seed(cols)
    w[::every] = ((torch.rand(w[::every].shape, generator=g) - 0.5) * 0.1 * heavy).to(DEV)
    return (w * factor).to(dtype)


# From 1024 rows a launch on (8-bit formats with one ratio: 2048; with more: 8192) the search writes codes ahead.  The smallest such
# tensors and rows that leave the last workgroup less than it takes at a time (rows / 512, 2 to 16); rows of one chunk, rows that
# end inside a step of the redo loop; with a tally of the finished rows (8192 rows; one ratio: 128 MB).  One or the other
# format mostly, both alike, and a few heavy rows that decide against all others; one ratio (any type) and the
# histogram searches.
@pytest.mark.parametrize("every,heavy", [(1, 1.0), (2, 1.0), (5, 1.0), (32, 100.0)])
@pytest.mark.parametrize("dtype,bits,clips,shapes", [
    ("f32", 4, 1, [(1024, 8), (1025, 264), (1537, 16384)]),
    ("f16", 4, 1, [(1024, 8), (1055, 4104)]),
    ("bf16", 8, 1, [(2048, 1032), (2049, 2056)]),
    ("f16", 4, 20, [(1024, 1024), (1041, 4104), (1027, 11008)]),
    ("bf16", 4, 20, [(1025, 2056), (1033, 5000), (1027, 8200)]),
    ("f32", 4, 1, [(8209, 4104)]),
    ("f16", 4, 20, [(8193, 1024)]),
    ("bf16", 8, 50, [(8193, 1024)]),
])
def test_rows_done_again(mq, dtype, bits, clips, shapes, every, heavy):  # noqa: F811
    for rows, cols in shapes:
        w = rows_that_disagree(rows, cols, every, DTYPES[dtype], heavy=heavy)
        check_tensor(mq, w, PAIRS[bits], orc.PER_CHANNEL, mi.clip_ratios(clips), label=f"every {every}, {heavy} times as large")


# Tensors of a few rows, down to one, in a launch of more than 1024: against the calls by themselves, whose codes the
# emission writes.
@pytest.mark.parametrize("dtype,cols,clips", [("f16", 1024, 20), ("f16", 4104, 20), ("bf16", 5000, 20), ("f32", 264, 1)])
def test_small_tensors_in_a_large_launch(mq, dtype, cols, clips):  # noqa: F811
    from tests.test_gpu_select_layers import _single
    ws_ = [rows_that_disagree(rows, cols, every, DTYPES[dtype], heavy=heavy)
           for rows, every, heavy in ((1024, 2, 1.0), (1, 1, 1.0), (1, 2, 1.0), (17, 5, 1.0), (33, 16, 100.0), (2, 2, 1.0))]
    cands, cfg = PAIRS[4], mq.Cfg(orc.PER_CHANNEL, mi.clip_ratios(clips))
    outs = [mq.alloc_qbuffers(*w.shape, 4, cfg, DEV) for w in ws_]
    batch = mq.LayerBatch(ws_, outs)
    results = mq.alloc_result(DEV, len(ws_))
    ws = torch.empty(batch.workspace_bytes(2, cfg), dtype=torch.uint8, device=DEV)
    print(f"[case] small tensors in a large launch, {dtype} {cols}", flush=True)
    mq.select_layers(batch, cands, cfg, results, ws)
    torch.cuda.synchronize()
    for w, o, r in zip(ws_, outs, mq.read_results(results)):
        q, ref = _single(mq, w, cands, cfg, 4)
        assert r.best == ref.best and list(r.err) == list(ref.err)
        assert torch.equal(o.codes, q.codes) and torch.equal(o.scales, q.scales)
        assert torch.equal(o.clip_idx, q.clip_idx) and torch.equal(o.unit_err, q.unit_err)


# Below those lines the codes come from the emission.  One row, rows of one chunk; one or the other format mostly, or both
# alike; one ratio (any type) and the histogram searches (16 bits, 4-bit formats).
@pytest.mark.parametrize("every", [1, 2, 5])
@pytest.mark.parametrize("dtype,bits,clips,shapes", [
    ("f32", 4, 1, [(1, 8), (3, 1024), (33, 8), (1025, 264), (17, 16384)]),
    ("f16", 4, 1, [(2, 8), (31, 4104)]),
    ("bf16", 8, 1, [(3, 1032), (65, 2056)]),
    ("f16", 4, 20, [(1, 1024), (17, 4096), (33, 4104), (5, 11008)]),
    ("bf16", 4, 20, [(1, 1024), (17, 2056), (33, 5000), (3, 22016)]),
])
def test_rows_that_disagree(mq, dtype, bits, clips, shapes, every):  # noqa: F811
    for rows, cols in shapes:
        w = rows_that_disagree(rows, cols, every, DTYPES[dtype])
        check_tensor(mq, w, PAIRS[bits], orc.PER_CHANNEL, mi.clip_ratios(clips), label=f"every {every}")


# Rows whose counted patterns reach down to subnormals beside rows whose patterns do not (fp16: below 2^-14).
@pytest.mark.parametrize("dtype,bits,cols,clips", [("f16", 4, 4096, 50), ("f16", 4, 8192, 20), ("f16", 8, 4096, 50), ("bf16", 4, 2048, 50),
                                                   ("bf16", 8, 2048, 50)])
def test_rows_with_counted_subnormals(mq, dtype, bits, cols, clips):  # noqa: F811
    w = rows_that_disagree(12, cols, 3, torch.float32)
    tiny = 2.0 ** -12 if dtype == "f16" else 2.0 ** -120
    w *= torch.tensor([1.0, tiny, tiny * 0.125] * 4, device=DEV)[:, None]
    check_tensor(mq, w.to(DTYPES[dtype]), PAIRS[bits][::1 if bits == 4 else -1], orc.PER_CHANNEL, mi.clip_ratios(clips), label="tiny rows")


def test_layer_output_chooses_against_the_rows(mq):  # noqa: F811
    """Weight-only layer output: the codes are those of the choice, whichever format a row preferred."""
    from tests import test_gpu_w_only_output as wo
    x = mi.activations(70, 256, seed=3, device=DEV)
    for every in (1, 2, 5):
        wo.check_layer(mq, x, rows_that_disagree(131, 256, every, torch.bfloat16), PAIRS[4], orc.PER_CHANNEL, mi.clip_ratios(1), f"every {every}")


@pytest.mark.parametrize("rows", [131, 1024, 1041])
def test_layer_output_against_the_tensor_error(mq, rows):  # noqa: F811
    """An input that meets the largest weights alone, where the integer grid is finer: the layer output chooses against the
    tensor error of nearly every row, so the codes written ahead (from 1024 rows on) are all done again."""
    from tests import test_gpu_w_only_output as wo
    g = torch.Generator().manual_seed(rows)
    w = torch.randn(rows, 512, generator=g)
    w[:, ::61] *= 4.0
    x = torch.randn(70, 512, generator=g) * 0.02
    x[:, ::61] *= 1500.0
    w, x = (t.to(torch.bfloat16).to(DEV) for t in (w, x))
    cands, clip = PAIRS[4], mi.clip_ratios(1)
    r = wo.check_layer(mq, x, w, cands, orc.PER_CHANNEL, clip, "against the rows")
    errs = [orc.quantize(mi.to_f32_numpy(w), f, orc.PER_CHANNEL, np.asarray(clip, dtype=np.float32)).err for f in cands]
    assert r.best != orc.select(errs)
