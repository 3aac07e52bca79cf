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


def rows_that_disagree(rows, cols, every, dtype, factor=1.0):
    """LLaMA-like rows (floating point wins), every so many of them uniform (integers win)."""
    w = mi.llama_like_weight(rows, cols, seed=rows + cols, dtype=torch.float32, device=DEV)
    g = torch.Generator().manual_seed(cols)
    w[::every] = ((torch.rand(w[::every].shape, generator=g) - 0.5) * 0.1).to(DEV)
    return (w * factor).to(dtype)


# One row, rows of one chunk, fewer rows than a workgroup redoes at a time, one more, rows that end inside a step of the redo
# loop; one or the other format mostly, or both alike; one ratio (any type) and the histogram searches (16 bits, 4-bit formats).
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
