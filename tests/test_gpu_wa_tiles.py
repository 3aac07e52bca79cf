"""GPU parity of the layer-output products of tensors whose rows lie far apart."""
import numpy as np
import pytest
import torch

import mofq_inputs as mi
from oracle import mofq_oracle as orc

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
I8, FP8 = orc.INT8, orc.FP8_E4M3


@pytest.fixture(scope="module")
def mq():
    from paper_2305_12356_amd import binding
    assert torch.cuda.is_available()
    return binding


@pytest.mark.parametrize("rows,ld", [(130, 36 << 20), (300, 9 << 20), (300, 18 << 20)])
def test_rows_far_apart(mq, rows, ld):
    """Row strides at which a tile's rows reach beyond 2^32 bytes: of 64 rows
    and of 256 (64-bit offsets)."""
    K = 128
    if torch.cuda.mem_get_info()[0] < rows * ld * 2 + (1 << 30):
        pytest.skip("needs the memory of the gaps between the rows")
    w = mi.llama_like_weight(rows, K, seed=8501, dtype=torch.bfloat16, device=DEV)
    apart = torch.empty(rows * ld, dtype=torch.bfloat16, device=DEV).view(rows, ld)[:, :K]
    apart.copy_(w)
    x = mi.activations(2100, K, seed=8500, device=DEV)
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    out, res = mq.alloc_qbuffers(rows, K, 8, cfg, DEV), mq.alloc_result(DEV, 2)
    for i, t in enumerate((w, apart)):
        ws = torch.empty(mq.workspace_bytes(t, x, 2, mq.ERR_LAYER_OUTPUT, cfg), dtype=torch.uint8, device=DEV)
        mq.select_layer(t, x, [I8, FP8], mq.ERR_LAYER_OUTPUT, cfg, out, None, res[i], ws)
    torch.cuda.synchronize()
    a, b = mq.read_results(res)
    # the same accumulators; the error sums are added per tile
    assert a.best == b.best and np.allclose(list(a.err)[:2] + [a.ref_energy], list(b.err)[:2] + [b.ref_energy], rtol=1e-13)
