"""GPU parity of the layer-output products in every tiling: which one a layer takes depends on its
sizes alone, and each is compared with the oracle at its ragged edges and K remainders."""
import numpy as np
import pytest
import torch

import mofq_inputs as mi
from oracle import mofq_oracle as orc
from tests import test_gpu_w_only_output as wo
from tests import test_gpu_wa as wa
from tests import test_gpu_wa_layers as layers

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
I4, FP4, I8, FP8 = orc.INT4, orc.FP4_E2M1, orc.INT8, orc.FP8_E4M3

# tokens, rows, columns: by the number of tiles and the stages of 64 columns (an odd number leaves the last stage of an
# 8-bit product half full)
SHAPES = {
    "small tiles": (65, 63, 192),
    "small tiles, the last number of stages that is not cut": (130, 190, 64 * 19),
    "cut to 11 stages": (70, 90, 64 * 21),
    "cut to 20 stages, one more than divides": (64, 65, 64 * 41),
    "most pieces of a few tiles": (63, 64, 64 * 331),
    "more than 48 tiles, cut to 40 stages": (449, 448, 64 * 41),
    "more than 160 tiles, cut into the products": (833, 832, 64 * 21),
    "medium tiles": (1601, 1345, 192),
    "large tiles": (2049, 2049, 128),
}


@pytest.fixture(scope="module")
def mq():
    from paper_2305_12356_amd import binding
    assert torch.cuda.is_available()
    return binding


def tensors(shape, seed):
    M, N, K = shape
    return mi.activations(M, K, seed=seed, device=DEV), mi.llama_like_weight(N, K, seed=seed + 1, dtype=torch.bfloat16, device=DEV)


@pytest.mark.parametrize("name", list(SHAPES))
def test_exact_products(mq, name):
    x, w = tensors(SHAPES[name], 8100)
    wa.check_layer(mq, x, w, [I8, FP8], orc.PER_TENSOR, name)          # the fused path
    wa.check_layer(mq, x, w, [FP8, I8], orc.PER_CHANNEL, name)         # the general one; a product alone


@pytest.mark.parametrize("shape", [(70, 300, 320), (64, 256, 64 * 41), (1601, 1345, 320), (2049, 2049, 256)])
def test_exact_products_widen_every_code(mq, shape):
    """Operands on E4M3's grid (scale 1), every finite code of it, one weight to a row: each output is a single product of
    two grid values, exact in fp32, so the E4M3 error is 0 in every tiling."""
    M, N, K = shape
    g = torch.Generator().manual_seed(K)
    grid = torch.arange(256, dtype=torch.uint8).view(torch.float8_e4m3fn).float()
    grid = grid[grid.isfinite()]
    x = grid[torch.randint(len(grid), (M, K), generator=g)]
    w = torch.zeros(N, K)
    w[torch.arange(N), torch.arange(N) % K] = grid[torch.arange(N) % len(grid)]
    x[0, 0] = w[0, 0] = 448.0
    x, w = x.to(torch.bfloat16).to(DEV), w.to(torch.bfloat16).to(DEV)
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    r, w_out, _ = layers.run_single(mq, [w], [x], [I8, FP8], mq.ERR_LAYER_OUTPUT, cfg)
    assert r[0].err[1] == 0.0 and r[0].err[0] > 0.0 and r[0].best == 1
    assert torch.equal(w_out[0].codes.view(-1), w.cpu().float().to(torch.float8_e4m3fn).view(torch.uint8).view(-1).to(DEV))


@pytest.mark.parametrize("name", list(SHAPES))
def test_exact_products_of_grid_values_have_no_error(mq, name):
    """Dense operands on E4M3's grid: the reference and the E4M3 product add up the same numbers in the same order in every
    tiling and piece, so the error is exactly 0 and an earlier candidate without error stays the choice."""
    M, N, K = SHAPES[name]
    g = torch.Generator().manual_seed(K + 1)
    grid = torch.arange(256, dtype=torch.uint8).view(torch.float8_e4m3fn).float()
    grid = grid[grid.isfinite()]
    x, w = grid[torch.randint(len(grid), (M, K), generator=g)], grid[torch.randint(len(grid), (N, K), generator=g)]
    x[0, 0] = w[0, 0] = 448.0
    x, w = x.to(torch.bfloat16).to(DEV), w.to(torch.bfloat16).to(DEV)
    r, _, _ = layers.run_single(mq, [w], [x], [I8, FP8], mq.ERR_LAYER_OUTPUT, mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1)))
    assert r[0].err[1] == 0.0 and r[0].err[0] > 0.0 and r[0].best == 1


@pytest.mark.parametrize("apart", [0, 64])
def test_layers_with_one_code_buffer(mq, apart):
    """Layers whose weights' codes go to the same memory, or to memory that overlaps: what is written there is not
    defined, the errors and choices are those of separate buffers."""
    ws = [mi.llama_like_weight(n, 320, seed=n, dtype=torch.bfloat16, device=DEV) for n in (200, 260, 130)]
    xs = [mi.activations(150, 320, seed=7, device=DEV)] * 3
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    want, _, _ = layers.run_batched(mq, ws, xs, [I8, FP8], mq.ERR_LAYER_OUTPUT, cfg)
    w_out, x_out = layers.alloc_outs(mq, ws, xs, cfg)
    memory = torch.empty(260 * 320 + 128, dtype=torch.uint8, device=DEV)
    for i, o in enumerate(w_out):
        o.codes = memory[i * apart:i * apart + ws[i].numel()]
    batch = mq.WaLayerBatch(ws, xs, w_out, x_out)
    wsp = torch.empty(batch.workspace_bytes(2, mq.ERR_LAYER_OUTPUT, cfg), dtype=torch.uint8, device=DEV)
    res = mq.alloc_result(DEV, 3)
    mq.select_layers_wa(batch, [I8, FP8], mq.ERR_LAYER_OUTPUT, cfg, res, wsp)
    torch.cuda.synchronize()
    for a, b in zip(mq.read_results(res), want):
        assert a.best == b.best and list(a.err)[:2] == list(b.err)[:2] and a.ref_energy == b.ref_energy


@pytest.mark.parametrize("name", list(SHAPES))
def test_weight_only_products(mq, name):
    x, w = tensors(SHAPES[name], 8200)
    wo.check_layer(mq, x, w, [I4, FP4], orc.PER_CHANNEL, mi.clip_ratios(1), name)


@pytest.mark.parametrize("cands,gran,ratios", [([I4, FP4], orc.PER_CHANNEL, 1), ([FP4, I4], orc.PER_TENSOR, 1), ([I8, FP8], orc.PER_CHANNEL, 1),
                                               ([I4, FP4], orc.PER_CHANNEL, 3)])
@pytest.mark.parametrize("name", list(SHAPES))
def test_weight_only_error_of_a_format_alone(mq, name, cands, gran, ratios):
    """mofq_score's error and energy are the select's, bit for bit: Algorithm 1 put together from scores chooses alike."""
    x, w = tensors(SHAPES[name], 8600)
    r, _ = wo.run_select(mq, x, w, cands, gran, mi.clip_ratios(ratios))
    for c, fmt in enumerate(cands):
        assert wo.run_score(mq, x, w, fmt, gran, mi.clip_ratios(ratios)) == (r.err[c], r.ref_energy)


@pytest.mark.parametrize("cands,gran", [([I8, FP8], orc.PER_CHANNEL), ([FP8, I8], orc.PER_TENSOR)])
@pytest.mark.parametrize("name", list(SHAPES))
def test_exact_error_of_a_format_alone(mq, name, cands, gran):
    """The same with the activation quantized too, in the general path and the fused one."""
    x, w = tensors(SHAPES[name], 8650)
    cfg = mq.Cfg(gran, mi.clip_ratios(1))
    r, _, _ = layers.run_single(mq, [w], [x], cands, mq.ERR_LAYER_OUTPUT, cfg)
    for c, fmt in enumerate(cands):
        err, en = (torch.zeros(1, dtype=torch.float64, device=DEV) for _ in range(2))
        ws = torch.empty(mq.workspace_bytes(w, x, 1, mq.ERR_LAYER_OUTPUT, cfg), dtype=torch.uint8, device=DEV)
        mq.score(w, x, fmt, mq.ERR_LAYER_OUTPUT, cfg, err, en, ws)
        assert (err.item(), en.item()) == (r[0].err[c], r[0].ref_energy)


@pytest.mark.parametrize("cands", [[I4, FP4], [FP4, I4], [I8, FP8]])
@pytest.mark.parametrize("name", list(SHAPES))
def test_weight_only_products_of_grid_values_have_no_error(mq, name, cands):
    """Weights on a format's grid (scale 1): the reference and that format's product add up the same numbers in the same
    order in every tiling and piece and from either kind of operand, so its error is exactly 0."""
    M, N, K = SHAPES[name]
    g = torch.Generator().manual_seed(K + 2)
    x = mi.activations(M, K, seed=8700, device=DEV)
    for fmt, levels in ((I4, torch.arange(-7.0, 8)), (FP4, torch.tensor([0.0, 0.5, 1, 1.5, 2, 3, 4, 6])), (I8, torch.arange(-127.0, 128))):
        if fmt not in cands:
            continue
        w = levels[torch.randint(len(levels), (N, K), generator=g)] * (torch.randint(2, (N, K), generator=g) * 2 - 1)
        w[:, 0] = levels.max()
        w = w.to(torch.bfloat16).to(DEV)
        c = cands.index(fmt)
        r, _ = wo.run_select(mq, x, w, cands, orc.PER_CHANNEL, mi.clip_ratios(1))
        assert r.err[c] == 0.0 and r.err[1 - c] > 0.0 and r.best == c
        assert wo.run_score(mq, x, w, fmt, orc.PER_CHANNEL, mi.clip_ratios(1)) == (0.0, r.ref_energy)


# Both candidates' 4-bit values in one operand, in either order, and what goes on as two operands, in each tile.
@pytest.mark.parametrize("cands,ratios", [([FP4, I4], 1), ([I4, orc.FP4_E2M1_IEEE], 1), ([I8, FP8], 1), ([I4, FP4], 3)])
@pytest.mark.parametrize("shape", [(449, 1040, 192), (65, 63, 64), (1601, 1345, 64), (2049, 2049, 128)])
def test_weight_only_operands(mq, shape, cands, ratios):
    x, w = tensors(shape, 8300)
    wo.check_layer(mq, x, w, cands, orc.PER_CHANNEL, mi.clip_ratios(ratios), f"{shape} {cands}")


# One stage of 64 columns, two, three and an odd number more, in each tile of the products that share X, with rows of W apart.
@pytest.mark.parametrize("shape", [(65, 63, 64), (65, 63, 128), (1601, 1345, 64), (1601, 1345, 64 * 7), (2049, 2049, 64), (2049, 2049, 192)])
def test_weight_only_products_share_the_input(mq, shape):
    M, N, K = shape
    x, w = tensors(shape, 8250)
    apart = torch.full((N, K + 72), float("nan"), dtype=torch.bfloat16, device=DEV)[:, :K]
    apart.copy_(w)
    wo.check_layer(mq, x, apart, [FP4, I4], orc.PER_CHANNEL, mi.clip_ratios(1), shape)


@pytest.mark.parametrize("name", list(SHAPES))
def test_fp8_unit_products(mq, name):
    M, N, K = SHAPES[name]
    x, w = tensors(SHAPES[name], 8300)
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    out, res = mq.alloc_qbuffers(N, K, 8, cfg, DEV), mq.alloc_result(DEV)
    ws = torch.empty(mq.workspace_bytes(w, x, 2, mq.ERR_LAYER_OUTPUT_FP8_UNIT, cfg), dtype=torch.uint8, device=DEV)
    print(f"[case] {name} {SHAPES[name]}", flush=True)
    mq.select_layer(w, x, [I8, FP8], mq.ERR_LAYER_OUTPUT_FP8_UNIT, cfg, out, None, res, ws)
    torch.cuda.synchronize()
    r = mq.read_result(res)
    ref = orc.select_layer_wa(mi.to_f32_numpy(x), mi.to_f32_numpy(w), [I8, FP8], orc.PER_TENSOR)
    assert np.isclose(r.err[0], ref.errs[0], rtol=wa.E_RTOL) and np.isclose(r.ref_energy, ref.ref_energy, rtol=wa.E_RTOL)
    # what the unit's alignment drops: see test_gpu_random_layers.py
    assert abs(r.err[1] / ref.errs[1] - 1.0) <= wa.FP8_UNIT_RTOL + (1e-3 / np.sqrt(M * N) if M * N < 20000 else 0.0)


@pytest.mark.parametrize("name", ["cut to 20 stages, one more than divides", "small tiles"])
def test_unused_scratch_is_not_read(mq, name):
    """The pieces' partial sums are written before they are read: scratch full of NaN changes nothing."""
    x, w = tensors(SHAPES[name], 8400)
    cfg = mq.Cfg(mq.PER_TENSOR, mi.clip_ratios(1))
    out, res = mq.alloc_qbuffers(w.shape[0], w.shape[1], 8, cfg, DEV), mq.alloc_result(DEV, 2)
    n = mq.workspace_bytes(w, x, 2, mq.ERR_LAYER_OUTPUT, cfg)
    for i, fill in enumerate((0, 0xFF)):
        ws = torch.full((n,), fill, dtype=torch.uint8, device=DEV)
        mq.select_layer(w, x, [I8, FP8], mq.ERR_LAYER_OUTPUT, cfg, out, None, res[i], ws)
    torch.cuda.synchronize()
    assert torch.equal(res[0], res[1])


@pytest.mark.parametrize("rows,ld", [(130, 36 << 20), (300, 9 << 20), (300, 18 << 20)])
def test_rows_far_apart(mq, rows, ld):
    """Row strides at which a tile's rows reach beyond 2^32 bytes: of 64 rows (64-bit offsets), of 256 and of 128
    (smaller tiles)."""
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
