"""Sizes at the edges of the launch rules and tiles: where a pass changes its shape (one launch or
several, one or two stages of a sum, codes from the search or after it) and where a segment, a
row or a unit ends inside a workgroup's piece.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import mofq_inputs as mi
from oracle import mofq_oracle as orc
from tests.gpu_util import scales_to_f32, unpack_codes
from tests.test_gpu_w_only import check_tensor, mq  # noqa: F401

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
PAIR4, PAIR8 = [orc.INT4, orc.FP4_E2M1], [orc.FP8_E4M3, orc.INT8]


def _strided(rows, cols, pad, seed, dtype):
    w = mi.llama_like_weight(rows, cols + pad, seed=seed, dtype=dtype, device=DEV, outlier_frac=2e-3)
    return w[:, :cols]


# one launch (one workgroup, several), then three; one chunk; rows that lie apart
@pytest.mark.parametrize("rows,cols,pad", [(1, 8, 0), (8, 8192, 0), (8, 8200, 0), (3, 1000, 8), (67, 1000, 24), (1025, 2056, 0)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_per_tensor_passes(mq, rows, cols, pad, dtype):  # noqa: F811
    w = _strided(rows, cols, pad, rows + cols, dtype)
    check_tensor(mq, w, PAIR8, orc.PER_TENSOR, mi.clip_ratios(1), f16=rows == 67, label="tensor-edge")
    check_tensor(mq, w, PAIR4 + [orc.FP4_E2M1_IEEE], orc.PER_TENSOR, mi.clip_ratios(1), label="tensor-edge-4")


# rows of one chunk; units on both sides of the one-stage limit; segments that end inside rows and groups
@pytest.mark.parametrize("rows,cols,pad,group", [(700, 8, 0, 0), (1024, 40, 0, 0), (1025, 264, 8, 0), (2048, 24, 0, 0), (2049, 136, 8, 0), (5, 32768, 0, 0),
                                                 (33, 4128, 32, 32), (9, 16640, 0, 256), (70, 640, 64, 64)])
def test_emission_segments(mq, rows, cols, pad, group):  # noqa: F811
    w = _strided(rows, cols, pad, rows + cols, torch.float16)
    gran = orc.PER_GROUP if group else orc.PER_CHANNEL
    check_tensor(mq, w, PAIR4, gran, mi.clip_ratios(1), group, bool(group), label="emit-edge")
    check_tensor(mq, w, PAIR8, gran, mi.clip_ratios(3), group, False, label="emit-edge-8")


# inputs large enough that the search writes the codes itself; the first and last rows favour the format
# that the tensor as a whole does not take, so rows are done twice
@pytest.mark.parametrize("dtype,rows,cols,pad,cands,f16", [
    (torch.float32, 4100, 8192, 0, PAIR4, False), (torch.bfloat16, 3001, 23008, 32, PAIR8, True),
    (torch.float16, 16400, 4104, 0, [orc.FP4_E2M1, orc.INT4], False)])
def test_codes_written_by_the_single_candidate_search(mq, dtype, rows, cols, pad, cands, f16):  # noqa: F811
    w = _strided(rows, cols, pad, rows, dtype)
    g = torch.Generator(device=DEV).manual_seed(rows)
    for r in (slice(0, 40), slice(rows - 9, rows)):      # small integers: exact in the integer format
        w[r] = torch.randint(-7, 8, w[r].shape, generator=g, device=DEV).to(dtype)
        w[r, 5] = 7.0
    check_tensor(mq, w, cands, orc.PER_CHANNEL, mi.clip_ratios(1), f16=f16, label="ahead-single")


# bf16 rows searched through prefixes per bit pattern: tiles of the row, one and two groups of 64 candidates,
# one format and two, ratios that stretch the histogram; rows of zeros, of equal elements, of powers of two
# over the whole range, and rows so small that the scales or the elements are subnormal
@pytest.mark.parametrize("cols,n_clip,lo_clip,f16", [
    (1024, 32, 0.5, False), (2048, 16, 0.3, False), (2056, 64, 0.5, True), (4104, 8, 0.9, False), (5000, 50, 0.5, False), (3000, 20, 0.115, False), (3000, 20, 0.111, False),
    (6152, 65, 0.5, False), (8200, 100, 0.25, True), (12296, 20, 0.5, False), (24576, 9, 0.05, False),
    # from these on for every list of formats
    (1024, 52, 0.4, False), (2048, 26, 0.5, True), (4104, 13, 0.7, False)])
def test_bf16_pattern_prefixes(mq, cols, n_clip, lo_clip, f16):  # noqa: F811
    w = _strided(21, cols, 8, cols, torch.bfloat16)
    g = torch.Generator(device=DEV).manual_seed(cols)
    w[1] = 0.0
    w[2] = 0.75
    w[3] = torch.exp2(torch.randint(-40, 3, (cols,), generator=g, device=DEV).float()).to(torch.bfloat16) * w[3].sign()
    w[4] *= 1e-36
    w[5] = (w[5].float() * 2.0 ** -118).to(torch.bfloat16)
    w[6] = torch.where(w[6] > 0, w[6], -w[6] * 3).to(torch.bfloat16)
    w[7, 3] = -3.3e38 if not f16 else -6e4
    ratios = [lo_clip + (1.0 - lo_clip) * (i + 1) / n_clip for i in range(n_clip)]
    for cands in (PAIR8, [orc.INT8], [orc.FP8_E4M3], PAIR4, [orc.INT4], [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_CHANNEL, ratios, f16=f16, label="bf16-edge")


def test_bf16_search_writes_codes(mq):  # noqa: F811
    w = _strided(8209, 1048, 8, 3, torch.bfloat16)
    g = torch.Generator(device=DEV).manual_seed(3)
    w[:40] = torch.randint(-7, 8, (40, 1048), generator=g, device=DEV).to(torch.bfloat16)
    w[:40, 5] = 7.0
    check_tensor(mq, w, PAIR8, orc.PER_CHANNEL, mi.clip_ratios(40), label="bf16-ahead-8")
    check_tensor(mq, w, PAIR4, orc.PER_CHANNEL, mi.clip_ratios(40), label="bf16-ahead-4")


# groups searched through ranks of bit patterns: one and several rounds of candidates, 32- and 64-bit words,
# rows that lie apart, a last wave that is not full; groups of zeros, of equal or all-negative elements, of
# powers of two over the whole range, nearly exact ones, with subnormal scales, with one huge element
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("group,n_clip,lo_clip,f16,pad", [
    (64, 24, 0.5, True, 0), (64, 33, 0.2, False, 64), (128, 12, 0.9, False, 0), (128, 50, 0.5, True, 128),
    (128, 128, 0.02, False, 0), (256, 18, 0.5, True, 0), (256, 45, 0.3, False, 256),
    # from these on for every type and list of formats
    (64, 80, 0.5, True, 64), (128, 27, 0.4, True, 0), (256, 40, 0.6, False, 0)])
def test_group_pattern_ranks(mq, dtype, group, n_clip, lo_clip, f16, pad):  # noqa: F811
    w = _strided(13, 7 * group, pad, n_clip, dtype)
    g = torch.Generator(device=DEV).manual_seed(n_clip)
    v = [w[r, (r % 3) * group:(r % 3 + 1) * group] for r in range(13)]
    v[0][:] = 0.0
    v[1][:] = 0.75
    v[2][:] = -v[2].abs()
    v[3][:] = torch.exp2(torch.randint(-13, 3, (group,), generator=g, device=DEV).float()).to(dtype)
    v[4][:] = torch.randint(-7, 8, (group,), generator=g, device=DEV).to(dtype)
    v[5][:] = v[5] * 2.0 ** -11
    v[6][:] = (v[6].float() * (2.0 ** -17 if dtype == torch.float16 else 2.0 ** -119)).to(dtype)
    v[7][3] = -6.0e4
    v[8][:] = -1.5
    v[9][5:] = 0.0
    ratios = [lo_clip + (1.0 - lo_clip) * (i + 1) / n_clip for i in range(n_clip)]
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_GROUP, ratios, group, f16, label="group-rank-edge")


# the candidates of a last round that does not fill the group's lanes: eight, four, two and one lane to each; with scales
# in fp16 of groups so small that their rounding moves the scale off the counted patterns
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("group,n_clip", [(64, 81), (64, 82), (64, 84), (64, 86), (128, 33), (128, 36), (128, 40), (128, 47), (256, 68), (256, 72),
                                          (256, 80), (256, 91)])
def test_group_last_round(mq, dtype, group, n_clip):  # noqa: F811
    w = _strided(6, 5 * group, 0, n_clip, dtype)
    w[1, :2 * group] = (w[1, :2 * group].float() * 2.0 ** -15).to(dtype)
    w[2, group:] = (w[2, group:].float() * 2.0 ** -17).to(dtype)
    ratios = [0.45 + 0.55 * (i + 1) / n_clip for i in range(n_clip)]
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_GROUP, ratios, group, True, label="group-last-round")


# tables that descend and are long enough to be searched coarsely first: one more ratio than that takes, the longest;
# equal neighbours, neighbours an ulp apart, a wide geometric table, one that ends in a plateau
def _descending(kind, n):
    if kind == "even":
        return [float(r) for r in mi.clip_ratios(n)]
    if kind == "pairs":
        return [1.0 - 0.5 * (i // 2) / n for i in range(n)]
    if kind == "ulps":
        return [float(np.float32(0.8) - np.float32(2.0 ** -24) * i) for i in range(n)]
    if kind == "wide":
        return [0.02 ** (i / (n - 1)) for i in range(n)]
    return [max(1.0 - 0.9 * i / n, 0.6) for i in range(n)]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("group,n_clip,kind", [
    (64, 50, "even"), (64, 128, "wide"), (64, 61, "pairs"), (64, 100, "ulps"), (128, 33, "even"), (128, 50, "even"), (128, 64, "plateau"),
    (128, 128, "even"), (128, 99, "ulps"), (128, 40, "wide"), (256, 65, "even"), (256, 128, "wide"), (256, 90, "pairs")])
def test_group_gaps(mq, dtype, group, n_clip, kind):  # noqa: F811
    w = _strided(14, 6 * group, group, n_clip, dtype)
    g = torch.Generator(device=DEV).manual_seed(group + n_clip)
    v = [w[r, (r % 3) * group:(r % 3 + 2) * group] for r in range(14)]
    v[0][:] = 0.0
    v[1][:] = 0.75
    v[2][:] = -v[2].abs()
    v[3][:] = torch.exp2(torch.randint(-9, 3, (2 * group,), generator=g, device=DEV).float()).to(dtype)
    v[4][:] = torch.randint(-7, 8, (2 * group,), generator=g, device=DEV).to(dtype)      # nearly on one grid
    v[5][:] = (torch.randint(0, 8, (2 * group,), generator=g, device=DEV) + 0.5).to(dtype)   # on its boundaries
    v[6][:] = torch.rand(2 * group, generator=g, device=DEV).to(dtype)
    v[7][3] = -6.0e4
    v[8][:] = (v[8].float() * (2.0 ** -14 if dtype == torch.float16 else 2.0 ** 120)).to(dtype)
    v[9][5:] = 0.0
    v[10][:] = (v[10].float() * (2.0 ** -9 if dtype == torch.float16 else 2.0 ** -115)).to(dtype)
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_GROUP, _descending(kind, n_clip), group, label=f"group-gaps {kind}")


# the best ratio in every part of a table that descends, its last gap included: groups whose one large element is 3 to 9
# standard deviations of the others
@pytest.mark.parametrize("group,n_clip", [(64, 50), (128, 50), (128, 77), (256, 66), (256, 120)])
def test_group_gaps_everywhere(mq, group, n_clip):  # noqa: F811
    g = torch.Generator(device=DEV).manual_seed(n_clip)
    w = 0.02 * torch.randn(64, 8 * group, generator=g, device=DEV)
    large = torch.linspace(3.0, 9.0, 64 * 8, device=DEV).view(64, 8)
    w.view(64, 8, group)[:, :, 5] = 0.02 * large
    w = w.to(torch.float16)
    for cands in (PAIR4, [orc.INT4]):
        check_tensor(mq, w, cands, orc.PER_GROUP, _descending("even", n_clip), group, label="group-gaps-everywhere")


# fp16 rows and 8-bit formats, looked up by groups of patterns: one to four chunks per thread, one and two groups of 64
# candidates, tables as far as they reach and, in the last case, beyond (scored directly)
@pytest.mark.parametrize("cols,n_clip,lo_clip,f16", [
    (2048, 88, 0.5, True), (4096, 49, 0.7, False), (4104, 128, 0.5, False), (5000, 64, 0.3, True), (8200, 25, 0.5, False),
    (11008, 65, 0.6, False), (12296, 17, 0.5, True), (16384, 13, 0.5, False), (3072, 38, 0.5, False), (4096, 27, 0.5, True),
    (1544, 128, 0.6, False), (8192, 25, 0.26, False), (8192, 40, 0.02, False)])
def test_half_pattern_groups(mq, cols, n_clip, lo_clip, f16):  # noqa: F811
    w = _strided(15, cols, 8, cols, torch.float16)
    g = torch.Generator(device=DEV).manual_seed(cols)
    w[1] = 0.0
    w[2] = 0.75
    w[3] = torch.exp2(torch.randint(-24, 3, (cols,), generator=g, device=DEV).float()).to(torch.float16) * w[3].sign()
    w[4] = (w[4].float() * 2.0 ** -14).to(torch.float16)      # few patterns below the largest
    w[5] = (w[5].float() * 2.0 ** -19).to(torch.float16)
    w[6] = torch.where(w[6] > 0, w[6], -w[6] * 3)
    w[7, 3] = -6e4
    w[8] = torch.randint(-127, 128, (cols,), generator=g, device=DEV).to(torch.float16)
    w[9] = (torch.randint(0, 128, (cols,), generator=g, device=DEV) + 0.5).to(torch.float16)
    w[10] = -w[10].abs()
    w[11, 9:] = 0.0
    w[12] = torch.rand(cols, generator=g, device=DEV).to(torch.float16)
    w[13] = torch.randint(0, 0x7BFF, (cols,), generator=g, device=DEV).to(torch.int16).view(torch.float16)   # every pattern
    ratios = [lo_clip + (1.0 - lo_clip) * (i + 1) / n_clip for i in range(n_clip)]
    for cands in (PAIR8[::-1], PAIR8, [orc.INT8], [orc.FP8_E4M3]):
        check_tensor(mq, w, cands, orc.PER_CHANNEL, ratios, f16=f16, label="half-groups")


# enough rows that the search writes the codes itself
def test_half_pattern_groups_write_codes(mq):  # noqa: F811
    w = _strided(8200, 4096, 0, 3, torch.float16)
    w[:50] = (w[:50].float().sign() * 0.02).to(torch.float16)
    check_tensor(mq, w, PAIR8, orc.PER_CHANNEL, mi.clip_ratios(35), label="half-groups-ahead")


# groups whose candidates are scored by bisection of the ratios: groups of 32, and fp32 elements (16-bit ones are looked up,
# but for some formats alone); the numbers of ratios leave one and two candidates in the last gaps, after two to four halvings
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("group,n_clip,kind,f16", [
    (32, 64, "even", True), (32, 65, "even", False), (32, 128, "wide", False), (32, 86, "pairs", True), (32, 100, "ulps", False),
    (64, 43, "even", True), (64, 44, "plateau", False), (128, 33, "even", False), (128, 43, "even", True), (128, 44, "wide", True),
    (256, 65, "even", True), (256, 86, "pairs", False), (128, 40, "ascending", False)])
def test_direct_group_bisection(mq, dtype, group, n_clip, kind, f16):  # noqa: F811
    w = _strided(14, 6 * group, group, n_clip, dtype)
    g = torch.Generator(device=DEV).manual_seed(group + n_clip)
    v = [w[r, (r % 3) * group:(r % 3 + 2) * group] for r in range(14)]
    v[0][:] = 0.0
    v[1][:] = 0.75
    v[2][:] = -v[2].abs()
    v[3][:] = torch.exp2(torch.randint(-9, 3, (2 * group,), generator=g, device=DEV).float()).to(dtype)
    v[4][:] = torch.randint(-7, 8, (2 * group,), generator=g, device=DEV).to(dtype)      # nearly on one grid
    v[5][:] = (torch.randint(0, 8, (2 * group,), generator=g, device=DEV) + 0.5).to(dtype)   # on its boundaries
    v[6][:] = torch.rand(2 * group, generator=g, device=DEV).to(dtype)
    v[7][3] = -6.0e4
    small, large = (2.0 ** -14, 1.0) if dtype == torch.float16 else (2.0 ** -115, 2.0 ** 100)
    v[8][:] = (v[8].float() * large).to(dtype)      # squares beyond fp32
    v[9][5:] = 0.0
    v[10][:] = (v[10].float() * small).to(dtype)    # and below it
    v[11][:] = (v[11].float() * 2.0 ** -16).to(dtype)   # fp16 scales below the normal numbers
    ratios = _descending("even", n_clip)[::-1] if kind == "ascending" else _descending(kind, n_clip)
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1], [orc.FP4_E2M1_IEEE]):
        check_tensor(mq, w, cands, orc.PER_GROUP, ratios, group, f16, label=f"direct-group {kind}")


@pytest.mark.parametrize("group,n_clip", [(32, 64), (64, 40), (128, 64), (256, 120)])
def test_direct_group_bisection_everywhere(mq, group, n_clip):  # noqa: F811
    g = torch.Generator(device=DEV).manual_seed(n_clip)
    w = 0.02 * torch.randn(64, 8 * group, generator=g, device=DEV)
    w.view(64, 8, group)[:, :, 5] = 0.02 * torch.linspace(2.5, 9.0, 64 * 8, device=DEV).view(64, 8)
    for cands in (PAIR4, [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_GROUP, _descending("even", n_clip), group, True, label="direct-group-everywhere")


# as many groups as are resident at once, where bisection starts at fewer ratios
@pytest.mark.parametrize("dtype,group,rows,n_clip", [(torch.float32, 32, 1024, 20), (torch.float32, 64, 2048, 16), (torch.bfloat16, 32, 1024, 23),
                                                     (torch.float32, 128, 3072, 18), (torch.float32, 256, 4096, 22), (torch.float16, 64, 3100, 40)])
def test_direct_group_bisection_many_groups(mq, dtype, group, rows, n_clip):  # noqa: F811
    w = _strided(rows, 2048, 0, group, dtype)
    check_tensor(mq, w, PAIR4, orc.PER_GROUP, _descending("even", n_clip), group, True, label="direct-group-many")


# rows whose candidates are scored by bisection of the ratios: one wave per row to sixteen, masks of one and two words,
# even and uneven tables, long runs of equal errors, and a table that does not descend
@pytest.mark.parametrize("dtype,cols,n_clip,kind,f16", [
    (torch.float32, 264, 44, "even", False), (torch.float16, 600, 64, "pairs", True), (torch.bfloat16, 1000, 65, "ulps", False),
    (torch.float32, 2056, 18, "even", False), (torch.float32, 4104, 128, "wide", False), (torch.float32, 5000, 100, "even", True),
    (torch.float32, 8200, 63, "plateau", False), (torch.float32, 12296, 127, "ulps", False), (torch.float32, 16392, 20, "pairs", False),
    (torch.float32, 24584, 90, "even", False), (torch.float32, 4104, 50, "ascending", False)])
def test_row_bisection(mq, dtype, cols, n_clip, kind, f16):  # noqa: F811
    w = _strided(13, cols, 8, n_clip, dtype)
    g = torch.Generator(device=DEV).manual_seed(cols + n_clip)
    w[0] = 0.0
    w[1] = 0.75
    w[2] = -w[2].abs()
    w[3] = torch.exp2(torch.randint(-9, 3, (cols,), generator=g, device=DEV).float()).to(dtype)
    w[4] = torch.randint(-7, 8, (cols,), generator=g, device=DEV).to(dtype)                # nearly on one grid
    w[5] = (torch.randint(0, 8, (cols,), generator=g, device=DEV) + 0.5).to(dtype)         # on its boundaries
    w[6, 3] = -6.0e4
    w[7] = (w[7].float() * (2.0 ** -14 if dtype == torch.float16 else 2.0 ** 100)).to(dtype)    # squares beyond fp32
    w[8] = (w[8].float() * (2.0 ** -9 if dtype == torch.float16 else 2.0 ** -115)).to(dtype)    # and below it
    w[9, 5:] = 0.0
    # the best ratio in many places of the table
    for r in (10, 11, 12):
        w[r] = (0.02 * torch.randn(cols, generator=g, device=DEV)).to(dtype)
        w[r, 7] = 0.02 * (4.0 + 3.0 * (r - 10))
    ratios = _descending("even", n_clip)[::-1] if kind == "ascending" else _descending(kind, n_clip)
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1], [orc.FP4_E2M1_IEEE]):
        check_tensor(mq, w, cands, orc.PER_CHANNEL, ratios, 0, f16, label=f"row-bisection {kind}")


@pytest.mark.parametrize("cols,n_clip", [(520, 50), (4104, 100)])
def test_row_bisection_everywhere(mq, cols, n_clip):  # noqa: F811
    g = torch.Generator(device=DEV).manual_seed(n_clip)
    w = 0.02 * torch.randn(200, cols, generator=g, device=DEV)
    w[:, 5] = 0.02 * torch.linspace(3.5, 14.0, 200, device=DEV)
    for cands in (PAIR4, [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_CHANNEL, _descending("even", n_clip), 0, label="row-bisection-everywhere")


# The last ratios are so small that their scales become 1, beside a scale just above 1 (index 31) and the row's best ones
# below it: the scales of the gap between them are not between its ends.  Rows of an even index that way for INT4, of an odd
# one for E2M1; the last two with all scales above 1 and with all of them 1.
@pytest.mark.parametrize("cols", [2056, 8200, 16392])
@pytest.mark.parametrize("f16,tiny", [(True, 1e-9), (False, 1e-39)])
def test_row_bisection_degenerate_scales(mq, cols, f16, tiny):  # noqa: F811
    ratios = [1.0 - 0.9 * i / 39 for i in range(40)] + [tiny] * 24
    g = torch.Generator(device=DEV).manual_seed(cols)
    w = 0.5 * torch.randn(26, cols, generator=g, device=DEV)
    above = torch.linspace(1.0005, 1.02, 13, device=DEV)
    w[0::2, 0] = orc.qmax(orc.INT4) / ratios[31] * above
    w[1::2, 0] = orc.qmax(orc.FP4_E2M1) / ratios[31] * above
    w[24, 0] = 100.0
    w[25] = w[25] * (2.0 ** -30 if f16 else 2.0 ** -130)
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1], [orc.FP4_E2M1_IEEE]):
        check_tensor(mq, w, cands, orc.PER_CHANNEL, ratios, 0, f16, label=f"row-bisection-degenerate {tiny}")


# ratios so small that a group's largest elements are 2^31 ulps of the first counted pattern and more: the last tables
# of the rank kernel and, beyond them, the direct kernel (bf16: 128 patterns per binade)
@pytest.mark.parametrize("lo_clip", [1e-5, 4e-6, 2e-6, 1e-6, 1e-7])
@pytest.mark.parametrize("group", [64, 128, 256])
def test_group_tiny_ratios(mq, group, lo_clip):  # noqa: F811
    w = _strided(9, 4 * group, 0, group, torch.bfloat16)
    w[2, :group] = 0.75
    w[3, :group] = -w[3, :group].abs()
    ratios = [1.0 - 0.5 * i / 44 for i in range(44)] + [lo_clip]
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_GROUP, ratios, group, label=f"group-tiny-ratio {lo_clip}")


# The reported unit error is the sum of the squared residuals element by element.  x - g s is one fused operation
# (2^-53 of it, twice that in the square), a lane adds at most `per_lane` squares, the lanes and waves of a unit
# are summed in `levels` additions, all terms positive: the sum is within (2 + per_lane + levels) 2^-53 of the exact one.
@pytest.mark.parametrize("dtype,cols,group,fmts,per_lane,levels", [
    (torch.bfloat16, 2048, 0, [orc.INT8, orc.FP8_E4M3], 8, 9), (torch.bfloat16, 5000, 0, [orc.INT8, orc.FP8_E4M3], 24, 9),
    (torch.bfloat16, 24576, 0, [orc.INT8, orc.FP8_E4M3], 96, 9),
    (torch.bfloat16, 1024, 64, PAIR4, 8, 3), (torch.bfloat16, 1024, 128, PAIR4, 8, 4), (torch.bfloat16, 1024, 256, PAIR4, 8, 5),
    (torch.float16, 1024, 64, PAIR4, 8, 3), (torch.float16, 1024, 128, PAIR4, 8, 4), (torch.float16, 1024, 256, PAIR4, 8, 5)])
def test_unit_errors_are_sums_of_residuals(mq, dtype, cols, group, fmts, per_lane, levels):  # noqa: F811
    rows = 64 if group else 24
    w = _strided(rows, cols, 0, cols + group, dtype)
    x = w.double().cpu().numpy().reshape(-1, group or cols)
    cfg = mq.Cfg(orc.PER_GROUP if group else orc.PER_CHANNEL, mi.clip_ratios(50), group)
    bits = orc.bits(fmts[0])
    for cands in ([fmts[0]], [fmts[1]], fmts):
        out = mq.alloc_qbuffers(rows, cols, bits, cfg, DEV)
        res = mq.alloc_result(DEV)
        ws = torch.empty(mq.workspace_bytes(w, None, len(cands), mq.ERR_TENSOR, cfg), dtype=torch.uint8, device=DEV)
        mq.select_layer(w, None, cands, mq.ERR_TENSOR, cfg, out, None, res, ws)
        torch.cuda.synchronize()
        fmt = cands[mq.read_result(res).best]
        print(f"[case] residual sums {dtype} cols={cols} group={group} cands={cands}", flush=True)
        g = orc.decode_array(fmt, unpack_codes(out.codes, rows, cols, bits)).astype(np.float64).reshape(x.shape)
        s = scales_to_f32(out.scales).astype(np.float64)[:, None]
        d = x.astype(np.longdouble) - (g * s)      # g s is exact in fp64
        want = (d * d).sum(axis=1)
        got = out.unit_err.cpu().numpy().astype(np.longdouble)
        assert np.max(np.abs(got - want) / want) <= (2 + per_lane + levels) * 2.0 ** -53


# fp16 rows searched through the histogram: every tile of the row (one to three masks of noted negative
# elements), all elements in a group's last pattern (the largest weighted count), all of them negative
@pytest.mark.parametrize("cols", [2048, 4096, 8200, 12296, 24576])
def test_fp16_histogram_counts(mq, cols):  # noqa: F811
    w = _strided(7, cols, 8, cols, torch.float16)
    last = torch.tensor([0x3807], dtype=torch.int16, device=DEV).view(torch.float16)   # pattern 7 modulo 8
    w[1] = last
    w[2] = -last
    w[3] = -w[3].abs()
    w[4, : cols // 2] = last
    w[5, cols - 1] = -w[5].abs().max() * 2
    for cands in (PAIR4, [orc.INT4], [orc.FP4_E2M1]):
        check_tensor(mq, w, cands, orc.PER_CHANNEL, mi.clip_ratios(100), label="fp16-edge")
