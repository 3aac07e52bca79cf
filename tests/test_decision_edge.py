"""The arithmetic of the histogram searches, as the kernels have it (native/arithmetic.hip): the largest bit pattern below a
level boundary, the top bits of decision_edge(threshold) / inv in fp64, against the decision fl32(|x| * inv) <= threshold
on every pattern; scales and their reciprocals without a division, against the division."""
import numpy as np
import pytest

from tests import native

E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]
E4M3 = [m * 2.0 ** -9 for m in range(8)] + [(8 + m) * 2.0 ** (e - 10) for e in range(1, 16) for m in range(8)][:119]


def thresholds(levels):
    mid = np.array([(a + b) / 2 for a, b in zip(levels, levels[1:])], dtype=np.float32)
    odd = np.arange(len(mid)) % 2 == 1   # the tie goes to the even code above
    return np.where(odd, np.nextafter(mid, np.float32(0)), mid)


def scales(amax, qmax):
    """Clip ratios of absolute maxima with few bits (ties are common) and with many, fp32 and fp16 scales."""
    r = np.linspace(0.5, 1.0, 16, dtype=np.float32)
    s = (r[:, None] * amax[None, :].astype(np.float32)).ravel() / np.float32(qmax)
    return np.unique(np.concatenate([s, s.astype(np.float16).astype(np.float32)]).astype(np.float32))


@pytest.mark.parametrize("fmt", ["int4", "e2m1", "int8", "e4m3"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_largest_pattern_below_a_boundary(fmt, dtype):
    lib = native.load()
    levels = {"int4": list(range(9)), "e2m1": E2M1, "int8": list(range(129)), "e4m3": E4M3}[fmt]
    thr = thresholds([float(v) for v in levels])
    qmax = {"int4": 7, "e2m1": 6, "int8": 127, "e4m3": 448}[fmt]
    if dtype == "f16":
        first = 1 << 10
        v = np.arange(first, 0x7C00, dtype=np.uint16).view(np.float16).astype(np.float32)
    else:   # 20 binades and more below 1
        first = 90 << 7
        v = (np.arange(first, 130 << 7, dtype=np.uint32) << 16).view(np.float32)
    rng = np.random.default_rng(5)
    few = np.array([0.5, 0.75, 1.0, 1.75, 7 / 8, 0.375, 3.0], dtype=np.float32)
    amax = np.concatenate([few, rng.choice(v[(v > 0.01) & (v < 4)], 5 if len(thr) > 8 else 40)])
    for s in scales(amax, qmax):
        if s == 0:
            continue
        inv = np.float32(1) / s
        passes = np.searchsorted(v * inv, thr, side="right")   # products are monotone: how many patterns pass
        n = np.empty(len(thr), dtype=np.int32)
        lib.arithmetic_patterns(dtype == "bf16", thr.ctypes.data, len(thr), s, inv, first, n.ctypes.data)
        assert np.array_equal(np.clip(n, 0, len(v)), passes), (fmt, dtype, s)


@pytest.mark.parametrize("qmax", [7, 6])
def test_scales_are_the_quotients(qmax):
    """Every mantissa: of an exponent in the middle, and of those that leave the smallest normal quotients."""
    lib = native.load()
    least = np.float32(qmax * 2.0 ** -126).view(np.uint32)   # its quotient is 2^-126
    for first, count in ((127 << 23, 1 << 23), (int(least), 1 << 23)):
        assert lib.arithmetic_quotients(qmax == 6, first, count) == 0


@pytest.mark.gpu
def test_reciprocals_are_the_quotients():
    """Every float from 2^-126 to 2^125."""
    import torch
    lib = native.load()
    bad = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    assert lib.arithmetic_reciprocals(1 << 23, (251 << 23) + 1, bad.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert bad.item() == 0
