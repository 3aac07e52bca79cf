"""The largest bit pattern below a level boundary, as the histogram searches take it: the top bits of
decision_edge(threshold) / inv in fp64, against the decision fl32(|x| * inv) <= threshold on every pattern."""
import numpy as np
import pytest

E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]
E4M3 = [m * 2.0 ** -9 for m in range(8)] + [(8 + m) * 2.0 ** (e - 10) for e in range(1, 16) for m in range(8)][:119]


def thresholds(levels):
    mid = np.array([(a + b) / 2 for a, b in zip(levels, levels[1:])], dtype=np.float32)
    odd = np.arange(len(mid)) % 2 == 1   # the tie goes to the even code above
    return np.where(odd, np.nextafter(mid, np.float32(0)), mid)


def edge(thr):
    up = np.nextafter(thr, np.float32(np.inf))
    mid = 0.5 * (thr.astype(np.float64) + up.astype(np.float64))
    return mid * np.where(thr.view(np.uint32) & 1, 1 - 2.0 ** -40, 1 + 2.0 ** -40)


def scales(amax, qmax):
    """Clip ratios of absolute maxima with few bits (ties are common) and with many, fp32 and fp16 scales."""
    r = np.linspace(0.5, 1.0, 16, dtype=np.float32)
    s = (r[:, None] * amax[None, :].astype(np.float32)).ravel() / np.float32(qmax)
    return np.unique(np.concatenate([s, s.astype(np.float16).astype(np.float32)]).astype(np.float32))


@pytest.mark.parametrize("fmt", ["int4", "e2m1", "int8", "e4m3"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_largest_pattern_below_a_boundary(fmt, dtype):
    levels = {"int4": list(range(9)), "e2m1": E2M1, "int8": list(range(129)), "e4m3": E4M3}[fmt]
    thr = thresholds([float(v) for v in levels])
    qmax = {"int4": 7, "e2m1": 6, "int8": 127, "e4m3": 448}[fmt]
    if dtype == "f16":
        first, mant, bias = 1 << 10, 10, 15
        v = np.arange(first, 0x7C00, dtype=np.uint16).view(np.float16).astype(np.float32)
    else:   # 20 binades and more below 1
        first, mant, bias = 90 << 7, 7, 127
        v = (np.arange(first, 130 << 7, dtype=np.uint32) << 16).view(np.float32)
    rng = np.random.default_rng(5)
    few = np.array([0.5, 0.75, 1.0, 1.75, 7 / 8, 0.375, 3.0], dtype=np.float32)
    amax = np.concatenate([few, rng.choice(v[(v > 0.01) & (v < 4)], 5 if len(thr) > 8 else 40)])
    for s in scales(amax, qmax):
        if s == 0:
            continue
        inv = np.float32(1) / s
        passes = np.searchsorted(v * inv, thr, side="right")   # products are monotone: how many patterns pass
        s64, i64 = np.float64(s), np.float64(inv)
        unit = s64 + s64 * (1.0 - s64 * i64)   # 1 - s inv has fewer than 53 bits: what a fused step gives too
        top = ((edge(thr) * unit).view(np.uint64) >> np.uint64(32 + 20 - mant)).astype(np.int64)
        n = top - ((1023 - bias) << mant) - first + 1
        assert np.array_equal(np.clip(n, 0, len(v)), passes), (fmt, dtype, s)
