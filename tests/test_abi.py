"""The C-ABI library loads on a host without a GPU and exports every symbol that
include/mofq.h declares; host-only entry points and argument validation (which
happens before anything is enqueued) behave as documented."""
import ctypes as C
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2305_12356_amd import build as b
    if not os.path.exists(b.LIB):
        b.build()
    from paper_2305_12356_amd import binding
    return binding


def _declared():
    text = open(os.path.join(ROOT, "include", "mofq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mofq_[a-z_]+)\s*\(", text)))


def test_header_symbols_exported(lib):
    names = _declared()
    assert {"mofq_quantize", "mofq_score", "mofq_select_layer", "mofq_workspace_bytes",
            "mofq_num_units", "mofq_status_string"} <= set(names)
    raw = C.CDLL(lib.LIB_PATH)
    for n in names:
        assert hasattr(raw, n), n


def test_struct_layout_matches_header(lib):
    assert C.sizeof(lib.TensorDesc) == 40
    assert C.sizeof(lib.ScaleCfg) == 24
    assert C.sizeof(lib.QOut) == 32
    assert C.sizeof(lib.Result) == 8 + 8 * 4 + 8


def test_num_units_and_status_strings(lib):
    assert lib.num_units(4096, 11008, lib.PER_CHANNEL) == 4096
    assert lib.num_units(4096, 11008, lib.PER_GROUP, 128) == 4096 * 86
    assert lib.num_units(4096, 11008, lib.PER_TENSOR) == 1
    assert lib.num_units(4096, 11000, lib.PER_GROUP, 128) == -1
    assert lib.num_units(0, 8, lib.PER_CHANNEL) == -1
    for s in (0, -1, -2, -3, -4, -5):
        assert lib.status_string(s) and "unknown" not in lib.status_string(s)
    assert "unknown" in lib.status_string(-99)


def test_host_side_validation_without_gpu(lib):
    """Errors are detected on the host before anything is enqueued."""
    L = lib._lib
    clip = np.ones(1, dtype=np.float32)
    cfg = lib.ScaleCfg(lib.PER_CHANNEL, 0, lib.F32, 1, clip.ctypes.data_as(C.POINTER(C.c_float)))
    good = lib.TensorDesc(0x1000, lib.F16, 16, 64, 64)
    out = lib.QOut(0x2000, 0x3000, None, None)
    ws = C.c_void_p(0x4000)
    # null tensor, null data
    assert L.mofq_quantize(None, 0, C.byref(cfg), C.byref(out), None, ws, 1 << 20, None) == -1
    bad = lib.TensorDesc(None, lib.F16, 16, 64, 64)
    assert L.mofq_quantize(C.byref(bad), 0, C.byref(cfg), C.byref(out), None, ws, 1 << 20, None) == -1
    # cols not a multiple of 8, misaligned data
    bad = lib.TensorDesc(0x1000, lib.F16, 16, 60, 64)
    assert L.mofq_quantize(C.byref(bad), 0, C.byref(cfg), C.byref(out), None, ws, 1 << 20, None) == -3
    bad = lib.TensorDesc(0x1004, lib.F16, 16, 64, 64)
    assert L.mofq_quantize(C.byref(bad), 0, C.byref(cfg), C.byref(out), None, ws, 1 << 20, None) == -3
    # unknown format, too many clip ratios, bad ratio
    assert L.mofq_quantize(C.byref(good), 9, C.byref(cfg), C.byref(out), None, ws, 1 << 20, None) == -1
    cfg2 = lib.ScaleCfg(lib.PER_CHANNEL, 0, lib.F32, 1000, clip.ctypes.data_as(C.POINTER(C.c_float)))
    assert L.mofq_quantize(C.byref(good), 0, C.byref(cfg2), C.byref(out), None, ws, 1 << 20, None) == -1
    zero = np.zeros(1, dtype=np.float32)
    cfg3 = lib.ScaleCfg(lib.PER_CHANNEL, 0, lib.F32, 1, zero.ctypes.data_as(C.POINTER(C.c_float)))
    assert L.mofq_quantize(C.byref(good), 0, C.byref(cfg3), C.byref(out), None, ws, 1 << 20, None) == -1
    # group size that does not divide the row
    cfg4 = lib.ScaleCfg(lib.PER_GROUP, 128, lib.F32, 1, clip.ctypes.data_as(C.POINTER(C.c_float)))
    assert L.mofq_quantize(C.byref(good), 0, C.byref(cfg4), C.byref(out), None, ws, 1 << 20, None) == -2
    # workspace too small / missing
    assert L.mofq_quantize(C.byref(good), 0, C.byref(cfg), C.byref(out), None, ws, 16, None) == -4
    assert L.mofq_quantize(C.byref(good), 0, C.byref(cfg), C.byref(out), None, None, 1 << 20, None) == -4
    # candidates of different bit-widths
    cands = (C.c_int32 * 2)(lib.INT4, lib.FP8_E4M3)
    res = C.c_void_p(0x5000)
    assert L.mofq_select_layer(C.byref(good), None, cands, 2, lib.ERR_TENSOR, C.byref(cfg),
                               C.byref(out), None, res, ws, 1 << 20, None) == -1
    # weight-only select with the layer-output metric
    cands = (C.c_int32 * 2)(lib.INT4, lib.FP4_E2M1)
    assert L.mofq_select_layer(C.byref(good), None, cands, 2, lib.ERR_LAYER_OUTPUT, C.byref(cfg),
                               C.byref(out), None, res, ws, 1 << 20, None) == -1


def test_workspace_bytes_host_only(lib):
    L = lib._lib
    clip = np.ones(4, dtype=np.float32)
    cfg = lib.ScaleCfg(lib.PER_GROUP, 128, lib.F16, 4, clip.ctypes.data_as(C.POINTER(C.c_float)))
    t = lib.TensorDesc(0x1000, lib.F16, 4096, 11008, 11008)
    n1 = L.mofq_workspace_bytes(C.byref(t), None, 1, lib.ERR_TENSOR, C.byref(cfg))
    n2 = L.mofq_workspace_bytes(C.byref(t), None, 2, lib.ERR_TENSOR, C.byref(cfg))
    units = 4096 * 86
    assert n1 >= units * (4 + 4 + 8 + 8) and n2 >= units * (2 * 16 + 8) and n2 > n1
    assert L.mofq_workspace_bytes(C.byref(t), None, 0, lib.ERR_TENSOR, C.byref(cfg)) == 0


def test_search_groups_host_only(lib):
    """mofq_select_layers_search_groups: tensors of one row length and dtype inside a batch
    (at most 12 tensors / 512 MB) share a launch, at most 8 per launch."""
    L = lib._lib

    def groups(descs, cands):
        n = len(descs)
        w = (lib.TensorDesc * n)(*descs)
        c = (C.c_int32 * len(cands))(*cands)
        first = (C.c_int32 * n)()
        assert L.mofq_select_layers_search_groups(n, w, c, len(cands), first) == 0
        return list(first)

    def t(rows, cols, dtype=None):
        return lib.TensorDesc(0x1000, lib.F16 if dtype is None else dtype, rows, cols, cols)

    pair = [lib.INT4, lib.FP4_E2M1]
    # one 7B-shaped block (386 MB): every 4096-column tensor in one group, the down projection alone
    block = [t(4096, 4096)] * 4 + [t(11008, 4096)] * 2 + [t(4096, 11008)]
    assert groups(block, pair) == [0, 0, 0, 0, 0, 0, 6]
    # not adjacent, other dtype in between, more than 8 members
    mixed = [t(8, 1024), t(8, 2048), t(16, 1024), t(8, 1024, lib.BF16)] + [t(8, 1024)] * 8
    assert groups(mixed, pair) == [0, 1, 0, 3] + [0] * 6 + [10, 10]
    # a batch ends after 12 tensors ...
    assert groups([t(8, 1024)] * 14, pair) == [0] * 8 + [8] * 4 + [12] * 2
    # ... or before it would exceed 512 MB (the first tensor of a batch may be larger than that)
    big = [t(16384, 8192)] * 3                                # 256 MB each
    assert groups(big, pair) == [0, 0, 2]
    assert groups([t(32768, 16384), t(8, 16384)], pair) == [0, 1]
    # three candidates need two launches per tensor: nothing is joined
    assert groups(block, [lib.INT4, lib.FP4_E2M1, lib.FP4_E2M1_IEEE]) == list(range(7))
    # invalid arguments
    c = (C.c_int32 * 2)(*pair)
    w = (lib.TensorDesc * 1)(t(8, 1024))
    first = (C.c_int32 * 1)()
    assert L.mofq_select_layers_search_groups(0, w, c, 2, first) != 0
    assert L.mofq_select_layers_search_groups(1, w, c, 2, None) != 0
    assert L.mofq_select_layers_search_groups(1, w, c, 0, first) != 0


def test_select_layers_long_candidate_lists_host_only(lib):
    """Candidate lists of three and four formats are legal (MOFQ_MAX_CANDIDATES = 4): the batched
    call must take them through launches of at most two formats each and never index past its
    per-launch tables.  Without a GPU the first launch fails, so the call returns the launch
    status (a crash here is the bug this guards against); five candidates are rejected on the
    host."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("uses made-up device pointers: only where nothing can be launched")
    L = lib._lib
    clip = np.array([1.0, 0.9], dtype=np.float32)
    cfg = lib.ScaleCfg(lib.PER_CHANNEL, 0, lib.F32, 2, clip.ctypes.data_as(C.POINTER(C.c_float)))
    n = 3
    w = (lib.TensorDesc * n)(*[lib.TensorDesc(0x10000, lib.F16, 16, 4096, 4096)] * n)
    out = (lib.QOut * n)(*[lib.QOut(0x20000, 0x30000, None, None)] * n)
    res, ws = C.c_void_p(0x50000), C.c_void_p(0x100000)
    for cands in ([lib.INT4, lib.FP4_E2M1, lib.FP4_E2M1_IEEE],
                  [lib.INT4, lib.FP4_E2M1, lib.FP4_E2M1_IEEE, lib.INT4],
                  [lib.FP4_E2M1, lib.FP4_E2M1, lib.INT4]):
        c = (C.c_int32 * len(cands))(*cands)
        need = L.mofq_select_layers_workspace_bytes(n, w, len(cands), C.byref(cfg))
        assert need > 0
        rc = L.mofq_select_layers(n, w, c, len(cands), C.byref(cfg), out, res, ws, need, None, None)
        assert rc in (0, -5), rc
    c5 = (C.c_int32 * 5)(lib.INT4, lib.FP4_E2M1, lib.INT4, lib.FP4_E2M1, lib.INT4)
    assert L.mofq_select_layers(n, w, c5, 5, C.byref(cfg), out, res, ws, 1 << 20, None, None) == -1


def test_select_layers_wa_host_side(lib):
    """mofq_select_layers_wa: workspace sizing and argument validation happen on the host, before
    anything is enqueued (fake device addresses are never touched)."""
    L = lib._lib
    one = np.ones(1, dtype=np.float32)
    cfg = lib.ScaleCfg(lib.PER_TENSOR, 0, lib.F32, 1, one.ctypes.data_as(C.POINTER(C.c_float)))
    # a decoder block at a small size: q, k, v share one activation, gate and up another
    dims = [(256, 128), (256, 128), (256, 128), (128, 128), (384, 128), (384, 128), (128, 384)]
    n = len(dims)
    w = (lib.TensorDesc * n)(*[lib.TensorDesc(0x100000 * (i + 1), lib.BF16, o, k, k) for i, (o, k) in enumerate(dims)])
    xaddr = [0xA00000, 0xA00000, 0xA00000, 0xB00000, 0xC00000, 0xC00000, 0xD00000]
    x = (lib.TensorDesc * n)(*[lib.TensorDesc(xaddr[i], lib.BF16, 64, k, k) for i, (o, k) in enumerate(dims)])
    w_out = (lib.QOut * n)(*[lib.QOut(0x2000000 + 0x100000 * i, 0x3000000 + 256 * i, None, None) for i in range(n)])
    cand = (C.c_int32 * 2)(lib.INT8, lib.FP8_E4M3)
    need = {m: L.mofq_select_layers_wa_workspace_bytes(n, w, x, 2, m, C.byref(cfg))
            for m in (lib.ERR_LAYER_OUTPUT, lib.ERR_LAYER_OUTPUT_FP8_UNIT)}
    single = max(L.mofq_workspace_bytes(C.byref(w[i]), C.byref(x[i]), 2, lib.ERR_LAYER_OUTPUT, C.byref(cfg)) for i in range(n))
    assert need[lib.ERR_LAYER_OUTPUT] >= single > 0
    # the exact product also keeps the E4M3 grid values of X and W as bf16
    assert need[lib.ERR_LAYER_OUTPUT] > need[lib.ERR_LAYER_OUTPUT_FP8_UNIT] > 0
    # operands of one group of layers, not of the whole model: a second block adds nothing
    w2 = (lib.TensorDesc * (2 * n))(*(list(w) + list(w)))
    x2 = (lib.TensorDesc * (2 * n))(*(list(x) + list(x)))
    assert L.mofq_select_layers_wa_workspace_bytes(2 * n, w2, x2, 2, lib.ERR_LAYER_OUTPUT, C.byref(cfg)) <= 2 * need[lib.ERR_LAYER_OUTPUT]
    # sizes: wrong metric, mismatched inner dimension
    assert L.mofq_select_layers_wa_workspace_bytes(n, w, x, 2, lib.ERR_TENSOR, C.byref(cfg)) == 0
    xbad = (lib.TensorDesc * n)(*[lib.TensorDesc(xaddr[i], lib.BF16, 64, 64, 64) for i in range(n)])
    assert L.mofq_select_layers_wa_workspace_bytes(n, w, xbad, 2, lib.ERR_LAYER_OUTPUT, C.byref(cfg)) == 0
    res, ws = C.c_void_p(0x5000000), C.c_void_p(0x6000000)
    args = lambda **kw: [kw.get("n", n), kw.get("w", w), kw.get("x", x), kw.get("cand", cand), kw.get("n_cand", 2),
                         kw.get("metric", lib.ERR_LAYER_OUTPUT), C.byref(cfg), kw.get("w_out", w_out), None,
                         res, ws, kw.get("ws_bytes", need[lib.ERR_LAYER_OUTPUT]), None]
    assert L.mofq_select_layers_wa(*args(n=0)) == -1
    assert L.mofq_select_layers_wa(*args(metric=lib.ERR_TENSOR)) == -1
    assert L.mofq_select_layers_wa(*args(x=xbad)) == -1
    assert L.mofq_select_layers_wa(*args(ws_bytes=need[lib.ERR_LAYER_OUTPUT] - 1)) == -4
    cand4 = (C.c_int32 * 2)(lib.INT4, lib.FP4_E2M1)
    assert L.mofq_select_layers_wa(*args(cand=cand4)) == -2          # no 4-bit matrix-core path
    w16 = (lib.TensorDesc * n)(*[lib.TensorDesc(0x100000 * (i + 1), lib.F16, o, k, k) for i, (o, k) in enumerate(dims)])
    assert L.mofq_select_layers_wa(*args(w=w16)) == -2               # the reference product takes bf16
    no_codes = (lib.QOut * n)(*[lib.QOut(None, 0x3000000, None, None) for _ in range(n)])
    assert L.mofq_select_layers_wa(*args(w_out=no_codes)) == -1


def test_units_workspace_is_the_search_records(lib):
    clip = np.ones(1, dtype=np.float32)
    w = lib.TensorDesc(0x100000, lib.F16, 4096, 4096, 4096)
    for gran, group in ((lib.PER_CHANNEL, 0), (lib.PER_GROUP, 128)):
        cfg = lib.ScaleCfg(gran, group, lib.F32, 1, clip.ctypes.data_as(C.POINTER(C.c_float)))
        need = lib._lib.mofq_workspace_bytes(C.byref(w), None, 2, lib.ERR_TENSOR, C.byref(cfg))
        assert lib._lib.mofq_select_units_workspace_bytes(C.byref(w), 2, C.byref(cfg)) == need > 0
