"""GPU parity of the row kernels that spread a row over the waves of a
workgroup (contiguous leaves of 64, strided lanes off the one-wave kernels),
against the CPU oracle, bit for bit, at the edges of their passes (4096
elements a wave), leaves, vectors and wave counts."""
import numpy as np
import pytest

import oracle
from paper_2609_11356_amd import inputs
from tests.gpu_util import assert_bits_equal, dev_bf16, dev_f32, host_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_11356_amd import dg as _dg
    _dg.lib()
    return _dg


ORDERS = [dict(leaf_w=64), dict(leaf_w=256, leaf_layout="strided", lane_fold="down"),
          dict(leaf_w=128, leaf_layout="strided"), dict(leaf_w=64, leaf_layout="strided", lane_fold="down")]
# one leaf, one pass and one more, 2 / 4 / 8 / 16 waves and past them (walked
# in super-passes), odd lengths (rows off every vector), 64 passes and past
COLS = [1, 63, 65, 4095, 4096, 4097, 8191, 8193, 16385, 32769, 65536, 65537, 131071, 262144, 262147]


@pytest.mark.parametrize("cols", COLS)
@pytest.mark.parametrize("oi", range(len(ORDERS)))
@pytest.mark.parametrize("op", ["rowsum", "sumsq", "rmsnorm", "layernorm", "softmax"])
def test_rows_over_waves(dg, op, oi, cols):
    import torch
    rows = 5 if cols < 70000 else 2
    out = "bf16" if (oi + cols) % 2 else "f32"
    desc = dict(ORDERS[oi], out="f32" if op in ("rowsum", "sumsq") else out,
                reduce="sumsq" if op in ("sumsq", "rmsnorm") else "sum")
    if cols % 2:
        desc["norm_round"] = "pre_weight"
    X = inputs.lognormal_f32(cols + 7 * oi, (rows, cols), sigma=1.0)
    if op == "layernorm":
        X = (X + 5).astype(np.float32)
    elif op == "softmax" and cols > 8:
        X[0, cols // 2] = -np.inf        # a masked element
        X[1, :] = -200.0                 # all exponentials 1 from a low maximum
        X[1, cols - 1] = 3.0             # ... and the rest below the exponential's range
    w, b = inputs.normal_bf16(cols + 5, (cols,), 1.0), inputs.normal_bf16(cols + 6, (cols,), 1.0)
    print("%s %s rows %d cols %d" % (op, desc, rows, cols), flush=True)
    d = dg.Desc(**desc)
    tdt = torch.bfloat16 if desc["out"] == "bf16" else torch.float32
    dX = dev_f32(X)
    if op in ("rowsum", "sumsq"):
        got = torch.full((rows,), float("nan"), device="cuda")
        dg.dg_rowsum(d, dX, got)
        want = oracle.rowsum(desc, X)
    else:
        got = torch.full(X.shape, float("nan"), dtype=tdt, device="cuda")
        if op == "rmsnorm":
            dg.dg_rmsnorm(d, dX, dev_bf16(w), 1e-5, got)
            want = oracle.rmsnorm(desc, X, w, eps=1e-5)
        elif op == "layernorm":
            dg.dg_layernorm(d, dX, dev_bf16(w), dev_bf16(b), 1e-5, got)
            want = oracle.layernorm(desc, X, w, b, eps=1e-5)
        else:
            dg.dg_softmax(d, dX, got)
            want = oracle.softmax(desc, X)
    torch.cuda.synchronize()
    assert_bits_equal(host_bits(got), want, "%s %s cols %d" % (op, desc, cols))


@pytest.mark.parametrize("cols", [70, 5000, 70000])
def test_softmax_special_rows(dg, cols):
    """NaN, +inf and all -inf rows: NaN throughout, as the order's steps give;
    neighbouring rows untouched."""
    import torch
    X = inputs.lognormal_f32(cols, (5, cols), sigma=1.0)
    X[1, cols - 2] = np.nan
    X[2, 3] = np.inf
    X[3, :] = -np.inf
    desc = dict(leaf_w=64, out="f32")
    Y = torch.zeros(X.shape, device="cuda")
    dg.dg_softmax(dg.Desc(**desc), dev_f32(X), Y)
    torch.cuda.synchronize()
    assert_bits_equal(host_bits(Y), oracle.softmax(desc, X), "cols %d" % cols)
    assert torch.isnan(Y[1:4]).all() and not torch.isnan(Y[0]).any() and not torch.isnan(Y[4]).any()


# both sides of each line at which row_fused_pays hands a call to the one-wave
# kernels: (operation, leaf order, rows, cols)
LINES = [("rmsnorm", 0, 256, 640), ("rmsnorm", 0, 257, 640), ("rmsnorm", 0, 2049, 640), ("rmsnorm", 0, 4, 2052),
         ("rmsnorm", 0, 5, 2052), ("rmsnorm", 0, 513, 2052), ("rmsnorm", 1, 2048, 65), ("rmsnorm", 2, 2049, 65),
         ("rmsnorm", 2, 4097, 513), ("layernorm", 1, 4096, 129), ("layernorm", 2, 4097, 129), ("softmax", 2, 2048, 129),
         ("softmax", 1, 2049, 129), ("rmsnorm", 3, 1, 16384), ("rmsnorm", 3, 2, 16384), ("rmsnorm", 3, 9, 8196),
         ("rmsnorm", 2, 3, 8196), ("rmsnorm", 2, 4, 8196), ("rmsnorm", 3, 257, 20000), ("rmsnorm", 2, 256, 20000),
         ("rmsnorm", 2, 257, 20000), ("rmsnorm", 3, 33, 65540), ("rmsnorm", 1, 257, 65540), ("rowsum", 3, 1, 20000),
         ("rowsum", 1, 2, 20000), ("rowsum", 1, 257, 16385), ("rowsum", 2, 513, 16388), ("layernorm", 3, 769, 16388)]


@pytest.mark.parametrize("op,oi,rows,cols", LINES)
def test_lines_between_row_kernels(dg, op, oi, rows, cols):
    import torch
    desc = dict(ORDERS[oi], out="f32", reduce="sumsq" if op == "rmsnorm" else "sum")
    X = inputs.lognormal_f32(rows + cols, (rows, cols), sigma=1.0)
    print("%s %s rows %d cols %d" % (op, desc, rows, cols), flush=True)
    d, dX = dg.Desc(**desc), dev_f32(X)
    got = torch.full((rows,) if op == "rowsum" else X.shape, float("nan"), device="cuda")
    if op == "rowsum":
        dg.dg_rowsum(d, dX, got)
        want = oracle.rowsum(desc, X)
    elif op == "rmsnorm":
        dg.dg_rmsnorm(d, dX, None, 1e-5, got)
        want = oracle.rmsnorm(desc, X, None, eps=1e-5)
    elif op == "layernorm":
        dg.dg_layernorm(d, dX, None, None, 1e-5, got)
        want = oracle.layernorm(desc, X, None, None, eps=1e-5)
    else:
        dg.dg_softmax(d, dX, got)
        want = oracle.softmax(desc, X)
    torch.cuda.synchronize()
    assert_bits_equal(host_bits(got), want, "%s %s %d x %d" % (op, desc, rows, cols))


@pytest.mark.parametrize("op,oi,rows,cols", [("rmsnorm", 2, 2100, 65), ("softmax", 2, 2100, 129), ("layernorm", 1, 4100, 129)])
def test_captured_normalisation_takes_no_workspace(dg, op, oi, rows, cols):
    """Calls that eagerly go through a workspace because that is faster: under
    capture they take the launch that needs none, on a stream that has none,
    and replay to the eager bits."""
    import ctypes

    import torch
    desc = dict(ORDERS[oi], out="f32", reduce="sumsq" if op == "rmsnorm" else "sum")
    X = dev_f32(inputs.lognormal_f32(rows + cols, (rows, cols), sigma=1.0))
    d, got, want = dg.Desc(**desc), torch.zeros((rows, cols), device="cuda"), torch.zeros((rows, cols), device="cuda")

    def call(Y):
        if op == "rmsnorm":
            dg.dg_rmsnorm(d, X, None, 1e-5, Y)
        elif op == "layernorm":
            dg.dg_layernorm(d, X, None, None, 1e-5, Y)
        else:
            dg.dg_softmax(d, X, Y)

    print(op, desc, rows, cols, flush=True)
    call(want)
    torch.cuda.synchronize()
    hip, raw = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(raw)) == 0
    free = torch.cuda.mem_get_info()[0]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.ExternalStream(raw.value)):
        call(got)
    for _ in range(3):
        got.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))
        call(want)
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20
    del g
    torch.cuda.synchronize()
    assert hip.hipStreamDestroy(raw) == 0
