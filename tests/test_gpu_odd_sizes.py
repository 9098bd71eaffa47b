"""GPU parity of the GEMM on sizes, part starts and pointers off the
8-element grid, against the CPU oracle, bit for bit.  The operands lie one
element into buffers full of NaN, and single rows and columns of them hold
NaN and infinities: a chunk that takes in a neighbour's elements, or elements
past a matrix, shows up as NaN where the oracle has none."""
import numpy as np
import pytest

import oracle
from paper_2609_11356_amd import inputs
from tests.gpu_util import assert_bits_equal, host_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_11356_amd import dg as _dg
    _dg.lib()
    return _dg


def inside(bits, dtype):
    """A matrix of 16-bit patterns one element into a buffer of NaN patterns."""
    import torch
    buf = torch.full((bits.size + 9,), -1, dtype=torch.int16, device="cuda")
    buf[1:1 + bits.size] = torch.from_numpy(bits.reshape(-1).view(np.int16)).cuda()
    return buf[1:1 + bits.size].view(dtype).view(bits.shape)


CARRY = [dict(), dict(out="bf16", epilogue="bias"), dict(out="bf16", epilogue="bias_silu", epi_round="pre_act"),
         dict(in_dtype="f16", out="bf16"), dict(split_k=3, split_combine="tree", partial="bf16", out="bf16", epilogue="bias"),
         dict(split_k=4, k_cuts=[3, 77, 200], epilogue="bias_silu"), dict(tail="first", tile_k=64)]
GEN = [dict(tile_k=32, tile_combine="tree"), dict(tile_k=64, tile_combine="seq", out="bf16", epilogue="bias"),
       dict(tile_k=64, fma=0), dict(tile_k=32, tile_combine="tree", in_dtype="f16", split_k=2, split_combine="tree"),
       dict(tile_k=96, tile_combine="seq", fma=0)]
# the few-row shapes, the 64-row tiles, their edges and remainders, the
# smallest sizes, N and K of every residue class the chunks care about
SHAPES = [(1, 9, 233), (16, 15, 255), (17, 33, 249), (33, 65, 511), (65, 127, 257), (129, 131, 513), (130, 8, 250),
          (200, 257, 8 * 32 + 1), (64, 300, 1037)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("di", range(len(CARRY) + len(GEN)))
def test_odd_sizes(dg, di, shape):
    import torch
    desc = dict(tile_k=32, **(CARRY + GEN)[di]) if di < len(CARRY) and "tile_k" not in CARRY[di] else dict((CARRY + GEN)[di])
    M, N, K = shape
    if desc.get("tail") == "first":
        K = K // 64 * 64 + 40          # a short first tile of whole chunks
    f16 = desc.get("in_dtype") == "f16"
    spread = inputs.spread_f16 if f16 else inputs.spread_bf16
    A, B = spread(di + 17 * M, (M, K)), spread(di + 17 * M + 1, (K, N))
    bias = inputs.normal_bf16(M + 2, (N,), 1.0) if "epilogue" in desc else None
    if M > 4:
        A[M // 2, 0] = 0x7FFF          # NaN at the start of a row: the row before must not see it
        A[M // 3, 0] = 0x7C00 if f16 else 0x7F80
    if N > 16:
        B[K // 2, 0] = 0x7FFF          # and of a column-run
    print("shape %s desc %s" % ((M, N, K), desc), flush=True)
    dt = torch.float16 if f16 else torch.bfloat16
    C = torch.full((M * N + 2,), float("nan"), dtype=torch.bfloat16 if desc.get("out") == "bf16" else torch.float32,
                   device="cuda")
    Cv = C[1:1 + M * N].view(M, N)
    dg.dg_gemm(dg.Desc(**desc), inside(A, dt), inside(B, dt), None if bias is None else inside(bias, torch.bfloat16), Cv)
    torch.cuda.synchronize()
    assert_bits_equal(host_bits(Cv), oracle.gemm(desc, A, B, bias), "%s %s" % (shape, desc))
    assert torch.isnan(C[0]) and torch.isnan(C[-1])          # nothing written outside


@pytest.mark.parametrize("shape", [(1030, 1537, 77), (2049, 4097, 33), (3000, 4099, 40)])
def test_odd_sizes_wide(dg, shape):
    """The ping-pong kernel's 256 x 256 blocks at odd sizes, column sums of the
    output included, and (1030 x 1537) the ring beside its own column-sum launch."""
    import torch
    M, N, K = shape
    A, B = inputs.spread_bf16(M, (M, K)), inputs.spread_bf16(N, (K, N))
    bias = inputs.normal_bf16(3, (N,), 1.0)
    desc = dict(tile_k=32, epilogue="bias")
    dA, dB, db = inside(A, torch.bfloat16), inside(B, torch.bfloat16), inside(bias, torch.bfloat16)
    print("shape %s" % (shape,), flush=True)
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    s = torch.empty((N,), dtype=torch.float32, device="cuda")
    d = dg.Desc(**desc)
    dg.dg_gemm_colsum(d, dA, dB, db, C, s)
    C2 = torch.empty_like(C)
    dg.dg_gemm(d, dA, dB, db, C2, knobs=dict(kernel=1))      # the generic kernel: every output
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int32), C2.view(torch.int32))
    rows = np.array([0, 1, M // 2, M - 2, M - 1])
    assert_bits_equal(host_bits(C)[rows], oracle.gemm(desc, A[rows], B, bias), "rows of %s" % (shape,))
    assert_bits_equal(host_bits(s), oracle.colsum(host_bits(C)), "column sums of %s" % (shape,))


# parts of one slab: both sides of the line between the generic kernel and the
# tiled ones, and every block shape of the latter with a single slab
SHORT = [(25, 333, 20), (40, 333, 71), (64, 2999, 45), (91, 3001, 45), (500, 1021, 9), (500, 1021, 61), (700, 2999, 63),
         (1500, 3001, 64)]


@pytest.mark.parametrize("shape", SHORT)
@pytest.mark.parametrize("di", range(5))
def test_odd_short_parts(dg, di, shape):
    import torch
    desc = [dict(tile_k=32, out="bf16", epilogue="bias"), dict(tile_k=32, tile_combine="tree"),
            dict(tile_k=64, tile_combine="seq", in_dtype="f16"), dict(tile_k=32, fma=0),
            dict(tile_k=32, split_k=2, split_combine="tree")][di]
    M, N, K = shape
    if desc.get("split_k") and K <= 32:
        K += 32
    f16 = desc.get("in_dtype") == "f16"
    dt = torch.float16 if f16 else torch.bfloat16
    spread = inputs.spread_f16 if f16 else inputs.spread_bf16
    A, B = spread(di + M, (M, K)), spread(di + N, (K, N))
    bias = inputs.normal_bf16(M + 2, (N,), 1.0) if "epilogue" in desc else None
    print("shape %s desc %s" % ((M, N, K), desc), flush=True)
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16 if desc.get("out") == "bf16" else torch.float32, device="cuda")
    dg.dg_gemm(dg.Desc(**desc), inside(A, dt), inside(B, dt), None if bias is None else inside(bias, torch.bfloat16), C)
    torch.cuda.synchronize()
    rows = np.unique(np.r_[0:min(M, 70), M // 2, M - 66 if M > 66 else 0:M])
    assert_bits_equal(host_bits(C)[rows], oracle.gemm(desc, np.ascontiguousarray(A[rows]), B, bias), "%s %s" % (shape, desc))


@pytest.mark.parametrize("M,dtype", [(1, "bf16"), (33, "f16"), (130, "bf16")])
def test_odd_past_31_bits(dg, M, dtype):
    """A weight so wide that 66 of its rows pass 31-bit offsets: the few-row and
    transposing-read kernels with chunks loaded where they lie, against the
    generic kernel on every output and the oracle on the first and last columns."""
    import torch
    K, N = 9, 16268817
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device="cuda").manual_seed(M)

    def operand(rows, cols):
        buf = torch.full((rows * cols + 9,), float("nan"), dtype=dt, device="cuda")
        buf[1:1 + rows * cols] = torch.randn(rows * cols, generator=g, device="cuda", dtype=torch.float32).to(dt)
        return buf[1:1 + rows * cols].view(rows, cols)

    print("M %d %s" % (M, dtype), flush=True)
    A, B, bias = operand(M, K), operand(K, N), torch.randn(N, generator=g, device="cuda").to(torch.bfloat16)
    desc = dict(tile_k=32, in_dtype=dtype, out="bf16", epilogue="bias")
    C = [torch.zeros((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    dg.dg_gemm(dg.Desc(**desc), A, B, bias, C[0])
    dg.dg_gemm(dg.Desc(**desc), A, B, bias, C[1], knobs=dict(kernel=1))
    torch.cuda.synchronize()
    assert torch.equal(C[0].view(torch.int16), C[1].view(torch.int16))
    for cols in (slice(0, 128), slice(N - 77, N)):
        a, b, z, c = (x.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
                      for x in (A, B[:, cols], bias[cols], C[0][:, cols]))
        assert_bits_equal(c, oracle.gemm(desc, a, b, z), "M %d columns %s" % (M, cols))
