"""GPU parity of the ring GEMM kernels at the edges of their blocks, slots and
parts: every block shape, operand type, K from one chunk to one slab more than the slots
hold and around it, parts shorter than a slab, tile chains and trees, aligned and odd, against the
generic kernel on every output and the CPU oracle on some rows, bit for bit."""
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


def device(bits, dtype, off):
    """A matrix of 16-bit patterns `off` elements into a buffer of NaN patterns."""
    import torch
    buf = torch.full((bits.size + off + 8,), -1, dtype=torch.int16, device="cuda")
    buf[off:off + bits.size] = torch.from_numpy(bits.reshape(-1).view(np.int16)).cuda()
    return buf[off:off + bits.size].view(dtype).view(bits.shape)


# 64 x 64 blocks, few rows over many columns, 64 x 128, 128 x 128 (a block,
# its edge, one row or chunk past it)
SIZES = [(33, 104), (64, 64), (65, 200), (128, 72), (3, 6408), (32, 5000), (1000, 1104), (961, 2056), (2000, 2056)]
DESCS = [dict(), dict(out="bf16", epilogue="bias_silu", epi_round="pre_act"), dict(in_dtype="f16", out="bf16", epilogue="bias"),
         dict(split_k=3, split_combine="tree", partial="bf16", out="bf16", epilogue="bias"), dict(split_k=2, in_dtype="f16"),
         dict(tail="first", tile_k=64), dict(tile_combine="tree", tile_k=32), dict(tile_combine="tree", tile_k=64, out="bf16",
         epilogue="bias_silu"), dict(tile_combine="seq", tile_k=96, in_dtype="f16"), dict(tile_combine="tree", tile_k=32,
         in_dtype="f16", split_k=2, split_combine="tree", partial="bf16"), dict(tile_combine="seq", tile_k=32, tail="first")]
KS = [8, 64, 72, 128, 192, 256, 320, 328, 384, 448, 520, 2080, 8192]


@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("di", range(len(DESCS)))
def test_ring(dg, di, size, odd):
    import torch
    desc = dict(tile_k=32)
    desc.update(DESCS[di])
    f16 = desc.get("in_dtype") == "f16"
    dt = torch.float16 if f16 else torch.bfloat16
    spread = inputs.spread_f16 if f16 else inputs.spread_bf16
    for K in KS if size[0] < 900 else KS[di % 3:-1:3]:
        M, N = size[0], size[1] - 3 * odd
        if desc.get("tail") != "first":
            K = K + 1 if odd else K
        elif K % 32:
            K = K // 32 * 32 + 32                 # a tile tree or chain starts on a 32-k step
        parts = desc.get("split_k", 1)
        if parts > 1 and (parts - 1) * (-(-K // (32 * parts)) * 32) >= K:
            continue                              # the cut plan would leave a part empty
        A, B = spread(di + 17 * M + K, (M, K)), spread(di + 17 * M + 1, (K, N))
        bias = inputs.normal_bf16(M + 2, (N,), 1.0) if "epilogue" in desc else None
        A[M // 2, 0] = 0x7FFF                     # a NaN row, an infinite one and a NaN column
        A[M // 3, K // 2] = 0x7C00 if f16 else 0x7F80
        B[K // 2, 5] = 0x7FFF
        print("size %s K %d odd %d desc %s" % ((M, N), K, odd, desc), flush=True)
        dA, dB = device(A, dt, odd), device(B, dt, odd)
        db = None if bias is None else device(bias, torch.bfloat16, odd)
        ct = torch.bfloat16 if desc.get("out") == "bf16" else torch.float32
        buf = torch.full((M * N + 16,), 7.0, dtype=ct, device="cuda")
        C, ref = buf[8 + odd:8 + odd + M * N].view(M, N), torch.empty((M, N), dtype=ct, device="cuda")
        d = dg.Desc(**desc)
        dg.dg_gemm(d, dA, dB, db, C)
        dg.dg_gemm(d, dA, dB, db, ref, knobs=dict(kernel=1))
        torch.cuda.synchronize()
        assert_bits_equal(host_bits(C), host_bits(ref), "M %d N %d K %d %s" % (M, N, K, desc))
        rows = np.unique([0, M // 3, M // 2, M - 1])
        assert_bits_equal(host_bits(C)[rows], oracle.gemm(desc, A[rows], B, bias), "M %d N %d K %d %s" % (M, N, K, desc))
        assert (buf[:8 + odd] == 7).all() and (buf[8 + odd + M * N:] == 7).all()   # nothing written outside


@pytest.mark.parametrize("size", [(33, 112), (64, 64), (65, 208), (3, 6416), (1000, 1104), (961, 2064), (2000, 2064)])
@pytest.mark.parametrize("desc", [dict(), dict(out="bf16", epilogue="bias_silu"), dict(split_k=3, split_combine="tree", out="bf16"),
                                  dict(tail="first", tile_k=64)])
def test_ring_e4m3(dg, desc, size):
    import torch
    desc = dict(dict(tile_k=32, mma="16x16x32_fp8", in_dtype="e4m3"), **desc)
    M, N = size
    for K in (16, 64, 128, 144, 512, 640, 656, 784, 1040):
        parts = desc.get("split_k", 1)
        if parts > 1 and (parts - 1) * (-(-K // (32 * parts)) * 32) >= K:
            continue
        rng = np.random.default_rng(M + N + K)
        A, B = (rng.integers(0, 256, n, dtype=np.uint8) & 0xF7 for n in ((M, K), (K, N)))   # every sign and exponent, no NaN
        A[M // 2, 0] = B[K // 2, 5] = 0x7F                                                 # a NaN row and column
        bias = inputs.normal_bf16(M + 2, (N,), 1.0) if "epilogue" in desc else None
        print("size %s K %d desc %s" % ((M, N), K, desc), flush=True)
        dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
        db = None if bias is None else device(bias, torch.bfloat16, 0)
        ct = torch.bfloat16 if desc.get("out") == "bf16" else torch.float32
        buf, ref = torch.full((M * N + 16,), 7.0, dtype=ct, device="cuda"), torch.empty((M, N), dtype=ct, device="cuda")
        C = buf[8:8 + M * N].view(M, N)
        d = dg.Desc(**desc)
        dg.dg_gemm(d, dA, dB, db, C)
        dg.dg_gemm(d, dA, dB, db, ref, knobs=dict(kernel=1))
        torch.cuda.synchronize()
        assert_bits_equal(host_bits(C), host_bits(ref), "M %d N %d K %d %s" % (M, N, K, desc))
        rows = np.unique([0, M // 3, M // 2, M - 1])
        assert_bits_equal(host_bits(C)[rows], oracle.gemm(desc, A[rows], B, bias), "M %d N %d K %d %s" % (M, N, K, desc))
        assert (buf[:8] == 7).all() and (buf[8 + M * N:] == 7).all()


@pytest.mark.parametrize("desc", [dict(), dict(out="bf16", epilogue="bias_silu"), dict(tile_combine="tree", tile_k=64),
                                  dict(tile_combine="seq", tile_k=64, epilogue="bias"), dict(tail="first", tile_combine="seq"),
                                  dict(in_dtype="e4m3", mma="16x16x32_fp8")])
def test_no_k(dg, desc):
    """K = 0: the epilogue of zero."""
    import torch
    desc = dict(dict(tile_k=32), **desc)
    for M, N in [(40, 64), (1000, 1104)]:
        print("K 0", (M, N), desc, flush=True)
        dt = torch.uint8 if desc.get("in_dtype") == "e4m3" else torch.bfloat16
        A, B = torch.empty((M, 0), dtype=dt, device="cuda"), torch.empty((0, N), dtype=dt, device="cuda")
        bias = device(inputs.normal_bf16(M, (N,), 1.0), torch.bfloat16, 0) if "epilogue" in desc else None
        ct = torch.bfloat16 if desc.get("out") == "bf16" else torch.float32
        C, ref = (torch.full((M, N), 7.0, dtype=ct, device="cuda") for _ in range(2))
        d = dg.Desc(**desc)
        dg.dg_gemm(d, A, B, bias, C)
        dg.dg_gemm(d, A, B, bias, ref, knobs=dict(kernel=1))
        torch.cuda.synchronize()
        assert_bits_equal(host_bits(C), host_bits(ref), "%s %s" % ((M, N), desc))


@pytest.mark.parametrize("size", [(1300, 6144, 320), (1001, 10656, 72), (2048, 4616, 264), (2300, 4101, 263), (1001, 10655, 201)])
@pytest.mark.parametrize("desc", [dict(out="bf16", epilogue="bias_silu"), dict()])
def test_third_round(dg, desc, size):
    """Sizes whose 128 x 128 blocks would take a third round of the chip: the
    256-row blocks, against the generic kernel's bits."""
    import torch
    M, N, K = size
    print("size", size, desc, flush=True)
    A, B = (device(inputs.normal_bf16(M + i, n, 1.0), torch.bfloat16, 0) for i, n in enumerate([(M, K), (K, N)]))
    bias = device(inputs.normal_bf16(N, (N,), 1.0), torch.bfloat16, 0) if "epilogue" in desc else None
    ct = torch.bfloat16 if desc.get("out") == "bf16" else torch.float32
    C, ref = (torch.full((M, N), 7.0, dtype=ct, device="cuda") for _ in range(2))
    d = dg.Desc(tile_k=64, **desc)
    dg.dg_gemm(d, A, B, bias, C)
    dg.dg_gemm(d, A, B, bias, ref, knobs=dict(kernel=1))
    torch.cuda.synchronize()
    assert_bits_equal(host_bits(C), host_bits(ref), "%s %s" % (size, desc))


# few rows over many columns, on both sides of each line between the ring, the
# few-row kernel's 16- and 64-column blocks and the 256-row blocks
FEW = [(1, 4224, 1024, 1), (16, 2176, 2048, 2), (17, 2176, 2048, 2), (1, 32768, 128, 1), (16, 33280, 128, 1), (17, 33280, 128, 1),
       (3, 16640, 512, 2), (16, 49152, 72, 1), (64, 49152, 72, 1), (65, 49152, 72, 1), (64, 49153, 65, 1), (64, 128257, 33, 1),
       (32, 128257, 33, 1), (33, 512, 8192, 1), (64, 512, 8184, 1), (65, 512, 8192, 1), (128, 4096, 4096, 1)]


@pytest.mark.parametrize("M,N,K,S", FEW)
def test_few_rows(dg, M, N, K, S):
    import torch
    desc = dict(tile_k=32, split_k=S, split_combine="tree", out="bf16", epilogue="bias")
    A, B = inputs.spread_bf16(N + M, (M, K)), inputs.spread_bf16(N, (K, N))
    bias = inputs.normal_bf16(K, (N,), 1.0)
    odd = (N % 8 or K % 8) != 0
    a, b, z = device(A, torch.bfloat16, odd), device(B, torch.bfloat16, odd), device(bias, torch.bfloat16, odd)
    print("M %d N %d K %d S %d" % (M, N, K, S), flush=True)
    C = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    dg.dg_gemm(dg.Desc(**desc), a, b, z, C[0])
    dg.dg_gemm(dg.Desc(**desc), a, b, z, C[1], knobs=dict(kernel=1))
    torch.cuda.synchronize()
    assert torch.equal(C[0].view(torch.int16), C[1].view(torch.int16))
    cols = np.r_[0:64, N // 2:N // 2 + 64, N - 64:N]
    assert_bits_equal(host_bits(C[0])[:, cols], oracle.gemm(desc, A, np.ascontiguousarray(B[:, cols]), bias[cols]),
                      "columns of %s" % ((M, N, K, S),))


# trees of nine to sixteen tiles, on both sides of the line between the ring and
# the tile-combine kernel (rounds of the chip that each would take)
TREES = [(400, 5696, 512, 32), (1000, 5696, 512, 32), (64, 5696, 512, 32), (2048, 2056, 288, 32), (400, 5696, 576, 64),
         (1000, 5696, 1024, 64), (400, 5696, 2304, 256), (1280, 5696, 576, 64), (1280, 8192, 576, 64),
         (2000, 4096, 576, 64), (2000, 4096, 2304, 256), (6100, 2048, 576, 64), (1792, 8192, 576, 64)]


@pytest.mark.parametrize("M,N,K,tile_k", TREES)
def test_tree_of_nine_to_sixteen(dg, M, N, K, tile_k):
    import torch
    desc = dict(tile_k=tile_k, tile_combine="tree", out="bf16", epilogue="bias")
    A, B = inputs.spread_bf16(N + M, (M, K)), inputs.spread_bf16(N, (K, N))
    bias = inputs.normal_bf16(K, (N,), 1.0)
    a, b, z = device(A, torch.bfloat16, 0), device(B, torch.bfloat16, 0), device(bias, torch.bfloat16, 0)
    print("M %d N %d K %d tile_k %d" % (M, N, K, tile_k), flush=True)
    C = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    dg.dg_gemm(dg.Desc(**desc), a, b, z, C[0])
    dg.dg_gemm(dg.Desc(**desc), a, b, z, C[1], knobs=dict(kernel=1))
    torch.cuda.synchronize()
    assert torch.equal(C[0].view(torch.int16), C[1].view(torch.int16))
    rows = np.array([0, M // 2, M - 1])
    assert_bits_equal(host_bits(C[0])[rows], oracle.gemm(desc, A[rows], B, bias), "rows of %s" % ((M, N, K, tile_k),))
