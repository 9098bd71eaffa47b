"""GPU parity of the packed kernel where its parts meet inside one workgroup
(two to eight parts, both merge orders and roundings), and where A's rows lie
at any 2-byte address with NaN past K and past the matrix, against the CPU
oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2609_11356_amd import inputs
from tests.gpu_util import assert_bits_equal, dev_bf16, dev_f16, host_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_11356_amd import dg as _dg
    _dg.lib()
    return _dg


def run(dg, desc, A, B, bias, off):
    """The packed product with A `off` elements into a buffer of NaN patterns."""
    import torch
    kind = desc.get("in_dtype", "bf16")
    buf = np.full(A.size + off + 8, 0xFFFF, np.uint16)
    buf[off:off + A.size] = A.reshape(-1)
    dA = (dev_f16 if kind == "f16" else dev_bf16)(buf)[off:off + A.size].view(A.shape)
    if kind == "bf16_e4m3":
        Bp = dg.dg_pack_b(torch.from_numpy(np.ascontiguousarray(B)).cuda())
    else:
        Bp = dg.dg_pack_b((dev_f16 if kind == "f16" else dev_bf16)(B))
    C = torch.full((A.shape[0], B.shape[1]), 7.0, device="cuda",
                   dtype=torch.bfloat16 if desc.get("out") == "bf16" else torch.float32)
    dg.dg_gemm_packed(dg.Desc(**desc), dA, Bp, None if bias is None else dev_bf16(bias), C)
    torch.cuda.synchronize()
    return host_bits(C)


@pytest.mark.parametrize("kind", ["bf16", "f16", "bf16_e4m3"])
@pytest.mark.parametrize("S", [1, 2, 3, 5, 7, 8, 9])
@pytest.mark.parametrize("off", [0, 1, 3])
def test_parts_and_addresses(dg, kind, S, off):
    rng = np.random.default_rng(S + off)
    forms = [dict(split_combine="tree"), dict(split_combine="seq", out="bf16", epilogue="bias_silu"),
             dict(split_combine="tree", partial="bf16", merge="bf16", out="bf16", epilogue="bias")]
    # rows of 1 to 4 tiles, panel edges, K on and off the 32- and 64-k runs and
    # cut inside the first and the second block of a run; 3000 k on 3 panels: apart
    for n, (M, N, K) in enumerate([(1, 33, 64 * S + 9), (16, 16, 64 * S + 33), (17, 47, 64 * S), (40, 17, 64 * S + 63),
                                   (64, 40, 64 * S + 32), (5, 48, 3001)]):
        desc = dict(dict(tile_k=64, split_k=S, in_dtype=kind), **forms[n % 3])
        if (S - 1) * (-(-K // (64 * S)) * 64) >= K:
            K = 64 * S - 31
        A = (inputs.spread_f16 if kind == "f16" else inputs.spread_bf16)(n + K, (M, K))
        if kind == "bf16_e4m3":
            B = rng.integers(0, 256, (K, N), dtype=np.uint8) & 0xF7
        else:
            B = (inputs.spread_f16 if kind == "f16" else inputs.spread_bf16)(n + N, (K, N))
        A[M // 2, 0] = 0x7FFF           # the row before must not see it
        bias = inputs.normal_bf16(n, (N,)) if "epilogue" in desc else None
        print("packed", desc, (M, N, K), off, flush=True)
        assert_bits_equal(run(dg, desc, A, B, bias, off), oracle.gemm(desc, A, B, bias), "%s %s" % (desc, (M, N, K)))


@pytest.mark.parametrize("kind", ["bf16", "bf16_e4m3"])
@pytest.mark.parametrize("shape", [(48, 4112, 512, 2), (48, 4112, 4096, 2), (64, 1024, 512, 4), (64, 1024, 2048, 4),
                                   (16, 512, 8192, 8), (16, 512, 2048, 8), (9, 8192, 1024, 3), (17, 5760, 6144, 8)])
def test_merged_and_apart(dg, kind, shape):
    """Both sides of the line between parts that meet in the kernel and parts
    that a second launch merges, against the row-major product."""
    import torch
    M, N, K, S = shape
    desc = dict(tile_k=64, split_k=S, split_combine="tree", in_dtype=kind, out="bf16", epilogue="bias")
    rng = np.random.default_rng(K)
    A = inputs.spread_bf16(M, (M, K))
    B = rng.integers(0, 256, (K, N), dtype=np.uint8) & 0xF7 if kind == "bf16_e4m3" else inputs.spread_bf16(N, (K, N))
    bias = inputs.normal_bf16(N, (N,))
    print("packed", desc, shape, flush=True)
    got = run(dg, desc, A, B, bias, 0)
    dB = torch.from_numpy(np.ascontiguousarray(B)).cuda() if kind == "bf16_e4m3" else dev_bf16(B)
    C = torch.full((M, N), 7.0, device="cuda", dtype=torch.bfloat16)
    dg.dg_gemm(dg.Desc(**desc), dev_bf16(A), dB, dev_bf16(bias), C)
    torch.cuda.synchronize()
    assert_bits_equal(got, host_bits(C), "%s %s" % (desc, shape))


@pytest.mark.parametrize("M,K,off", [(9, 119304647, 7), (11, 97612893, 7), (9, 119304647, 1)])
def test_a_at_two_gib(dg, M, K, off):
    """A of 2 GiB less a few bytes, off 16 bytes: the offsets of its last
    elements pass 2^31.  Zeros but for the first and last k, small integers
    there, so that every sum is exact whatever its order."""
    import torch
    N, S, n = 16, 64, 48
    desc = dict(tile_k=64, split_k=S, split_combine="tree", in_dtype="bf16_e4m3", out="f32")
    rng = np.random.default_rng(M + off)
    head, tail = (rng.integers(-3, 4, (M, n)).astype(np.float32) for _ in range(2))
    bh, bt = (rng.integers(-3, 4, (n, N)).astype(np.float32) for _ in range(2))
    print("M %d K %d off %d" % (M, K, off), flush=True)
    buf = torch.zeros(M * K + off + 9, dtype=torch.bfloat16, device="cuda")
    buf[:off] = float("nan")
    buf[off + M * K:] = float("nan")
    A = buf[off:off + M * K].view(M, K)
    assert A.data_ptr() % 16 == 2 * off
    A[:, :n], A[:, K - n:] = torch.from_numpy(head).cuda(), torch.from_numpy(tail).cuda()
    B = torch.zeros((K, N), dtype=torch.float8_e4m3fn, device="cuda")
    B[:n], B[K - n:] = (torch.from_numpy(x).cuda().to(torch.float8_e4m3fn) for x in (bh, bt))
    Bp = dg.dg_pack_b(B)
    del B
    C = torch.full((M, N), 7.0, device="cuda")
    dg.dg_gemm_packed(dg.Desc(**desc), A, Bp, None, C)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), head @ bh + tail @ bt)


def test_merged_takes_no_workspace(dg):
    """Parts that meet in the kernel leave no partials: on a stream of its own,
    whose workspace would have to grow by S M N 4 bytes, no device memory goes."""
    import ctypes

    import torch
    M, N, K, S = 64, 65536, 512, 8
    A = torch.ones((M, K), dtype=torch.bfloat16, device="cuda")
    Bp = dg.dg_pack_b(torch.ones((K, N), dtype=torch.bfloat16, device="cuda"))
    C = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    hip = ctypes.CDLL("libamdhip64.so")
    stream = ctypes.c_void_p()
    torch.cuda.synchronize()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    free = torch.cuda.mem_get_info()[0]
    dg.dg_gemm_packed(dg.Desc(tile_k=64, split_k=S, split_combine="tree", out="bf16"), A, Bp, None, C, stream=stream.value)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < S * M * N * 4 // 2
    assert hip.hipStreamDestroy(stream) == 0
    assert (C == K).all()
