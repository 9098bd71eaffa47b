"""GPU parity of the attention kernels on transposed score tiles (tree row
sums accumulated in place) against the CPU oracle, bit for bit: 32-row waves
(heads enough to fill the chip; the first heads compared), 16-row waves, their
row and key edges, and scores that are -inf or NaN."""
import numpy as np
import pytest

import oracle
from paper_2609_11356_amd import inputs
from tests.gpu_util import assert_bits_equal
from tests.test_gpu_attention import qkv, run, scale

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_11356_amd import dg as _dg
    _dg.lib()
    return _dg


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("w", [32, 64, 128])
@pytest.mark.parametrize("shape", [(260, 128, 128, 128), (128, 257, 257, 128), (64, 513, 513, 256), (1024, 1, 97, 0),
                                   (512, 33, 193, 0), (3, 47, 129, 0), (2, 191, 191, 32), (2, 130, 130, 64)])
def test_tiles(dg, d, w, shape):
    H, Lq, Lk, q_block = shape
    desc = dict(key_block=w, causal=int(q_block > 0), q_block=q_block or 1, block_sum="tree", pv_fma=1,
                l_fma=(w // 32) % 2, final="recip" if d == 64 else "div", out="bf16" if w == 64 else "f32")
    Q, K, V = qkv(w + Lq, H, Lq, Lk, d, spread_v=w == 32)
    print("attention", desc, shape, d, flush=True)
    got = run(dg, desc, Q, K, V, scale(d))
    n = 2
    assert_bits_equal(got[:n], oracle.attention(desc, Q[:n], K[:n], V[:n], scale(d)), "%s %s d %d" % (desc, shape, d))
    # heads are independent: the last one again, alone in a call (16-row waves)
    assert np.array_equal(run(dg, desc, Q[-1:], K[-1:], V[-1:], scale(d))[0], got[-1])


@pytest.mark.parametrize("H,causal", [(4, 0), (4, 1), (600, 0), (600, 1)])
def test_tiles_special_scores(dg, H, causal):
    """Keys whose scores overflow to -inf (probability zero), a row of -inf
    only, NaN scores, and infinities in V under a zero probability: the
    oracle's steps, NaN as a class."""
    d, L = 64, 70
    Q, K, V = qkv(5, H, L, L, d)
    Q[:, :, 0] = 0x7F00                   # 1.7e38
    K[:, :, 0] = 0x0000
    K[:, 3, 0] = 0xC000                   # score -inf for every query
    K[0, :, 0] = 0xC000                   # head 0: every score -inf
    K[1, 9, 1] = 0x7FC0                   # head 1: one NaN key
    V[2, 3, 5] = 0x7F80                   # head 2: inf where the probability is 0
    desc = dict(key_block=32, causal=causal, q_block=64, block_sum="tree", out="f32")
    got = run(dg, desc, Q, K, V, scale(d))
    assert_bits_equal(got[:4], oracle.attention(desc, Q[:4], K[:4], V[:4], scale(d)), "special scores, %d heads" % H)
    assert np.isnan(got[0]).all() and np.isfinite(got[3]).all()


# few rows over many keys (the split path): one and several 16-row tiles, odd
# and short last blocks, the ring's remainders, causal walks cut at 16 .. 128
SPLIT = [(1, 1, 769, 0), (3, 17, 1100, 0), (2, 5, 1024 + 31, 0), (1, 33, 2049, 0), (1, 1030, 1030, 16), (1, 1025, 1025, 128),
         (2, 800, 800, 64)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("w", [32, 64, 128])
@pytest.mark.parametrize("shape", SPLIT)
def test_split(dg, d, w, shape):
    H, Lq, Lk, q_block = shape
    desc = dict(key_block=w, causal=int(q_block > 0), q_block=q_block or 1, block_sum="tree", pv_fma=1,
                l_fma=(w // 32) % 2, final="recip" if d == 64 else "div", out="bf16" if w == 64 else "f32")
    Q, K, V = qkv(w + Lq, H, Lq, Lk, d, spread_v=w == 32)
    print("attention", desc, shape, d, flush=True)
    got = run(dg, desc, Q, K, V, scale(d))
    if Lq <= 64:
        assert_bits_equal(got, oracle.attention(desc, Q, K, V, scale(d)), "%s %s d %d" % (desc, shape, d))
        return
    ii = np.unique(np.concatenate([np.arange(0, Lq, 37), [0, 1, 15, 16, Lq // 2, Lq - 2, Lq - 1]]))
    want = oracle.attention_rows(desc, Q, K, V, scale(d), np.zeros(len(ii), dtype=np.int64), ii)
    rows = got[0][ii]
    rows = (rows.astype(np.uint32) << 16).view(np.float32) if rows.dtype == np.uint16 else rows
    assert_bits_equal(rows, want, "%s %s d %d" % (desc, shape, d))


def test_split_special_scores(dg):
    """-inf and NaN scores, an all -inf row, infinities in V at probability
    zero and in the block cut short by the causal split."""
    d, L = 64, 1100
    Q, K, V = qkv(9, 4, 3, L, d)
    Q[:, :, 0] = 0x7F00
    K[:, :, 0] = 0x0000
    K[:, 3, 0] = 0xC000
    K[0, :, 0] = 0xC000
    K[1, 900, 1] = 0x7FC0
    V[2, 3, 5] = 0x7F80
    desc = dict(key_block=64, block_sum="tree", out="f32")
    assert_bits_equal(run(dg, desc, Q, K, V, scale(d)), oracle.attention(desc, Q, K, V, scale(d)), "special scores")
    # causal: stage 1 of rows 48 .. 63 ends at key 48, inside a 64-key block
    # whose later V rows are infinite and must not be read into its products
    Q, K, V = qkv(11, 1, 1100, 1100, d)
    V[0, 48:, 7] = 0x7F80
    desc = dict(key_block=64, causal=1, q_block=48, block_sum="tree", out="f32")
    ii = np.array([0, 16, 33, 47])
    got = run(dg, desc, Q, K, V, scale(d))
    assert_bits_equal(got[0][ii], oracle.attention_rows(desc, Q, K, V, scale(d), np.zeros(4, dtype=np.int64), ii), "cut stage")


def test_few_rows_under_capture(dg):
    """A captured call takes no workspace and replays to the eager bits."""
    import torch
    from tests.gpu_util import dev_bf16
    Q, K, V = (dev_bf16(x) for x in qkv(3, 2, 4, 1500, 128))
    desc = dg.AttnDesc(key_block=64)
    want = torch.empty(Q.shape, dtype=torch.bfloat16, device="cuda")
    dg.dg_attention(desc, Q, K, V, want, scale(128))
    got = torch.zeros_like(want)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dg.dg_attention(desc, Q, K, V, got, scale(128))
    for _ in range(3):
        got.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
        dg.dg_attention(desc, Q, K, V, want, scale(128))
        torch.cuda.synchronize()


def test_attention_leaves_a_captured_workspace(dg):
    """Attention on a stream does not touch the workspace that a captured
    split-K product of the same stream holds: the graph replays to the eager
    bits after an attention call that needs far more."""
    import torch
    from tests.gpu_util import dev_bf16
    stream = torch.cuda.Stream()
    A, B = dev_bf16(inputs.normal_bf16(1, (16, 512))), dev_bf16(inputs.normal_bf16(2, (512, 256)))
    Q, K, V = (dev_bf16(x) for x in qkv(5, 16, 4, 2048, 128))
    O = torch.empty(Q.shape, dtype=torch.bfloat16, device="cuda")
    gemm, attn = dg.Desc(tile_k=64, split_k=4, split_combine="tree"), dg.AttnDesc(key_block=64)
    want, got = torch.empty((16, 256), device="cuda"), torch.empty((16, 256), device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        dg.dg_gemm(gemm, A, B, None, want)       # the workspace is there before the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        dg.dg_gemm(gemm, A, B, None, got)
    for n in range(3):
        with torch.cuda.stream(stream):
            dg.dg_attention(attn, Q, K, V, O, scale(128))
        torch.cuda.synchronize()
        keep = torch.full((1 << 20,), 3.0, device="cuda")    # memory that the replay must not write
        got.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want) and (keep == 3.0).all()


def test_two_threads_on_the_per_thread_stream(dg):
    """hipStreamPerThread is one handle for two queues: calls of two host
    threads on it share no workspace (attention's records, split-K partials)."""
    import threading

    import torch
    from tests.gpu_util import dev_bf16
    PER_THREAD = 2                       # hipStreamPerThread
    attn, gemm = dg.AttnDesc(key_block=64), dg.Desc(tile_k=64, split_k=4, split_combine="tree")
    work = []
    for t in range(2):
        Q, K, V = (dev_bf16(x) for x in qkv(40 + t, 4, 1, 3001, 128))
        A, B = dev_bf16(inputs.normal_bf16(50 + t, (8, 1024))), dev_bf16(inputs.normal_bf16(60 + t, (1024, 512)))
        wants = torch.empty(Q.shape, dtype=torch.bfloat16, device="cuda"), torch.empty((8, 512), device="cuda")
        dg.dg_attention(attn, Q, K, V, wants[0], scale(128))
        dg.dg_gemm(gemm, A, B, None, wants[1])
        outs = [(torch.zeros_like(wants[0]), torch.zeros_like(wants[1])) for _ in range(100)]
        work.append((Q, K, V, A, B, wants, outs))
    torch.cuda.synchronize()
    start, failed = threading.Barrier(2), []

    def body(w):
        Q, K, V, A, B, _, outs = w
        try:
            start.wait(timeout=60)
            for o, c in outs:
                dg.dg_attention(attn, Q, K, V, o, scale(128), stream=PER_THREAD)
                dg.dg_gemm(gemm, A, B, None, c, stream=PER_THREAD)
            torch.cuda.synchronize()
        except BaseException as e:
            failed.append(e)

    threads = [threading.Thread(target=body, args=(w,)) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not failed and not any(t.is_alive() for t in threads), failed
    torch.cuda.synchronize()
    for _, _, _, _, _, wants, outs in work:
        for o, c in outs:
            assert torch.equal(o.view(torch.int16), wants[0].view(torch.int16)) and torch.equal(c, wants[1])


@pytest.mark.parametrize("d,H,Lq,Lk,q_block", [
    # keys in blocks of 128: one block in 128-row workgroups; more of them, the
    # last half empty; 64-row workgroups in one round, two and more, few and long keys
    (128, 256, 128, 128, 0), (128, 256, 128, 129, 0), (128, 256, 129, 512, 0), (128, 256, 129, 513, 0),
    (128, 128, 416, 416, 128), (128, 128, 417, 417, 128), (128, 256, 64, 70, 0), (128, 257, 64, 319, 0),
    (128, 257, 64, 320, 0), (128, 128, 191, 191, 64), (128, 128, 192, 192, 64), (128, 513, 33, 1024, 0),
    (128, 513, 33, 1025, 0), (128, 171, 190, 190, 64), (64, 512, 64, 130, 0), (64, 512, 65, 130, 0)])
def test_keys_in_blocks_of_128(dg, d, H, Lq, Lk, q_block):
    desc = dict(key_block=128, causal=int(q_block > 0), q_block=q_block or 1, block_sum="tree", pv_fma=1, out="f32")
    Q, K, V = qkv(Lq + Lk, H, Lq, Lk, d)
    print("attention", H, Lq, Lk, d, q_block, flush=True)
    got = run(dg, desc, Q, K, V, scale(d))
    assert_bits_equal(got[:1], oracle.attention(desc, Q[:1], K[:1], V[:1], scale(d)), "%s %s" % (desc, (H, Lq, Lk, d)))
    # heads are independent: the last one again, alone in a call
    assert np.array_equal(run(dg, desc, Q[-1:], K[-1:], V[-1:], scale(d))[0], got[-1])
