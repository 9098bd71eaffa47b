"""The work whose speed is measured: what programs built on this library call.

Every case goes through the public Python entry points on tensors that the
program already holds.  The listed cases cover the matrix products (the
smallest descriptor, one row, a batch of rows, an odd-sized product, the fused
MLP projection, split-K decode on a packed weight, e4m3 operands), attention
(prefill and one-token decode) and the row reductions with the normalisations
on them; `draw` spreads over the sizes, operand types, splits and layouts
around them.  The descriptor fixes every bit of a result, so outputs are
compared exactly.
"""
import math

import torch

from paper_2609_11356_amd import dg

MAX_FLOPS = 2.0 * 2048 * 14336 * 4096     # the fused MLP projection
MAX_ELEMS = 16384 * 8192                  # the largest row reduction


def _gemm(name=None, M=0, N=0, K=0, in_dtype="bf16", out="bf16", epilogue="none", split_k=1, split_combine="tree",
          tile_k=64, tile_combine="carry", packed=False):
    c = dict(kind="gemm", M=M, N=N, K=K, in_dtype=in_dtype, out=out, epilogue=epilogue, split_k=split_k,
             split_combine=split_combine, tile_k=tile_k, tile_combine=tile_combine, packed=packed)
    if name:
        c["name"] = name
    return c


def _attn(name=None, H=32, Lq=0, Lk=0, dim=128, causal=0, key_block=64, q_block=128, block_sum="tree", out="bf16"):
    c = dict(kind="attention", H=H, Lq=Lq, Lk=Lk, dim=dim, causal=causal, key_block=key_block, q_block=q_block,
             block_sum=block_sum, out=out)
    if name:
        c["name"] = name
    return c


def _rows(name=None, op="rowsum", rows=0, cols=0, leaf_w=64, leaf_layout="contiguous", lane_fold="up", out="bf16"):
    c = dict(kind="rows", op=op, rows=rows, cols=cols, leaf_w=leaf_w, leaf_layout=leaf_layout, lane_fold=lane_fold,
             out=out)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: launches and the host path (the smoke check's descriptor)
        _gemm("tiny_split_tree", 16, 64, 256, out="f32", split_k=2, tile_k=32, tile_combine="tree"),
        # batch 1 against a row-major weight
        _gemm("gemv_row_major", 1, 4096, 4096),
        # eight decoding rows against a long-K weight packed at load time, parts merged by the tree
        _gemm("decode_packed_split", 8, 4096, 14336, split_k=8, packed=True),
        # a batch of prompts through a square projection
        _gemm("prefill_1024", 1024, 4096, 4096),
        # a product whose sizes are no multiple of anything (an odd vocabulary, a cut projection)
        _gemm("odd_sizes_bias", 515, 3001, 2047, epilogue="bias"),
        # the fused MLP projection of a training or prefill batch
        _gemm("mlp_bias_silu", 2048, 14336, 4096, epilogue="bias_silu"),
        # the same projection with both operands quantised to e4m3
        _gemm("mlp_e4m3", 2048, 14336, 4096, in_dtype="e4m3", tile_k=128),
        # causal prefill of one long prompt
        _attn("attention_prefill_causal", 32, 4096, 4096, causal=1),
        # one new token against a cache of odd length
        _attn("attention_decode_token", 32, 1, 4001),
        # the pinned row reduction at the benchmark's size
        _rows("rowsum_sum", "rowsum", 16384, 8192, out="f32"),
        # normalising the hidden states of a batch of tokens, the pinned count-up order
        _rows("layernorm_hidden", "layernorm", 4096, 4096),
        # probabilities over a vocabulary for a batch of tokens
        _rows("softmax_vocabulary", "softmax", 64, 100000),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _parts_ok(K, split_k, tile_k):
    """Whether the default cut plan (equal spans of whole tiles) leaves no part empty."""
    span = -(-(-(-K // split_k)) // tile_k) * tile_k
    return split_k == 1 or (split_k - 1) * span < K


def _draw_gemm(rng):
    M, N, K = _log(rng, 1, 2048), _log(rng, 64, 14336), _log(rng, 64, 14336)
    if rng.random() < 0.6:                      # model widths; else odd sizes
        N, K = -(-N // 64) * 64, -(-K // 64) * 64
    while 2.0 * M * N * K > MAX_FLOPS:
        M = -(-M // 2)
    split_k = rng.choice([1, 1, 1, 1, 2, 4, 8]) if M <= 256 else 1
    tile_k = 64
    while not _parts_ok(K, split_k, tile_k):
        split_k //= 2
    return _gemm(None, M, N, K, in_dtype=rng.choice(["bf16", "bf16", "bf16", "f16"]), out=rng.choice(["bf16", "f32"]),
                 epilogue=rng.choice(["none", "bias", "bias_silu"]), split_k=split_k,
                 split_combine=rng.choice(["seq", "tree"]), tile_k=tile_k,
                 tile_combine=rng.choice(["carry", "carry", "carry", "carry", "tree"]))


def _draw_packed(rng):
    M, N, K = _log(rng, 1, 64), _log(rng, 256, 14336), _log(rng, 256, 14336)
    if rng.random() < 0.6:
        N, K = -(-N // 64) * 64, -(-K // 64) * 64
    split_k = rng.choice([1, 2, 4, 8])
    while not _parts_ok(K, split_k, 64):
        split_k //= 2
    return _gemm(None, M, N, K, in_dtype=rng.choice(["bf16", "f16", "bf16_e4m3"]), out=rng.choice(["bf16", "f32"]),
                 epilogue=rng.choice(["none", "bias", "bias_silu"]), split_k=split_k,
                 split_combine=rng.choice(["seq", "tree"]), packed=True)


def _draw_e4m3(rng):
    M, N, K = _log(rng, 16, 2048), -(-_log(rng, 256, 14336) // 16) * 16, -(-_log(rng, 256, 14336) // 16) * 16
    while 2.0 * M * N * K > MAX_FLOPS:
        M = -(-M // 2)
    return _gemm(None, M, N, K, in_dtype="e4m3", tile_k=128, epilogue=rng.choice(["none", "bias", "bias_silu"]))


def _draw_attention(rng):
    H, dim, key_block = _log(rng, 1, 32), rng.choice([64, 128]), rng.choice([32, 64, 128])
    form = rng.choice(["causal", "cross", "decode"])
    if form == "causal":
        L = _log(rng, 64, 4096)
        return _attn(None, H, L, L, dim, 1, key_block, rng.choice([64, 128]))
    Lq = _log(rng, 64, 2048) if form == "cross" else _log(rng, 1, 16)
    return _attn(None, H, Lq, _log(rng, 64, 4096), dim, 0, key_block, 128)


def _draw_rows(rng):
    op = rng.choice(["rowsum", "rmsnorm", "layernorm", "softmax"])
    cols, rows = _log(rng, 64, 131072), _log(rng, 1, 16384)
    if rng.random() < 0.6:
        cols = -(-cols // 64) * 64
    rows = max(1, min(rows, MAX_ELEMS // cols))
    leaf = rng.choice([(64, "contiguous", "up"), (64, "contiguous", "up"), (256, "strided", "down"),
                       (128, "strided", "up"), (64, "strided", "down")])
    return _rows(None, op, rows, cols, leaf[0], leaf[1], leaf[2], "f32" if op == "rowsum" else rng.choice(["bf16", "f32"]))


def draw(rng):
    how = rng.choice([_draw_gemm] * 5 + [_draw_packed] + [_draw_e4m3] + [_draw_attention] * 2 + [_draw_rows] * 3)
    return how(rng)


# ------------------------------------------------------------------- inputs

def _inputs(c, seed):
    """The operands a program holds, on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, scale, dtype):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale).to(dtype)

    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        ta = {"bf16": torch.bfloat16, "f16": torch.float16, "bf16_e4m3": torch.bfloat16,
              "e4m3": torch.float8_e4m3fn}[c["in_dtype"]]
        tb = torch.float8_e4m3fn if c["in_dtype"] in ("e4m3", "bf16_e4m3") else ta
        # activations ~ N(0, 1); weights ~ N(0, 0.02), or scaled into e4m3's range
        A = normal((M, K), 1.0, ta)
        B = normal((K, N), 0.5 if tb is torch.float8_e4m3fn else 0.02, tb)
        bias = normal((N,), 0.02, torch.bfloat16) if c["epilogue"] != "none" else None
        return A, B, bias
    if c["kind"] == "attention":
        H, d = c["H"], c["dim"]
        return (normal((H, c["Lq"], d), 1.5, torch.bfloat16), normal((H, c["Lk"], d), 1.5, torch.bfloat16),
                normal((H, c["Lk"], d), 1.0, torch.bfloat16))
    rows, cols = c["rows"], c["cols"]
    X = normal((rows, cols), 2.0, torch.float32)
    if c["op"] == "rowsum":                     # values of many magnitudes, both signs
        X = torch.sign(X) * torch.exp(torch.abs(X))
    w = normal((cols,), 0.1, torch.bfloat16) + 1.0
    b = normal((cols,), 0.1, torch.bfloat16)
    return X, w, b


def _out(c):
    return torch.bfloat16 if c["out"] == "bf16" else torch.float32


def _qk_scale(c):
    """log2 e / sqrt(d), as the entry point takes it."""
    return math.log2(math.e) / math.sqrt(c["dim"])


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    if c["kind"] == "gemm":
        A, B, bias = x
        desc = dg.Desc(mma="16x16x128_f8f6f4" if c["in_dtype"] == "e4m3" else "16x16x32", tile_k=c["tile_k"],
                       split_k=c["split_k"], split_combine=c["split_combine"], tile_combine=c["tile_combine"],
                       in_dtype=c["in_dtype"], out=c["out"], epilogue=c["epilogue"])
        C = torch.empty((c["M"], c["N"]), dtype=_out(c), device="cuda")
        if c["packed"]:                         # the weight is packed once, when it is loaded
            B = dg.dg_pack_b(B)
        return dict(call="packed" if c["packed"] else "gemm", desc=desc, A=A, B=B, bias=bias, C=C)
    if c["kind"] == "attention":
        Q, K, V = x
        desc = dg.AttnDesc(key_block=c["key_block"], causal=c["causal"], q_block=c["q_block"],
                           block_sum=c["block_sum"], out=c["out"])
        return dict(call="attention", desc=desc, Q=Q, K=K, V=V, O=torch.empty(Q.shape, dtype=_out(c), device="cuda"),
                    scale=_qk_scale(c))
    X, w, b = x
    desc = dg.Desc(leaf_w=c["leaf_w"], leaf_layout=c["leaf_layout"], lane_fold=c["lane_fold"], out=c["out"],
                   reduce="sumsq" if c["op"] == "rmsnorm" else "sum")
    Y = torch.empty((c["rows"],) if c["op"] == "rowsum" else X.shape, dtype=_out(c), device="cuda")
    return dict(call=c["op"], desc=desc, X=X, w=w, b=b, Y=Y)


def run(state):
    s = state
    if s["call"] == "gemm":
        return dg.dg_gemm(s["desc"], s["A"], s["B"], s["bias"], s["C"])
    if s["call"] == "packed":
        return dg.dg_gemm_packed(s["desc"], s["A"], s["B"], s["bias"], s["C"])
    if s["call"] == "attention":
        return dg.dg_attention(s["desc"], s["Q"], s["K"], s["V"], s["O"], s["scale"])
    if s["call"] == "rowsum":
        return dg.dg_rowsum(s["desc"], s["X"], s["Y"])
    if s["call"] == "rmsnorm":
        return dg.dg_rmsnorm(s["desc"], s["X"], s["w"], 1e-5, s["Y"])
    if s["call"] == "layernorm":
        return dg.dg_layernorm(s["desc"], s["X"], s["w"], s["b"], 1e-5, s["Y"])
    return dg.dg_softmax(s["desc"], s["X"], s["Y"])


# ------------------------------------------------------- work and references

def _visible(c):
    """Query-key pairs that take part."""
    return c["Lq"] * (c["Lq"] + 1) / 2 if c["causal"] else c["Lq"] * c["Lk"]


def work(case):
    c = case
    ob = 2 if c["out"] == "bf16" else 4
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        ab = 1 if c["in_dtype"] == "e4m3" else 2
        bb = 1 if c["in_dtype"] in ("e4m3", "bf16_e4m3") else 2
        return dict(bytes=ab * M * K + bb * K * N + ob * M * N + (2 * N if c["epilogue"] != "none" else 0),
                    flops=2.0 * M * N * K)
    if c["kind"] == "attention":
        H, d = c["H"], c["dim"]
        return dict(bytes=H * d * (2 * c["Lq"] + 4 * c["Lk"] + ob * c["Lq"]), flops=4.0 * H * d * _visible(c))
    n = c["rows"] * c["cols"]
    if c["op"] == "rowsum":
        return dict(bytes=4 * n + 4 * c["rows"], flops=n)
    vec = {"rmsnorm": 2, "layernorm": 4, "softmax": 0}[c["op"]]
    return dict(bytes=(4 + ob) * n + vec * c["cols"], flops={"rmsnorm": 4, "layernorm": 7, "softmax": 12}[c["op"]] * n)


def tolerance(case):
    # the descriptor fixes the order of every sum and every rounding point:
    # an implementation of it has no freedom in any bit
    return "exact"


def _wide(t):
    """A tensor's values in 64 bits."""
    return (t.float() if t.dtype == torch.float8_e4m3fn else t).double()


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    if c["kind"] == "gemm":
        A, B, bias = x
        z = _wide(A) @ _wide(B)
        if bias is not None:
            z = z + bias.double()
        return z * torch.sigmoid(z) if c["epilogue"] == "bias_silu" else z
    if c["kind"] == "attention":
        Q, K, V = x
        O = torch.empty(Q.shape, dtype=torch.float64, device="cuda")
        for h in range(c["H"]):
            s = Q[h].double() @ K[h].double().t().contiguous() / math.sqrt(c["dim"])
            if c["causal"]:
                s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf)
            O[h] = torch.softmax(s, dim=1) @ V[h].double()
        return O
    X, w, b = x
    Y = torch.empty((c["rows"],) if c["op"] == "rowsum" else X.shape, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 24) // c["cols"])
    for r in range(0, c["rows"], step):         # in pieces: 64-bit copies are large
        v = X[r:r + step].double()
        if c["op"] == "rowsum":
            y = v.sum(1)
        elif c["op"] == "rmsnorm":
            y = v / torch.sqrt((v * v).mean(1, keepdim=True) + 1e-5) * w.double()
        elif c["op"] == "layernorm":
            d = v - v.mean(1, keepdim=True)
            y = d / torch.sqrt((d * d).mean(1, keepdim=True) + 1e-5) * w.double() + b.double()
        else:
            y = torch.softmax(v, dim=1)
        Y[r:r + step] = y
    return Y
