"""The work a program has this library do, as timed cases.

A case is one call of a public entry point: ``gemm`` (xgemm_run), ``bmm``
(xgemm_run_strided_batched), ``gemv`` (xgemv_run) or the allocation-free
``xgemm_run_noalloc``.  A user's program holds its operands and an output
buffer on the GPU and calls the entry point on torch's current stream; so do
the cases here.  The output is the whole of C (or y).

The ranges:

* products of 16-bit matrices from 128 to 8192 a side, whole tiles, multiples
  of 8 and odd sizes, contiguous or column slices of wider arrays;
* decoding steps: 1 to 64 rows of activations against a projection's weights;
* products with few outputs and a long K (the split-k problems);
* batches of small products, K from one attention head's width up;
* fp32 matrix-vector products, square and with few rows or few columns.
"""
import math

import torch

from paper_2609_16389_amd import xgemm as xg

_DTYPE = {"bf16": torch.bfloat16, "fp16": torch.float16}
_CODE = {"bf16": xg.XGEMM_BF16, "fp16": xg.XGEMM_FP16}


def _gemm(name, M, N, K, dtype, dist="uniform", param=1.0, pad=0, op="gemm"):
    return {"name": name, "op": op, "M": M, "N": N, "K": K, "dtype": dtype, "dist": dist, "param": param, "pad": pad}


def _bmm(name, L, M, N, K, dtype):
    return {"name": name, "op": "bmm", "L": L, "M": M, "N": N, "K": K, "dtype": dtype, "dist": "normal", "param": 1.0}


def _gemv(name, M, K):
    return {"name": name, "op": "gemv", "M": M, "K": K, "dtype": "fp32", "dist": "uniform", "param": 1.0}


def listed():
    return [
        # the smallest call: launches and latency
        _gemm("gemm256_fp16", 256, 256, 256, "fp16"),
        # one decoding step of 16 sequences through an up-projection, from a
        # serving loop that may not allocate: the weights' bytes
        _gemm("decode16x14336x4096_bf16", 16, 14336, 4096, "bf16", "normal", op="noalloc"),
        # an ordinary size that is no multiple of any tile
        _gemm("gemm1000_bf16", 1000, 1000, 1000, "bf16", "normal"),
        # odd everywhere: no row of A, B or C but the first is aligned
        _gemm("gemm2047_bf16", 2047, 2047, 2047, "bf16", "normal"),
        # one round of tiles on the whole GPU
        _gemm("gemm4096_bf16", 4096, 4096, 4096, "bf16", "normal"),
        # the headline size
        _gemm("gemm8192_bf16", 8192, 8192, 8192, "bf16"),
        # a projection over a prompt of 4096 tokens (prefill)
        _gemm("proj4096x14336x4096_fp16", 4096, 14336, 4096, "fp16", "normal", 0.02),
        # few outputs, long K, as in a weight gradient over many tokens
        _gemm("skinny1024x1024x65536_bf16", 1024, 1024, 65536, "bf16"),
        # many of the smallest products in one launch
        _bmm("bmm64x256_fp16", 64, 256, 256, 256, "fp16"),
        # attention scores of 32 heads: K is a head's width, C the bulk
        _bmm("bmm32x1024x1024x128_bf16", 32, 1024, 1024, 128, "bf16"),
        # matrix-vector products: one that the last-level cache holds, one from HBM
        _gemv("gemv4096_fp32", 4096, 4096),
        _gemv("gemv16384_fp32", 16384, 16384),
    ]


def _size(rng, lo, hi):
    """A size between lo and hi, even over its logarithm: a multiple of 64,
    a multiple of 8, or any number."""
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    step = rng.choice([64, 64, 8, 1])
    return max(lo, min(hi, (n + step // 2) // step * step))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "decode", "decode", "long", "bmm", "bmm", "gemv", "gemv"])
    dtype = rng.choice(["bf16", "fp16"])
    dist, param = rng.choice([("uniform", 1.0), ("normal", 1.0), ("normal", 0.02)])
    pad = rng.choice([0, 0, 0, 0, 8, 3])
    if kind == "gemm":
        while True:
            M, N, K = _size(rng, 128, 8192), _size(rng, 128, 8192), _size(rng, 128, 8192)
            if M * N * K <= 4096 ** 3 and M * N <= 4096 * 8192:
                break
        c = _gemm("", M, N, K, dtype, dist, param, pad)
    elif kind == "decode":
        M = int(math.exp(rng.uniform(0.0, math.log(64.9))))
        c = _gemm("", M, _size(rng, 1024, 16384), _size(rng, 1024, 16384), dtype, dist, param, pad,
                  rng.choice(["gemm", "noalloc"]))
    elif kind == "long":
        c = _gemm("", _size(rng, 128, 1024), _size(rng, 128, 1024), _size(rng, 8192, 65536), dtype, dist, param)
    elif kind == "bmm":
        while True:
            L = int(math.exp(rng.uniform(math.log(2), math.log(128))))
            M, N, K = _size(rng, 64, 1024), _size(rng, 64, 1024), _size(rng, 64, 1024)
            if L * M * N * K <= 2 ** 33 and L * M * N <= 2 ** 25:
                break
        c = _bmm("", L, M, N, K, dtype)
    else:
        while True:
            M, K = _size(rng, 16, 32768), _size(rng, 256, 65536)
            if 2 ** 16 <= M * K <= 2 ** 28:
                break
        c = _gemv("", M, K)
    # (the allocation-free call holds its operand copies in 64 MiB)
    if c["op"] == "noalloc" and (c["N"] % 8 or c["K"] % 8 or c["pad"] % 8) and c["N"] * c["K"] > 2 ** 24:
        c["op"] = "gemm"
    del c["name"]
    return c


def _values(case, shape, gen):
    """fp32 values of the case's distribution."""
    t = torch.empty(shape, dtype=torch.float32, device="cuda")
    if case["dist"] == "uniform":
        return t.uniform_(-case["param"], case["param"], generator=gen)
    return t.normal_(0.0, case["param"], generator=gen)


def _operands(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "gemv":
        return _values(case, (case["M"], case["K"]), gen), _values(case, (case["K"],), gen)
    dt, M, N, K = _DTYPE[case["dtype"]], case["M"], case["N"], case["K"]
    if case["op"] == "bmm":
        L = case["L"]
        return _values(case, (L, M, K), gen).to(dt), _values(case, (L, K, N), gen).to(dt)
    # with a pad, both operands are the first columns of wider arrays
    pad = case["pad"]
    return _values(case, (M, K + pad), gen).to(dt)[:, :K], _values(case, (K, N + pad), gen).to(dt)[:, :N]


def prepare(case, seed):
    A, B = _operands(case, seed)
    if case["op"] == "gemv":
        shape = (case["M"],)
    elif case["op"] == "bmm":
        shape = (case["L"], case["M"], case["N"])
    else:
        shape = (case["M"], case["N"])
    out = torch.empty(shape, dtype=torch.float32, device="cuda")
    state = {"op": case["op"], "A": A, "B": B, "out": out}
    if case["op"] == "noalloc":
        # a serving loop over the C interface keeps a handle and its arguments
        stream = torch.cuda.current_stream()
        state["args"] = (xg.handle(A.device.index, stream), case["M"], case["N"], case["K"], A.data_ptr(),
                         A.stride(0), B.data_ptr(), B.stride(0), out.data_ptr(), case["N"], _CODE[case["dtype"]],
                         stream.cuda_stream)
    return state


def run(state):
    op = state["op"]
    if op == "gemm":
        return xg.gemm(state["A"], state["B"], out=state["out"])
    if op == "bmm":
        return xg.bmm(state["A"], state["B"], out=state["out"])
    if op == "gemv":
        return xg.gemv(state["A"], state["B"], out=state["out"])
    rc = xg.xgemm_run_noalloc(*state["args"])
    if rc != xg.XGEMM_OK:
        raise xg.XgemmError(rc)
    return state["out"]


def work(case):
    M, K = case["M"], case["K"]
    if case["op"] == "gemv":
        return {"bytes": 4 * (M * K + K + M), "flops": 2 * M * K}
    L, N = case.get("L", 1), case["N"]
    return {"bytes": L * (2 * (M * K + K * N) + 4 * M * N), "flops": 2 * L * M * N * K}


def tolerance(case):
    # fp32 sums of exact products: measured against 64 bits the calls are
    # 0.4e-7 (K = 100) to 5.5e-7 (K = 8192, one chain of additions) off, and
    # another grouping of the sum is off by as much on its own; four times
    # the largest
    return {"rel": 2e-6}


def exact(case, seed):
    A, B = _operands(case, seed)
    return torch.matmul(A.double(), B.double())
