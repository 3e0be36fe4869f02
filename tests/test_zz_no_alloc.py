"""xgemm_run_noalloc: the allocation-free variant of xgemm_run (scratch in a
static per-GPU array).  Through the C ABI, against xgemm_run's output (the
same plan and kernels, so the same bits) and the oracle, on two calls in a
row, the second with a smaller input; the device's free memory does not
change across the calls."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import CODE, check_close, check_exact, to_device
from paper_2609_16389_amd import workloads as wl
from paper_2609_16389_amd import xgemm as xg

pytestmark = pytest.mark.gpu


def _launch(M, N, K):
    """Workspace bytes of the launch xgemm_run makes for these (contiguous)
    arguments, and which operands it copies (1: A, 2: B, 3: both)."""
    assert xg.xgemm_select_band(M, N, K, xg.XGEMM_BF16, 256).axis == xg.XGEMM_BAND_NONE
    cfg = xg.xgemm_launch_config(M, N, K, 1 << 20, K, 1 << 20, N, 256)
    info = xg.xgemm_trace_plan(M, N, K, 1 << 20, K, 1 << 20, N, 1 << 20, N, cfg, 256, 0)
    return xg.xgemm_workspace_bytes(M, N, K, 256, cfg), info.packed


def _call(fn, h, M, N, K, dA, dB, C, dtype, s):
    rc = fn(h, M, N, K, dA.data_ptr(), dA.stride(0), dB.data_ptr(), dB.stride(0), C.data_ptr(), N, CODE[dtype], s)
    return rc


@pytest.mark.parametrize("cases", [
    # split-k plans (partials in the scratch array), the second smaller
    [(1024, 1024, 16384, "bf16", 301), (512, 512, 8192, "bf16", 302)],
    # operand copies (N or K odd: both, or B, copied into the scratch array)
    [(2047, 1999, 777, "fp16", 305), (1500, 1501, 1024, "fp16", 306)],
    # the same layouts read in place, and one whose blocks the last workgroup of each tile adds
    [(1000, 1001, 1024, "fp16", 303), (300, 203, 777, "fp16", 304)],
], ids=["split_k", "packed", "in_place"])
def test_noalloc_matches_xgemm_run(cases, request):
    oracle.build(force=False)
    h = xg.xgemm_create()
    try:
        s = torch.cuda.current_stream().cuda_stream
        data = []
        for M, N, K, dtype, seed in cases:
            A, B = wl.make_inputs(M, N, K, dtype, "uniform", seed)
            C_ref, S = oracle.gemm(A, B, dtype)
            data.append((M, N, K, dtype, to_device(A, dtype), to_device(B, dtype), C_ref, S))
        # the scratch array is really used: split partials or copies
        used = [_launch(M, N, K) for M, N, K, *_ in data]
        assert max(ws for ws, _ in used) <= xg.XGEMM_NOALLOC_SCRATCH_BYTES
        assert [(ws > 0, packed) for ws, packed in used] == {
            "split_k": [(True, 0), (True, 0)], "packed": [(True, 3), (True, 2)], "in_place": [(False, 0), (True, 0)],
        }[request.node.callspec.id], used
        outs = [torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda") for M, N, *_ in data]
        torch.cuda.synchronize()
        free0, _ = torch.cuda.mem_get_info()
        for (M, N, K, dtype, dA, dB, _, _), C in zip(data, outs):
            assert _call(xg.xgemm_run_noalloc, h, M, N, K, dA, dB, C, dtype, s) == xg.XGEMM_OK, \
                xg.xgemm_last_error(h)
            torch.cuda.synchronize()
        free1, _ = torch.cuda.mem_get_info()
        assert free1 == free0, "device free memory changed by %d bytes" % (free0 - free1)
        for (M, N, K, dtype, dA, dB, C_ref, S), C in zip(data, outs):
            ref = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
            assert _call(xg.xgemm_run, h, M, N, K, dA, dB, ref, dtype, s) == xg.XGEMM_OK
            torch.cuda.synchronize()
            got = C.cpu().numpy()
            check_exact(got, ref.cpu().numpy().astype(np.float64), "noalloc vs xgemm_run %dx%dx%d" % (M, N, K))
            check_close(got, C_ref, S, "noalloc vs oracle %dx%dx%d" % (M, N, K))
    finally:
        torch.cuda.synchronize()
        xg.xgemm_destroy(h)


def test_noalloc_rejects_calls_beyond_the_scratch():
    """A call whose plan needs more scratch than the static array holds
    fails with XGEMM_ERR_INVALID_ARG before anything is enqueued; the
    buffers are sized for the call, and C is left as it was."""
    M, N, K = 4096, 4097, 4096        # N odd: B copied, 4096 x 4104 x 2 bytes = 32 MiB
    M2, N2, K2 = 8192, 8193, 8192     # B copy 8192 x 8200 x 2 bytes = 128 MiB, above 64 MiB
    h = xg.xgemm_create()
    try:
        s = torch.cuda.current_stream().cuda_stream
        A = torch.zeros((M2, K2), dtype=torch.bfloat16, device="cuda")
        B = torch.zeros((K2, N2), dtype=torch.bfloat16, device="cuda")
        C = torch.full((M2, N2), 5.0, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        rc = xg.xgemm_run_noalloc(h, M2, N2, K2, A.data_ptr(), K2, B.data_ptr(), N2, C.data_ptr(), N2,
                                  xg.XGEMM_BF16, s)
        assert rc == xg.XGEMM_ERR_INVALID_ARG
        assert "scratch" in xg.xgemm_last_error(h)
        torch.cuda.synchronize()
        assert torch.all(C == 5.0)
        # a call that fits still runs on the same handle (zeros in, zeros out)
        rc = xg.xgemm_run_noalloc(h, M, N, K, A.data_ptr(), K2, B.data_ptr(), N2, C.data_ptr(), N2,
                                  xg.XGEMM_BF16, s)
        assert rc == xg.XGEMM_OK, xg.xgemm_last_error(h)
        torch.cuda.synchronize()
        assert torch.all(C[:M, :N] == 0.0) and torch.all(C[:, N:] == 5.0) and torch.all(C[M:] == 5.0)
    finally:
        xg.xgemm_destroy(h)


@pytest.mark.parametrize("M,N,K", [(201, 571, 37855), (515, 207, 41455), (16, 10377, 8657)],
                         ids=lambda v: str(v))
def test_noalloc_at_the_scratch_limit(M, N, K):
    """Where the static array decides: a K split one deeper than it holds, and
    a decoding step read in place whose operand copies it could not hold.
    Taken, with xgemm_run's bits."""
    oracle.build(force=False)
    A, B = wl.make_inputs(M, N, K, "bf16", "uniform", seed=M)
    dA, dB = to_device(A, "bf16"), to_device(B, "bf16")
    outs = [torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
    h = xg.xgemm_create()
    try:
        s = torch.cuda.current_stream().cuda_stream
        for fn, C in zip((xg.xgemm_run_noalloc, xg.xgemm_run), outs):
            assert _call(fn, h, M, N, K, dA, dB, C, "bf16", s) == xg.XGEMM_OK, xg.xgemm_last_error(h)
        torch.cuda.synchronize()
        assert torch.equal(*outs)
        rows = np.unique(np.linspace(0, M - 1, 16).astype(int))
        C_ref, S = oracle.gemm_rows(A, B, "bf16", rows)
        check_close(outs[0].cpu().numpy()[rows], C_ref, S, "noalloc %dx%dx%d" % (M, N, K))
    finally:
        torch.cuda.synchronize()
        xg.xgemm_destroy(h)
