"""The register-direct kernel: the synchronisation checker's traces (bounds of
every load, every element of C stored once, the LDS exchange) and parity with
the oracle, at the edges of its blocks, slabs and dispatch."""
import numpy as np
import pytest

import oracle
from paper_2609_16389_amd import syncheck as sc
from paper_2609_16389_amd import workloads as wl
from paper_2609_16389_amd import xgemm as xg

DIRECT = list(range(xg.XGEMM_DIRECT_16x128, xg.XGEMM_DIRECT_END))

# (M, N, K, pad of lda, of ldb, of ldc, split): the smallest sizes, one block
# and one beyond it, a wave with no slab, partial slabs and partial vectors in
# N, odd rows, K splits whose last range is partial
EDGES = [(1, 8, 8, 0, 0, 0, 1), (1, 9, 9, 0, 0, 0, 1), (17, 65, 63, 3, 1, 1, 1), (64, 256, 64, 0, 0, 0, 1),
         (65, 257, 65, 8, 8, 4, 1), (33, 129, 520, 1, 0, 0, 1), (16, 300, 1101, 0, 0, 3, 2), (70, 136, 777, 0, 3, 0, 3)]


def _cfg(tile, split=1):
    return xg.xgemm_config(tile, split, 4, 0)


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("case", EDGES, ids=lambda c: "x".join(map(str, c)))
def test_traces(tile, case):
    M, N, K, pa, pb, pc, split = case
    info = xg.xgemm_trace_plan(M, N, K, sc.BASE_A, K + pa, sc.BASE_B, N + pb, sc.BASE_C, N + pc, _cfg(tile, split),
                               256, 0)
    assert info.family == xg.XGEMM_KERNEL_DIRECT and info.packed == 0
    rep = sc.check_launch(M, N, K, _cfg(tile, split), lda=K + pa, ldb=N + pb, ldc=N + pc)
    assert rep.ok, [str(v) for v in rep.violations]


def test_too_small_or_too_wide_falls_back():
    """Fewer than 8 columns or K, or rows so far apart that 32-bit offsets
    overflow: another family runs."""
    for M, N, K, lda, ldb in [(64, 7, 512, 512, 7), (64, 512, 7, 7, 512), (64, 64, 64, 1 << 26, 64),
                              (64, 64, 64, 64, 1 << 26)]:
        assert xg.xgemm_kernel_family(M, N, K, 1 << 20, lda, 1 << 20, ldb, _cfg(xg.XGEMM_DIRECT_64x64)) \
            != xg.XGEMM_KERNEL_DIRECT


K2 = xg.XGEMM_TILE_128x128_K2


@pytest.mark.parametrize("K", [256, 320, 384, 448, 264, 328])
def test_k2_tile_traces(K):
    """The four-stage wave-pair tile from its fewest steps up, both parities
    of its loop, whole and partial steps; fewer steps take another family."""
    assert xg.xgemm_kernel_family(200, 136, K, 1 << 20, K, 1 << 20, 136, _cfg(K2)) == xg.XGEMM_KERNEL_PIPELINED
    rep = sc.check_launch(200, 136, K, _cfg(K2))
    assert rep.ok, [str(v) for v in rep.violations]
    assert xg.xgemm_kernel_family(200, 136, 192, 1 << 20, 192, 1 << 20, 136, _cfg(K2)) == xg.XGEMM_KERNEL_GENERAL


@pytest.mark.gpu
@pytest.mark.parametrize("K,split", [(256, 1), (320, 1), (384, 1), (448, 1), (264, 1), (328, 1), (1097, 2), (4096, 16)])
def test_k2_tile_parity(K, split):
    from gpu_util import check_close, run_gpu
    M, N = 200, 136
    oracle.build(force=False)
    for dtype in ("bf16", "fp16"):
        A, B = wl.make_inputs(M, N, K, dtype, "uniform", K)
        C_ref, S = oracle.gemm(A, B, dtype)
        check_close(run_gpu(A, B, dtype, config=_cfg(K2, split)), C_ref, S, "K2 %s K=%d" % (dtype, K))


def test_dispatch():
    """Few output tiles take the direct kernel in any layout; whole rounds of
    large tiles, banded and persistent plans keep theirs; a launch that
    replaces a K-split plan adds at least as many partial sums."""
    def launch(M, N, K, lda=None, ldb=None):
        return xg.xgemm_launch_config(M, N, K, 1 << 20, lda or K, 1 << 20, ldb or N, 256)
    for shape in [(256, 256, 256), (1000, 1000, 1000), (16, 4096, 4096), (1, 2496, 5751), (300, 203, 777)]:
        assert launch(*shape).tile in DIRECT, shape
    assert launch(2048, 2048, 2048).tile == K2
    for shape in [(4096, 4096, 4096), (8192, 8192, 8192), (6144, 6144, 6144), (1024, 1024, 65536)]:
        c, b = launch(*shape), xg.xgemm_select_band(*shape, xg.XGEMM_BF16, 256)
        assert (c.tile, c.split_k, c.stream_k) == (b.body.tile, b.body.split_k, b.body.stream_k), shape
    # partial sums per element and K range: one per wave that takes slabs of its own
    chains = dict(zip(DIRECT, (8, 8, 8, 4, 2, 1, 1)))
    chains.update({xg.XGEMM_TILE_256x256: 1, xg.XGEMM_TILE_256x128: 2, xg.XGEMM_TILE_128x128: 1, K2: 2})
    rng = np.random.default_rng(5)
    # (the first two replace splits of the 256 x 128 tile, whose wave pairs split K too)
    shapes = [(186, 7641, 6040), (166, 7695, 6627)]
    shapes += [[int(2 ** rng.uniform(0, top)) for top in ((12, 12, 12), (10, 10, 16))[i % 2]] for i in range(3000)]
    replaced = {}
    for M, N, K in shapes:
        b = xg.xgemm_select_band(M, N, K, xg.XGEMM_BF16, 256)
        c, s = launch(M, N, K), b.body
        if b.axis == xg.XGEMM_BAND_NONE and c.tile != s.tile and s.split_k > 1:
            replaced[s.tile] = replaced.get(s.tile, 0) + 1
            assert c.split_k * chains[c.tile] >= s.split_k * chains[s.tile], (M, N, K)
    assert replaced[xg.XGEMM_TILE_256x128] > 0 and replaced[xg.XGEMM_TILE_128x128] >= 100, replaced


def _operand(bits, dtype, pad):
    import torch
    from gpu_util import to_device
    rows, cols = bits.shape
    wide = np.full((rows, cols + pad), 0x7E00 if dtype == "fp16" else 0x7FC0, dtype=np.uint16)   # NaN padding
    wide[:, :cols] = bits
    return to_device(wide, dtype)[:, :cols]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("case", EDGES, ids=lambda c: "x".join(map(str, c)))
def test_parity(tile, case, dtype):
    import torch
    from gpu_util import check_close
    M, N, K, pa, pb, pc, split = case
    oracle.build(force=False)
    A, B = wl.make_inputs(M, N, K, dtype, "uniform", M + N + K)
    C_ref, S = oracle.gemm(A, B, dtype)
    out = torch.full((M, N + pc), 7.0, dtype=torch.float32, device="cuda")
    xg.gemm(_operand(A, dtype, pa), _operand(B, dtype, pb), out=out[:, :N], config=_cfg(tile, split))
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    check_close(got[:, :N], C_ref, S, "direct %d %s" % (tile, case))
    assert np.all(got[:, N:] == 7.0)


# batches that take the direct kernel (tests/test_plan_calls.py checks it)
BATCHES = [(5, 70, 264, 64), (3, 33, 137, 129), (40, 200, 72, 200)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", BATCHES, ids=lambda s: "x".join(map(str, s)))
def test_batched_parity(shape):
    """Every problem's block edges."""
    import torch
    from gpu_util import check_close, to_device
    L, M, N, K = shape
    oracle.build(force=False)
    cases = [wl.make_inputs(M, N, K, "bf16", "normal", seed=b) for b in range(L)]
    A = torch.stack([to_device(a, "bf16") for a, _ in cases])
    B = torch.stack([to_device(b, "bf16") for _, b in cases])
    C = xg.bmm(A, B).cpu().numpy()
    for b, (a_bits, b_bits) in enumerate(cases):
        C_ref, S = oracle.gemm(a_bits, b_bits, "bf16")
        check_close(C[b], C_ref, S, "batched direct %s problem %d" % (shape, b))


@pytest.mark.gpu
def test_batched_under_a_workspace_limit():
    """A limit on the workspace does not refuse a batch that needs none (its
    tile plan would copy both operands)."""
    import torch
    from gpu_util import check_close, to_device
    L, M, N, K = 3, 300, 201, 1000
    oracle.build(force=False)
    A, B = wl.make_inputs(M, N, K, "bf16", "normal", seed=5)
    C_ref, S = oracle.gemm(A, B, "bf16")
    dA, dB = (torch.stack([to_device(x, "bf16")] * L) for x in (A, B))
    C = torch.full((L, M, N), float("nan"), device="cuda")
    h = xg.xgemm_create()
    try:
        assert xg.xgemm_set_workspace_limit(h, 4096) == xg.XGEMM_OK
        rc = xg.xgemm_run_strided_batched(h, L, M, N, K, dA.data_ptr(), K, M * K, dB.data_ptr(), N, K * N, C.data_ptr(),
                                          N, M * N, xg.XGEMM_BF16, torch.cuda.current_stream().cuda_stream)
        assert rc == xg.XGEMM_OK, xg.xgemm_last_error(h)
        torch.cuda.synchronize()
        for b in range(L):
            check_close(C[b].cpu().numpy(), C_ref, S, "batched under a limit, problem %d" % b)
    finally:
        torch.cuda.synchronize()
        xg.xgemm_destroy(h)


@pytest.mark.gpu
def test_infinities_stay_in_their_rows():
    """Zeroed lanes past K and clamped rows must not meet infinities of other
    rows: one infinite element of A reaches its own row only."""
    import torch
    M, N, K = 20, 40, 75
    A = torch.ones((M, K), dtype=torch.bfloat16, device="cuda")
    B = torch.ones((K, N), dtype=torch.bfloat16, device="cuda")
    A[M - 1, K - 1] = float("inf")
    for tile in DIRECT:
        C = xg.gemm(A, B, config=_cfg(tile))
        assert torch.all(torch.isinf(C[M - 1])) and torch.all(C[:M - 1] == K), tile


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("split", [1, 2])
def test_streaming_variant(dtype, split):
    """B of 98 MB in rows of whole cache lines, read with streaming loads:
    ragged rows, and a partial slab and vector of K."""
    import torch
    from gpu_util import check_close
    M, N, K = 5, 8192, 6001
    oracle.build(force=False)
    A, B = wl.make_inputs(M, N, K, dtype, "uniform", K)
    C_ref, S = oracle.gemm(A, B, dtype)
    out = torch.full((M, N), float("nan"), device="cuda")
    b = torch.from_numpy(B.view(np.int16)).cuda().view(torch.bfloat16 if dtype == "bf16" else torch.float16)
    assert b.data_ptr() % 128 == 0 and 96e6 < 2 * N * K < 140e6
    xg.gemm(_operand(A, dtype, 0), b, out=out, config=_cfg(xg.XGEMM_DIRECT_16x128, split))
    torch.cuda.synchronize()
    check_close(out.cpu().numpy(), C_ref, S, "streaming %s split %d" % (dtype, split))


# (M, N, K, split) with partial blocks added by the last workgroup of a tile:
# two ranges and the most, one tile and several, ragged rows and columns
COMBINED = [(1, 8, 512, 2), (16, 300, 1101, 4), (70, 136, 2000, 3), (65, 257, 4160, 4)]


@pytest.mark.parametrize("tile", [t for t in DIRECT if t <= xg.XGEMM_DIRECT_32x256])
@pytest.mark.parametrize("case", COMBINED, ids=lambda c: "x".join(map(str, c)))
def test_combined_split_traces(tile, case):
    M, N, K, split = case
    info = xg.xgemm_trace_plan(M, N, K, sc.BASE_A, K, sc.BASE_B, N, sc.BASE_C, N, _cfg(tile, split), 256, 0)
    assert info.reduce == 2
    rep = sc.check_launch(M, N, K, _cfg(tile, split))
    assert rep.ok, [str(v) for v in rep.violations]


def test_combined_split_planted_mistake():
    """A workgroup that reads the others' blocks without having found itself
    last, or a block that nobody stored, is caught as partials read back that
    no workgroup stores."""
    tile, (M, N, K, split) = xg.XGEMM_DIRECT_32x64, (40, 70, 900, 3)
    real = sc.trace_workgroup

    def without_first_range(m, n, k, lda, ldb, ldc, cfg, cu, seg, block, threads, capacity=None, schedule=0):
        ev, counts = real(m, n, k, lda, ldb, ldc, cfg, cu, seg, block, threads, capacity, schedule)
        part = (ev["op"] == sc.STORE) & (ev["addr"] >= sc.BASE_W + sc.PREFIX_BYTES) & (ev["arg"] == 16)
        if block == 0:
            ev["addr"][part] += 1 << 20
        return ev, counts
    mp = pytest.MonkeyPatch()
    try:
        mp.setattr(sc, "trace_workgroup", without_first_range)
        rep = sc.check_launch(M, N, K, _cfg(tile, split))
    finally:
        mp.undo()
    assert not rep.ok


def test_deep_splits_take_a_second_launch():
    """More partial blocks than one CU should read, or waves that share no
    block: the separate reduction."""
    for tile, split in [(xg.XGEMM_DIRECT_64x128, 5), (xg.XGEMM_DIRECT_64x64, 9), (xg.XGEMM_DIRECT_64x256, 2)]:
        info = xg.xgemm_trace_plan(64, 256, 16384, sc.BASE_A, 16384, sc.BASE_B, 256, sc.BASE_C, 256, _cfg(tile, split),
                                   256, 0)
        assert info.reduce == 1, tile


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [t for t in DIRECT if t <= xg.XGEMM_DIRECT_32x256])
@pytest.mark.parametrize("case", COMBINED, ids=lambda c: "x".join(map(str, c)))
def test_combined_split(tile, case):
    """Against the oracle; the same bits on every run (whichever workgroup is
    last, and with the counters left at zero) and on graph replays with eager
    calls between them."""
    import torch
    from gpu_util import check_close, to_device
    M, N, K, split = case
    oracle.build(force=False)
    A, B = wl.make_inputs(M, N, K, "bf16", "uniform", M + K)
    C_ref, S = oracle.gemm(A, B, "bf16")
    dA, dB, st = to_device(A, "bf16"), to_device(B, "bf16"), torch.cuda.Stream()
    cfg, out = _cfg(tile, split), torch.empty(M, N, device="cuda")
    torch.cuda.synchronize()
    xg.gemm(dA, dB, out=out, config=cfg, stream=st)
    st.synchronize()
    first = out.clone()
    check_close(first.cpu().numpy(), C_ref, S, "combined %d %s" % (tile, case))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        for _ in range(3):
            xg.gemm(dA, dB, out=out, config=cfg, stream=st)
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, first)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        xg.gemm(dA, dB, out=out, config=cfg, stream=st)
        torch.cuda.synchronize()
        assert torch.equal(out, first)
