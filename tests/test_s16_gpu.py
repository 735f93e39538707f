"""GPU parity of the product with 16-bit operands against the int16 oracle, bit for bit, through the
C ABI."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_11728_amd as M
    M.load_library()
    return M


def _flat(X, order, pad, fill):
    """X (r x c) as a flat buffer in the given order with padded ld; returns (buffer, ld)."""
    r, c = X.shape
    ld = max(1, (c if order == W.ROW_MAJOR else r)) + pad
    buf = np.full((max(1, r if order == W.ROW_MAJOR else c), ld), fill, dtype=X.dtype)
    if r and c:
        if order == W.ROW_MAJOR:
            buf[:r, :c] = X
        else:
            buf[:c, :r] = X.T
    return buf.reshape(-1), ld


def _operands(m, n, k, dist, seed):
    rng = np.random.default_rng([m, n, k, seed])
    if dist == "uniform":
        A = rng.integers(-32768, 32768, size=(m, k), dtype=np.int16)
        B = rng.integers(-32768, 32768, size=(k, n), dtype=np.int16)
    elif dist == "normal":          # what 16-bit quantized tensors look like
        A = np.clip(np.rint(rng.standard_normal((m, k)) * 3000), -32768, 32767).astype(np.int16)
        B = np.clip(np.rint(rng.standard_normal((k, n)) * 3000), -32768, 32767).astype(np.int16)
    elif dist == "min":
        A = np.full((m, k), -32768, dtype=np.int16)
        B = np.full((k, n), -32768, dtype=np.int16)
    else:                           # the byte boundaries: low byte 0x7f/0x80/0xff/0x00, high byte extremes
        vals = np.array([-32768, -32641, -32640, -129, -128, -1, 0, 1, 127, 128, 255, 256, 32639, 32640, 32767],
                        dtype=np.int16)
        A = rng.choice(vals, size=(m, k))
        B = rng.choice(vals, size=(k, n))
    return A, B


def _check(M, oracle, m, n, k, oa, ob, oc, mode, pad, dist="uniform", seed=0, variant=None, misalign=0):
    import torch
    A2, B2 = _operands(m, n, k, dist, seed)
    A, lda = _flat(A2, oa, pad, 0x5A5A)
    B, ldb = _flat(B2, ob, pad, 0x5A5A)
    rng = np.random.default_rng([seed, 7])
    ldc = max(1, (n if oc == W.ROW_MAJOR else m)) + pad
    C0 = rng.integers(-1000, 1000, size=max(1, m if oc == W.ROW_MAJOR else n) * ldc, dtype=np.int32)
    want = C0.copy()
    oracle.gemm_s16(m, n, k, A, lda, oa, B, ldb, ob, want, ldc, oc, mode)
    dA = torch.from_numpy(A.view(np.uint8)).cuda()
    dB = torch.from_numpy(B.view(np.uint8)).cuda()
    dC = torch.from_numpy(C0).cuda()
    need = M.mipgemm_workspace_size_s16(m, n, k)
    ws = torch.full((need + 64 + misalign,), 0x33, dtype=torch.uint8, device="cuda")
    with M.tuning(MIPGEMM_VARIANT=variant):
        M.mipgemm_s16s16s32(m, n, k, dA, lda, oa, dB, ldb, ob, dC, ldc, oc, mode,
                            workspace=ws[misalign:] if misalign else ws, workspace_bytes=need)
    torch.cuda.synchronize()
    got = dC.cpu().numpy()
    if need:
        assert (ws[misalign + need:].cpu().numpy() == 0x33).all()      # nothing written past the workspace
    if not np.array_equal(got, want):
        bad = np.flatnonzero(got != want)
        pytest.fail("(%d, %d, %d) orders %d%d%d mode %d %s: %d of %d words differ, first at %d: got %d want %d" % (
            m, n, k, oa, ob, oc, mode, dist, bad.size, got.size, bad[0], got[bad[0]], want[bad[0]]))


@pytest.mark.parametrize("orders", [(0, 0, 0), (0, 1, 0), (1, 0, 0), (1, 1, 0), (0, 0, 1), (1, 0, 1), (0, 1, 1), (1, 1, 1)])
@pytest.mark.parametrize("mode", [0, 1])
def test_s16_every_order_and_mode(gpu, oracle, orders, mode):
    oa, ob, oc = orders
    for (m, n, k, pad) in ((37, 50, 70, 3), (128, 192, 256, 0), (200, 65, 1030, 17)):
        for dist in ("uniform", "edges"):
            _check(gpu, oracle, m, n, k, oa, ob, oc, mode, pad, dist, seed=1)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 64, 64), (7, 7, 3), (64, 1, 4096), (3, 4096, 512), (256, 256, 1024),
                                   (512, 384, 2048), (1000, 999, 1001), (130, 70, 63), (16, 2048, 128)],
                         ids=lambda s: "x".join(map(str, s)))
def test_s16_shapes(gpu, oracle, shape):
    m, n, k = shape
    _check(gpu, oracle, m, n, k, 0, 0, 0, W.OVERWRITE, 0, "uniform", seed=2)
    _check(gpu, oracle, m, n, k, 0, 1, 0, W.ACCUMULATE, 8, "normal", seed=3)


def test_s16_wraps_and_extremes(gpu, oracle):
    """All -32768: every product is 2^30, the sums wrap from k = 2 on; and the largest positive
    products next to them."""
    for k in (1, 2, 3, 4, 64, 100, 4097):
        _check(gpu, oracle, 5, 9, k, 0, 0, 0, W.OVERWRITE, 0, "min", seed=4)
    _check(gpu, oracle, 70, 130, 520, 0, 0, 0, W.ACCUMULATE, 0, "min", seed=5)


@pytest.mark.parametrize("variant", ["s16_64", "s16_128"])
@pytest.mark.parametrize("ranges", [1, 2, 4])
def test_s16_under_forced_kernels_and_a_misaligned_workspace(gpu, oracle, variant, ranges):
    """Both tiles with k whole and in ranges; the workspace on a 256-byte boundary and three bytes behind one, with operands
    used as stored and rewritten into it."""
    with gpu.tuning(MIPGEMM_SPLITK=str(ranges)):
        for misalign in (0, 3):
            _check(gpu, oracle, 256, 384, 1024, 0, 0, 0, W.OVERWRITE, 0, "uniform", seed=6, variant=variant, misalign=misalign)
            _check(gpu, oracle, 100, 90, 1100, 0, 0, 0, W.ACCUMULATE, 1, "uniform", seed=7, variant=variant, misalign=misalign)


def test_s16_a_large_product_as_dispatched(gpu, oracle):
    _check(gpu, oracle, 1024, 1536, 2048, 0, 0, 0, W.OVERWRITE, 0, "normal", seed=8)


def test_s16_empty_problems_and_error_paths(gpu):
    import torch
    R, OVW, ACC = W.ROW_MAJOR, W.OVERWRITE, W.ACCUMULATE
    assert gpu.mipgemm_workspace_size_s16(0, 5, 5) == 0 and gpu.mipgemm_workspace_size_s16(-1, 5, 5) == 0
    dA = torch.zeros(256, dtype=torch.int16, device="cuda")
    C0 = np.arange(12, dtype=np.int32) + 5
    dC = torch.from_numpy(C0).cuda()
    gpu.mipgemm_s16s16s32(0, 4, 5, dA, 5, R, dA, 4, R, dC, 4, R, OVW)
    gpu.mipgemm_s16s16s32(3, 0, 5, dA, 5, R, dA, 1, R, dC, 1, R, OVW)
    gpu.mipgemm_s16s16s32(3, 3, 0, dA, 1, R, dA, 3, R, dC, 4, R, ACC)
    torch.cuda.synchronize()
    assert np.array_equal(dC.cpu().numpy(), C0)
    gpu.mipgemm_s16s16s32(3, 3, 0, dA, 1, R, dA, 3, R, dC, 4, R, OVW)        # k == 0: C := 0
    torch.cuda.synchronize()
    want = C0.reshape(3, 4).copy()
    want[:, :3] = 0
    assert np.array_equal(dC.cpu().numpy().reshape(3, 4), want)
    dC = torch.from_numpy(C0).cuda()
    need = gpu.mipgemm_workspace_size_s16(3, 4, 5)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    call = lambda *a, **kw: gpu.mipgemm_s16s16s32(*a, check=False, **kw)
    assert call(3, 4, 5, dA, 5, R, dA, 4, R, dC, 4, R, OVW) == -14                         # no workspace
    assert call(3, 4, 5, dA, 5, R, dA, 4, R, dC, 4, R, OVW, workspace=ws, workspace_bytes=need - 300) == -15
    assert call(3, 4, 5, dA, 4, R, dA, 4, R, dC, 4, R, OVW, workspace=ws, workspace_bytes=need) == -5
    assert call(3, 4, 5, dA, 5, R, dA, 3, R, dC, 4, R, OVW, workspace=ws, workspace_bytes=need) == -8
    assert call(3, 4, 5, dA, 5, R, dA, 4, R, dC, 3, R, OVW, workspace=ws, workspace_bytes=need) == -11
    assert call(3, 4, 5, dA, 5, R, dA, 4, R, dC, 4, R, 2, workspace=ws, workspace_bytes=need) == -13
    assert call(3, 4, 5, None, 5, R, dA, 4, R, dC, 4, R, OVW, workspace=ws, workspace_bytes=need) == -4
    assert call(-1, 4, 5, dA, 5, R, dA, 4, R, dC, 4, R, OVW, workspace=ws, workspace_bytes=need) == -1
    torch.cuda.synchronize()
    assert np.array_equal(dC.cpu().numpy(), C0)


@pytest.mark.parametrize("variant", ["s16_64", "s16_128"])
@pytest.mark.parametrize("orders", [(0, 1, 0), (0, 0, 0), (1, 0, 0), (1, 1, 1)])
def test_s16_tile_edges_block_counts_and_ranges(gpu, oracle, variant, orders):
    """Both tiles at their edges, one to five blocks of k and remainders in eights (streamed as stored)
    and in twos (one operand rewritten, the other not), and k in ranges whose sums meet in slots."""
    oa, ob, oc = orders
    for (m, n, k) in ((8, 8, 8), (64, 128, 64), (136, 120, 72), (72, 264, 128), (128, 64, 200), (136, 136, 264),
                      (136, 136, 70), (130, 136, 320)):
        _check(gpu, oracle, m, n, k, oa, ob, oc, W.OVERWRITE, 0, "edges", seed=9, variant=variant)
    for ranges in (2, 3, 5):
        with gpu.tuning(MIPGEMM_SPLITK=str(ranges)):
            _check(gpu, oracle, 136, 200, 1352, oa, ob, oc, W.ACCUMULATE, 8, "uniform", seed=10, variant=variant)


def test_s16_rows_further_apart_than_32_bit_offsets(gpu, oracle):
    import torch
    m, n, k, lda = 64, 16, 72, (1 << 25) + (1 << 21)   # the last row of A starts 4.5 GB behind the first
    A2, B2 = _operands(m, n, k, "uniform", 11)
    A = torch.empty(m * lda, dtype=torch.int16, device="cuda")
    A.view(m, lda)[:, :k] = torch.from_numpy(A2).cuda()
    B, C = torch.from_numpy(B2).cuda(), torch.zeros((m, n), dtype=torch.int32, device="cuda")
    ws = torch.empty(gpu.mipgemm_workspace_size_s16(m, n, k), dtype=torch.uint8, device="cuda")
    gpu.mipgemm_s16s16s32(m, n, k, A, lda, W.ROW_MAJOR, B, n, W.ROW_MAJOR, C, n, W.ROW_MAJOR, W.OVERWRITE,
                          workspace=ws, workspace_bytes=ws.numel())
    want = (A2.astype(np.int64) @ B2.astype(np.int64)).astype(np.int32)
    assert np.array_equal(C.cpu().numpy(), want)


@pytest.mark.parametrize("variant", ["s16_64", "s16_128"])
def test_s16_rows_of_k_further_apart_than_32_bit_offsets(gpu, variant):
    """The same for operands with k strided: the 64 rows of a block end 4.5 GB behind its first."""
    import torch
    m, n, k, ld = 136, 72, 70, (1 << 25) + (1 << 21)
    A2, B2 = _operands(m, n, k, "uniform", 16)
    C = torch.zeros((m, n), dtype=torch.int32, device="cuda")
    ws = torch.empty(gpu.mipgemm_workspace_size_s16(m, n, k), dtype=torch.uint8, device="cuda")
    far = torch.empty(k * ld, dtype=torch.int16, device="cuda")
    want = (A2.astype(np.int64) @ B2.astype(np.int64)).astype(np.int32)
    with gpu.tuning(MIPGEMM_VARIANT=variant):
        far.view(k, ld)[:, :m] = torch.from_numpy(A2.T.copy()).cuda()
        B = torch.from_numpy(B2).cuda()
        gpu.mipgemm_s16s16s32(m, n, k, far, ld, W.COL_MAJOR, B, n, W.ROW_MAJOR, C, n, W.ROW_MAJOR, W.OVERWRITE,
                              workspace=ws, workspace_bytes=ws.numel())
        assert np.array_equal(C.cpu().numpy(), want)
        C.zero_()
        far.view(k, ld)[:, :n] = torch.from_numpy(B2).cuda()
        A = torch.from_numpy(A2).cuda()
        gpu.mipgemm_s16s16s32(m, n, k, A, k, W.ROW_MAJOR, far, ld, W.ROW_MAJOR, C, n, W.ROW_MAJOR, W.OVERWRITE,
                              workspace=ws, workspace_bytes=ws.numel())
        assert np.array_equal(C.cpu().numpy(), want)


def test_s16_replayed_from_a_graph(gpu):
    import torch
    m, n, k = 64, 192, 1024                            # a shape that splits k outside a capture
    A2, B2 = _operands(m, n, k, "uniform", 12)
    A, B = torch.from_numpy(A2).cuda(), torch.from_numpy(B2).cuda()
    C, E = (torch.zeros((m, n), dtype=torch.int32, device="cuda") for _ in range(2))
    ws, ws2 = (torch.empty(gpu.mipgemm_workspace_size_s16(m, n, k), dtype=torch.uint8, device="cuda") for _ in range(2))
    call = lambda out, w: gpu.mipgemm_s16s16s32(m, n, k, A, k, 0, B, n, 0, out, n, 0, W.OVERWRITE, workspace=w,
                                                workspace_bytes=w.numel())
    want = (A2.astype(np.int64) @ B2.astype(np.int64)).astype(np.int32)
    call(E, ws2)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(C, ws)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call(C, ws)
    for _ in range(3):
        C.zero_()
        graph.replay()
        call(E, ws2)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy(), want) and np.array_equal(E.cpu().numpy(), want)


@pytest.mark.parametrize("variant", ["s16_64", "s16_128"])
@pytest.mark.parametrize("orders", [(0, 1, 0), (1, 0, 1)])
@pytest.mark.parametrize("mode", [W.OVERWRITE, W.ACCUMULATE])
def test_s16_ranges_that_add_into_c(gpu, variant, orders, mode):
    """A captured call, and one whose workspace has no room for slots: ranges of k meet in C itself, inside
    its leading dimension, on every replay."""
    import torch
    oa, ob, oc = orders
    m, n, k, pad = 130, 201, 1352, 3
    A2, B2 = _operands(m, n, k, "uniform", 13)
    A, lda = _flat(A2, oa, 8, 0x5A5A)
    B, ldb = _flat(B2, ob, 8, 0x5A5A)
    ldc = (n if oc == W.ROW_MAJOR else m) + pad
    C0 = np.random.default_rng(14).integers(-1000, 1000, size=(m if oc == W.ROW_MAJOR else n) * ldc, dtype=np.int32)
    want = C0.copy()
    view = want.reshape(-1, ldc)[:, :ldc - pad]
    product = (A2.astype(np.int64) @ B2.astype(np.int64)).astype(np.int32)
    view[:] = (product if oc == W.ROW_MAJOR else product.T) + (view if mode == W.ACCUMULATE else 0)
    dA, dB, first = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), torch.from_numpy(C0).cuda()
    dC = first.clone()
    ws = torch.empty(gpu.mipgemm_workspace_size_s16(m, n, k), dtype=torch.uint8, device="cuda")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with gpu.tuning(MIPGEMM_VARIANT=variant, MIPGEMM_SPLITK="3"):
        with torch.cuda.graph(graph, stream=stream):
            gpu.mipgemm_s16s16s32(m, n, k, dA, lda, oa, dB, ldb, ob, dC, ldc, oc, mode, workspace=ws,
                                  workspace_bytes=ws.numel())
    for replay in range(3):
        dC.copy_(first)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(dC.cpu().numpy(), want), "replay %d" % replay


def _time_of_a_call(gpu, m, n, k, captured, shift=0):
    """us a call, the best of several; shift: elements between a 16-byte boundary and the operands."""
    import torch
    A = torch.zeros(m * k + 8, dtype=torch.int16, device="cuda")[shift:]
    B = torch.zeros(k * n + 8, dtype=torch.int16, device="cuda")[shift:]
    C = torch.zeros(m * n, dtype=torch.int32, device="cuda")
    ws = torch.empty(gpu.mipgemm_workspace_size_s16(m, n, k), dtype=torch.uint8, device="cuda")
    calls = 10

    def body():
        for _ in range(calls):
            gpu.mipgemm_s16s16s32(m, n, k, A, k, 0, B, k, 1, C, n, 0, W.OVERWRITE, workspace=ws,
                                  workspace_bytes=ws.numel())
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        body()
    stream.synchronize()
    if captured:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            body()
        body = graph.replay
    times = []
    with torch.cuda.stream(stream):
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            body()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 1e3 / calls)
    return min(times)


@pytest.mark.parametrize("m,n,k", [(64, 192, 16384), (1, 1024, 16384), (5, 7, 30000)])
def test_s16_few_tiles_keep_their_ranges_of_k(gpu, m, n, k):
    """A few tiles with k whole run on as many compute units, five times as long as in ranges: neither a
    capture nor operands rewritten into the workspace, which leave no room for slots there, may cost them."""
    plain = _time_of_a_call(gpu, m, n, k, False)
    assert _time_of_a_call(gpu, m, n, k, True) < 2.5 * plain
    assert _time_of_a_call(gpu, m, n, k, False, shift=1) < 2.5 * plain


def test_s16_rewritten_operands_of_very_many_blocks(gpu):
    """Two rows of 2^29 + 2 elements: 2^24 blocks of 64 x 64 to rewrite, more threads than one grid holds."""
    import torch
    k = (1 << 29) + 2
    torch.manual_seed(15)
    A = torch.randint(-32768, 32768, (k,), dtype=torch.int16, device="cuda")
    B = torch.randint(-32768, 32768, (k,), dtype=torch.int16, device="cuda")
    want = (A.int() * B.int()).sum(dtype=torch.int64).item()              # every product fits 32 bits
    C = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(gpu.mipgemm_workspace_size_s16(1, 1, k), dtype=torch.uint8, device="cuda")
    gpu.mipgemm_s16s16s32(1, 1, k, A, k, W.ROW_MAJOR, B, k, W.COL_MAJOR, C, 1, W.ROW_MAJOR, W.OVERWRITE,
                          workspace=ws, workspace_bytes=ws.numel())
    assert (C.item() - want) % (1 << 32) == 0


@pytest.mark.parametrize("shape", [(8, 8, 8), (16, 17, 9), (31, 65, 63), (64, 130, 65), (65, 64, 191), (129, 40, 200), (70, 96, 1000)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("mode", [0, 1])
def test_unaligned_operands_read_as_they_are(gpu, shape, mode):
    """Through registers: pieces that an edge of k, m or n cuts, rows beyond it, one to sixteen blocks of k, every order."""
    import torch
    m, n, k = shape
    rng = np.random.default_rng(m + k)
    for oa, ob, oc in ((a, b, c) for a in (0, 1) for b in (0, 1) for c in (0, 1)):
        for pad in (0, 3):
            X, Y = rng.integers(-32768, 32768, (m, k)), rng.integers(-32768, 32768, (k, n))

            def stored(x, order):
                y = x if order == 0 else x.T
                out = np.full((y.shape[0], y.shape[1] + pad), 0x5A5A, dtype=np.int16)
                out[:, :y.shape[1]] = y
                return torch.from_numpy(out).cuda(), y.shape[1] + pad
            (A, lda), (B, ldb) = stored(X, oa), stored(Y, ob)
            C0 = rng.integers(-100, 100, (m, n) if oc == 0 else (n, m)).astype(np.int32)
            S = X @ Y if oc == 0 else (X @ Y).T
            want = (S + (C0 if mode else 0)).astype(np.int64).astype(np.uint32).view(np.int32)
            C = torch.from_numpy(C0).cuda()
            ws = torch.empty(gpu.mipgemm_workspace_size_s16(m, n, k), dtype=torch.uint8, device="cuda")
            with gpu.tuning(MIPGEMM_VARIANT="s16_staged"):
                gpu.mipgemm_s16s16s32(m, n, k, A, lda, oa, B, ldb, ob, C, C0.shape[1], oc, mode, workspace=ws,
                                      workspace_bytes=ws.numel())
            assert np.array_equal(C.cpu().numpy(), want), (oa, ob, oc, pad)


@pytest.mark.parametrize("m,n,k,mode,rewritten", [(10, 10, 14213, 0, True), (10, 10, 14213, 1, True), (10, 10, 4003, 0, False),
                                                  (10, 10, 8001, 1, False), (70, 70, 14213, 0, False), (799, 757, 602, 0, False),
                                                  (1216, 2965, 2153, 0, True)])
def test_which_unaligned_operands_are_rewritten(gpu, kernels_of, m, n, k, mode, rewritten):
    import torch
    A = torch.zeros(m * (k + 1), dtype=torch.int16, device="cuda")
    B = torch.zeros(n * (k + 1), dtype=torch.int16, device="cuda")
    C = torch.zeros(m * n, dtype=torch.int32, device="cuda")
    size = gpu.mipgemm_workspace_size_s16(m, n, k)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    names = kernels_of(lambda: gpu.mipgemm_s16s16s32(m, n, k, A, k + 1, 0, B, k + 1, 1, C, n, 0, mode, workspace=ws, workspace_bytes=size))
    assert any("pack16" in x for x in names) == rewritten, names


@pytest.mark.parametrize("m,n,k", [(72, 151, 1289), (6, 7, 4315), (139, 223, 572)])
def test_adding_in_ranges_of_k_from_unaligned_operands(gpu, oracle, m, n, k):
    """The ranges meet in C, whatever room for slots the workspace has."""
    for oa in (0, 1):
        for ob in (0, 1):
            _check(gpu, oracle, m, n, k, oa, ob, 0, 1, 1)
