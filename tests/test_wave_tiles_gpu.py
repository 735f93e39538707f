"""GPU parity of the tiles whose waves split k, pinned one form at a time (MIPGEMM_VARIANT), on the sizes where
such a tile can go wrong: the edges of tiles, steps of 128 that k ends in, fewer steps than waves, more
than one round of them; every storage order, signedness, output type and mode; aligned operands (direct
loads) and unaligned ones (through registers).  Whole-number results are compared bit for bit."""
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


# (m, n, k, pad): pad 0 or 16 with everything else aligned takes direct loads, the rest goes through registers
ALIGNED = [(16, 16, 64, 0), (48, 80, 192, 16), (32, 64, 1024, 0), (64, 32, 1088, 0), (80, 144, 2112, 0), (208, 272, 128, 16)]
UNALIGNED = [(16, 16, 16, 1), (17, 33, 127, 0), (31, 65, 129, 17), (33, 64, 1000, 0), (65, 130, 1027, 0), (96, 81, 2064, 3)]


def _operands(m, n, k, oa, ob, pad, au, bu, seed):
    rng = np.random.default_rng(seed)
    low, high = {True: (0, 256), False: (-128, 128)}, np.int64
    A, B = rng.integers(*low[au], (m, k), dtype=high), rng.integers(*low[bu], (k, n), dtype=high)

    def stored(x, order):
        y = x if order == 0 else x.T
        out = np.full((y.shape[0], y.shape[1] + pad), W.SENTINEL_BYTE, dtype=np.uint8)
        out[:, :y.shape[1]] = y.astype(np.uint8)
        return out
    return A @ B, stored(A, oa), stored(B, ob)


@pytest.mark.parametrize("shape", ALIGNED + UNALIGNED, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("variant", ["wave32", "wave32x64"])
def test_every_order_type_and_mode(gpu, variant, shape):
    import torch
    m, n, k, pad = shape
    for at, (oa, ob, kind) in enumerate((oa, ob, kind) for oa in (0, 1) for ob in (0, 1) for kind in ("ss", "us", "su")):
        au, bu = kind[0] == "u", kind[1] == "u"
        S, A, B = _operands(m, n, k, oa, ob, pad, au, bu, at)
        dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
        for out, mode in (("s32", 0), ("s32", 1), ("f32", 0), ("f32", 1), ("s8", 0)):
            scale = np.float32(40.0 / (np.abs(S).max() + 1))
            C0 = np.random.default_rng(at).integers(-100, 100, (m, n + 5)).astype({"s32": np.int32, "f32": np.float32, "s8": np.int8}[out])
            want = C0.copy()
            if out == "s32":
                want[:, :n] = (S + (C0[:, :n] if mode else 0)).astype(np.int32)
            elif out == "f32":
                want[:, :n] = S.astype(np.float32) * scale
            else:
                want[:, :n] = np.clip(np.rint(S.astype(np.float32) * scale), -128, 127).astype(np.int8)
            dC = torch.from_numpy(C0.copy()).cuda()
            more = {} if out == "s32" else {"scale": float(scale)}
            with gpu.tuning(MIPGEMM_VARIANT=variant):
                getattr(gpu, "mipgemm_%s8%s8%s" % (kind[0], kind[1], out))(
                    m, n, k, dA, A.shape[1], oa, dB, B.shape[1], ob, dC, n + 5, 0, mode, **more)
            got = dC.cpu().numpy()
            if out == "f32" and mode:       # one rounding of the sum, one of the fused multiply-add
                exact = S * float(scale) + C0[:, :n]
                assert (np.abs(got[:, :n] - exact) <= 2.0 ** -23 * (np.abs(exact) + np.abs(C0[:, :n]) + np.abs(S * float(scale)))).all()
                got[:, :n] = want[:, :n]
            assert np.array_equal(got, want), (oa, ob, kind, out, mode)


@pytest.mark.parametrize("variant", ["wave32", "wave32x64"])
@pytest.mark.parametrize("pad", [0, 1])
def test_batches(gpu, variant, pad):
    import torch
    m, n, k, batch = 48, 80, 320, 3
    parts = [_operands(m, n, k, 1, 0, pad, False, True, 50 + z) for z in range(batch)]
    dA, dB = (torch.from_numpy(np.stack([p[i] for p in parts])).cuda() for i in (1, 2))
    C = torch.full((batch, m, n), 7, dtype=torch.int32, device="cuda")
    with gpu.tuning(MIPGEMM_VARIANT=variant):
        gpu.mipgemm_s8u8s32_batched(m, n, k, dA, m + pad, 1, k * (m + pad), dB, n + pad, 0, k * (n + pad), C, n, 0, m * n,
                                    batch, 1)
    assert np.array_equal(C.cpu().numpy(), np.stack([p[0] for p in parts]) + 7)


@pytest.mark.parametrize("variant", ["wave32", "wave32x64"])
@pytest.mark.parametrize("shape", [(2, 9, 11, 64, 48, 3, 3, 1, 1), (1, 17, 23, 64, 96, 3, 5, 2, 2), (3, 7, 7, 192, 80, 3, 3, 1, 1),
                                   (2, 14, 14, 128, 64, 1, 1, 2, 0)], ids=lambda s: "x".join(map(str, s)))
def test_convolutions(gpu, oracle, variant, shape):
    """Steps of 128 that hold two filter taps (64 channels, 192), taps outside the image, strides; with and without filter sums."""
    import torch
    b, hi, wi, ci, co, hf, wf, stride, pad = shape
    rng = np.random.default_rng(9)
    image = rng.integers(0, 256, (b, hi, wi, ci), dtype=np.uint8)
    filters = rng.integers(-128, 128, (co, hf, wf, ci), dtype=np.int8)
    want = oracle.conv_direct(image, filters, stride, pad)
    dI, dF = torch.from_numpy(image).cuda(), torch.from_numpy(filters.view(np.uint8)).cuda()
    sums = torch.from_numpy(filters.reshape(co, -1).sum(axis=1, dtype=np.int32)).cuda()
    for given in (False, True):
        dO = torch.full(want.shape, 5, dtype=torch.int32, device="cuda")
        with gpu.tuning(MIPGEMM_VARIANT=variant):
            fn, extra = (gpu.mipgemm_conv_s8u8s32_with_sums, (sums,)) if given else (gpu.mipgemm_conv_s8u8s32, ())
            fn(b, hi, wi, ci, co, hf, wf, stride, pad, dF, dI, dO, 1, *extra)
        assert np.array_equal(dO.cpu().numpy(), want + 5), given


def test_packed_weights_bring_their_sums(gpu):
    import torch
    m, n, k = 70, 100, 1100
    S, A, B = _operands(m, n, k, 0, 0, 0, True, False, 77)
    packed = torch.empty(gpu.mipgemm_packed_weights_bytes(k, n), dtype=torch.uint8, device="cuda")
    gpu.mipgemm_pack_weights(k, n, torch.from_numpy(B).cuda(), n, 0, packed)
    pitch = (k + 127) // 128 * 128
    Ap = np.zeros((m, pitch), dtype=np.uint8)
    Ap[:, :k] = A
    for order, shape in ((0, (m, n)), (1, (n, m))):
        C = torch.zeros(shape, dtype=torch.int32, device="cuda")
        with gpu.tuning(MIPGEMM_VARIANT="wave32"):
            gpu.mipgemm_u8s8s32_packed(m, n, k, torch.from_numpy(Ap).cuda(), pitch, 0, packed, C, shape[1], order, 0)
        got = C.cpu().numpy()
        assert np.array_equal(got if order == 0 else got.T, S)


def test_what_the_dispatcher_sends_there(gpu):
    """Few tiles, at both ends of a rule: the results of a call as dispatched, beside the one-thread-per-element kernel."""
    import torch
    for m, n, k, out in ((512, 512, 1024, "s32"), (256, 1024, 4096, "f32"), (70, 1024, 700, "s32"), (459, 500, 836, "s8"),
                         (1024, 512, 2048, "s32"), (1568, 512, 2432, "s8")):
        rng = np.random.default_rng(m)
        A = torch.from_numpy(rng.integers(-128, 128, (m, k), dtype=np.int8)).cuda()
        B = torch.from_numpy(rng.integers(-128, 128, (n, k), dtype=np.int8)).cuda()
        kind = {"s32": torch.int32, "f32": torch.float32, "s8": torch.int8}[out]
        results = []
        for variant in (None, "simple"):
            C = torch.zeros((m, n), dtype=kind, device="cuda")
            with gpu.tuning(MIPGEMM_VARIANT=variant):
                getattr(gpu, "mipgemm_s8s8" + out)(m, n, k, A, k, 0, B, k, 1, C, n, 0, 0, **({} if out == "s32" else {"scale": 0.0005}))
            results.append(C.cpu())
        assert torch.equal(*results), (m, n, k, out)


# (m, n, k, accumulate, pad, whether this form serves): both sides of the limits of k, which are the lower the fewer rows and
# tiles there are, lower still for a call that adds into C
@pytest.mark.parametrize("m,n,k,mode,pad,served", [
    (512, 512, 2048, 0, 0, True), (14, 512, 4096, 0, 0, True), (14, 512, 11136, 0, 0, False), (64, 512, 8192, 0, 0, True),
    (64, 1152, 53696, 0, 0, False), (206, 32, 1536, 1, 0, True), (206, 32, 3584, 1, 0, False), (512, 512, 3584, 1, 0, True),
    (40, 50, 900, 1, 1, True), (40, 50, 1200, 1, 1, False), (40, 50, 2900, 0, 1, True), (40, 50, 3500, 0, 1, False)])
def test_which_products_the_dispatcher_sends_there(gpu, kernels_of, m, n, k, mode, pad, served):
    import torch
    A = torch.zeros((m, k + pad), dtype=torch.int8, device="cuda")
    B = torch.zeros((n, k + pad), dtype=torch.int8, device="cuda")
    C = torch.zeros((m, n), dtype=torch.int32, device="cuda")
    names = kernels_of(lambda: gpu.mipgemm_s8s8s32(m, n, k, A, k + pad, 0, B, k + pad, 1, C, n, 0, mode))
    assert any("wave_tile_kernel" in x for x in names) == served, names


@pytest.mark.parametrize("m,n,k,batch,mode,served", [
    (357, 64, 64, 21, 0, False), (357, 64, 320, 21, 0, True), (357, 64, 320, 21, 1, False), (16, 16, 64, 44, 0, False),
    (16, 16, 96, 44, 0, True)])
def test_which_batches_the_dispatcher_sends_there(gpu, kernels_of, m, n, k, batch, mode, served):
    import torch
    A = torch.zeros((batch, m, k + 1), dtype=torch.int8, device="cuda")
    B = torch.zeros((batch, n, k + 1), dtype=torch.int8, device="cuda")
    C = torch.zeros((batch, m, n), dtype=torch.int32, device="cuda")
    names = kernels_of(lambda: gpu.mipgemm_s8s8s32_batched(m, n, k, A, k + 1, 0, m * (k + 1), B, k + 1, 1, n * (k + 1), C, n, 0,
                                                           m * n, batch, mode))
    assert any("wave_tile_kernel" in x for x in names) == served, names


@pytest.mark.parametrize("shape,served", [((8, 7, 7, 512, 512, 3, 3, 1, 1), True), ((22, 7, 16, 448, 7, 11, 11, 4, 5), False)])
def test_which_convolutions_the_dispatcher_sends_there(gpu, kernels_of, shape, served):
    import torch
    b, hi, wi, ci, co, hf, wf, stride, pad = shape
    I = torch.zeros(b * hi * wi * ci, dtype=torch.uint8, device="cuda")
    F = torch.zeros(co * hf * wf * ci, dtype=torch.int8, device="cuda")
    O = torch.zeros(b * ((hi + 2 * pad - hf) // stride + 1) * ((wi + 2 * pad - wf) // stride + 1) * co, dtype=torch.int32, device="cuda")
    names = kernels_of(lambda: gpu.mipgemm_conv_s8u8s32(*shape, F, I, O, 0))
    assert any("wave_tile_kernel" in x for x in names) == served, names


# (m, n, k, signs, orders of A and B, accumulate, whether this form serves), unaligned rows, no workspace: the limits are lower where
# every strided operand is made of whole 16-byte pieces, and two or three rounds of these tiles stand beside one of 64 x 64 ones
@pytest.mark.parametrize("m,n,k,signs,oa,ob,mode,served", [
    (8, 624, 1900, "s8u8", 0, 0, 0, True), (8, 624, 2500, "s8s8", 0, 0, 0, False), (8, 625, 2500, "s8s8", 0, 0, 0, True),
    (32, 384, 700, "s8u8", 0, 0, 1, True), (32, 384, 900, "s8u8", 0, 0, 1, False), (32, 381, 900, "s8u8", 0, 0, 1, True),
    (128, 1024, 1424, "s8u8", 0, 0, 1, True), (512, 640, 3097, "s8s8", 1, 0, 1, False), (512, 640, 3097, "s8s8", 1, 0, 0, True),
    (512, 640, 3097, "s8s8", 0, 0, 1, False), (512, 633, 3097, "s8s8", 1, 0, 1, True), (512, 1152, 640, "u8s8", 1, 0, 0, False),
    (512, 1152, 2100, "u8s8", 1, 0, 0, True), (512, 1152, 640, "s8s8", 0, 0, 0, True), (512, 1150, 640, "u8s8", 0, 0, 0, True)])
def test_which_unaligned_products_the_dispatcher_sends_there(gpu, kernels_of, m, n, k, signs, oa, ob, mode, served):
    import torch
    lda, ldb = (m if oa else k) + 3, (k if ob else n) + 3
    A = torch.zeros(((k if oa else m), lda), dtype=torch.uint8, device="cuda")
    B = torch.zeros(((n if ob else k), ldb), dtype=torch.uint8, device="cuda")
    C = torch.zeros((m, n), dtype=torch.int32, device="cuda")
    names = kernels_of(lambda: getattr(gpu, "mipgemm_%ss32" % signs)(m, n, k, A, lda, oa, B, ldb, ob, C, n, 0, mode))
    assert any("wave_tile_kernel" in x for x in names) == served, names
