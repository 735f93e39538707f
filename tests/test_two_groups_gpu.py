"""GPU parity of the 64-deep tiles on which two groups of waves share blocks of 128 k, at the sizes where that form can go wrong:
numbers of blocks around its three or four LDS stages, ragged tiles, operands as stored in every order, sums supplied and not,
batches, gathered convolutions.  The kernel that served a call is asserted by its name: its last template argument is the
number of groups.  Whole-number results are compared bit for bit."""
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


TILES = {"dma64": "64, 64", "dma64x128": "64, 128", "dma128x64": "128, 64"}


def _groups(names, variant):
    found = [x for x in names if "dma_tile_kernel<%s," % TILES[variant] in x]
    assert len(found) == 1, names
    return int(found[0].split("dma_tile_kernel<")[1].split(">")[0].split(",")[-1])


def _operand(rng, rows, cols, order, unsigned):
    values = rng.integers(0, 256, (rows, cols)) if unsigned else rng.integers(-128, 128, (rows, cols))
    stored = np.ascontiguousarray(values if order == 0 else values.T).astype(np.uint8)
    return values.astype(np.float64), stored


def _finished(S, C0, out, mode, scale):
    """The result in the output's type; sums of fewer than 2^24 steps of bytes are whole numbers in float64."""
    if out == "s32":
        return (S + (C0 if mode else 0)).astype(np.int32)
    if out == "f32":
        return S.astype(np.float32) * np.float32(scale)
    return np.clip(np.rint(S.astype(np.float32) * np.float32(scale)), -128, 127).astype(np.int8)


# k: numbers of 128-deep blocks that leave each remainder by the stages (four on 64 x 64 tiles, three on the wider ones)
@pytest.mark.parametrize("variant,k", [("dma64", 768), ("dma64", 896), ("dma64", 1024), ("dma64", 1152), ("dma64x128", 1536),
                                       ("dma64x128", 1664), ("dma64x128", 1792), ("dma128x64", 1536), ("dma128x64", 1664),
                                       ("dma128x64", 1792)])
@pytest.mark.parametrize("m,n", [(64, 128), (80, 144), (208, 16), (16, 272)])
def test_every_order_type_and_mode(gpu, kernels_of, variant, k, m, n):
    import torch
    outs = (("s32", 0), ("s32", 1), ("f32", 0), ("s8", 0))
    for at, (oa, ob, kind) in enumerate((a, b, s) for a in (0, 1) for b in (0, 1) for s in ("s8s8", "u8s8", "s8u8")):
        rng = np.random.default_rng(at)
        va, A = _operand(rng, m, k, oa, kind[0] == "u")
        vb, B = _operand(rng, k, n, ob, kind[2] == "u")
        S = va @ vb
        scale = float(np.float32(40.0 / (np.abs(S).max() + 1)))
        dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
        for out, mode in outs:
            C0 = rng.integers(-100, 100, (m, n)).astype({"s32": np.int32, "f32": np.float32, "s8": np.int8}[out])
            C = torch.from_numpy(C0).cuda()
            more = {} if out == "s32" else {"scale": scale}

            def call():
                getattr(gpu, "mipgemm_" + kind + out)(m, n, k, dA, A.shape[1], oa, dB, B.shape[1], ob, C, n, 0, mode, **more)
            with gpu.tuning(MIPGEMM_VARIANT=variant, MIPGEMM_SPLITK="1"):
                call()
                assert np.array_equal(C.cpu().numpy(), _finished(S, C0, out, mode, scale)), (oa, ob, kind, out, mode)
                if at == 0 and mode == 0:
                    assert _groups(kernels_of(call), variant) == 2


# (variant, m, n, k, orders of A and B, groups): both sides of the rule on sizes
@pytest.mark.parametrize("variant,m,n,k,oa,ob,groups", [
    ("dma64", 512, 512, 768, 0, 0, 2), ("dma64", 512, 512, 640, 0, 0, 1), ("dma64", 512, 512, 832, 0, 0, 1),
    ("dma64", 1024, 1088, 2304, 0, 1, 2), ("dma64", 1024, 1088, 2176, 0, 1, 1), ("dma64", 2112, 1024, 2304, 0, 1, 1),
    ("dma64x128", 512, 512, 1024, 0, 1, 2), ("dma64x128", 512, 512, 896, 0, 1, 1), ("dma64x128", 512, 512, 1408, 0, 0, 1),
    ("dma128x64", 512, 512, 1536, 1, 0, 2), ("dma128x64", 2112, 1024, 1536, 0, 1, 1)])
def test_which_products_two_groups_serve(gpu, kernels_of, variant, m, n, k, oa, ob, groups):
    import torch
    A, B = (torch.zeros(rows * k, dtype=torch.int8, device="cuda") for rows in (m, n))
    C = torch.zeros((m, n), dtype=torch.int32, device="cuda")
    with gpu.tuning(MIPGEMM_VARIANT=variant, MIPGEMM_SPLITK="1"):
        names = kernels_of(lambda: gpu.mipgemm_s8s8s32(m, n, k, A, m if oa else k, oa, B, k if ob else n, ob, C, n, 0, 0))
    assert _groups(names, variant) == groups, names


@pytest.mark.parametrize("variant,k", [("dma64", 1152), ("dma64x128", 1664), ("dma128x64", 1792)])
def test_sums_that_packed_weights_bring(gpu, kernels_of, variant, k):
    """The second group adds none of them; a column-major C swaps the operands, and with them whose sums these are."""
    import torch
    m, n = 96, 208
    rng = np.random.default_rng(3)
    vb, B = _operand(rng, k, n, 0, False)
    packed = torch.empty(gpu.mipgemm_packed_weights_bytes(k, n), dtype=torch.uint8, device="cuda")
    gpu.mipgemm_pack_weights(k, n, torch.from_numpy(B).cuda(), n, 0, packed)
    va, A = _operand(rng, m, k, 0, True)
    S, dA = va @ vb, torch.from_numpy(A).cuda()
    for order, shape in ((0, (m, n)), (1, (n, m))):
        for mode in (0, 1):
            C = torch.full(shape, 9, dtype=torch.int32, device="cuda")

            def call():
                gpu.mipgemm_u8s8s32_packed(m, n, k, dA, k, 0, packed, C, shape[1], order, mode)
            with gpu.tuning(MIPGEMM_VARIANT=variant, MIPGEMM_SPLITK="1"):
                call()
                got = C.cpu().numpy()
                assert np.array_equal(got if order == 0 else got.T, S + 9 * mode), (order, mode)
                name = [x for x in kernels_of(call) if "dma_tile_kernel" in x][0]
            args = name.split("dma_tile_kernel<")[1].split(">")[0].split(", ")
            assert args[-1] == "2" and args[4] == ("3" if order == 0 else "4"), name


def test_batches(gpu, kernels_of):
    import torch
    m, n, k, batch = 80, 112, 896, 5
    for at, (oa, ob, kind) in enumerate((a, b, s) for a in (0, 1) for b in (0, 1) for s in ("s8s8", "u8s8", "s8u8")):
        rng = np.random.default_rng(at)
        parts = [(_operand(rng, m, k, oa, kind[0] == "u"), _operand(rng, k, n, ob, kind[2] == "u")) for _ in range(batch)]
        dA, dB = (torch.from_numpy(np.stack([p[i][1] for p in parts])).cuda() for i in (0, 1))
        C = torch.zeros((batch, m, n), dtype=torch.int32, device="cuda")

        def call():
            getattr(gpu, "mipgemm_%ss32_batched" % kind)(m, n, k, dA, m if oa else k, oa, m * k, dB, k if ob else n, ob, k * n, C, n, 0,
                                                         m * n, batch, W.OVERWRITE)
        with gpu.tuning(MIPGEMM_VARIANT="dma64", MIPGEMM_SPLITK="1"):
            call()
            assert np.array_equal(C.cpu().numpy(), np.stack([a @ b for (a, _), (b, _) in parts])), (oa, ob, kind)
            if at == 0:
                assert _groups(kernels_of(call), "dma64") == 2


@pytest.mark.parametrize("variant", sorted(TILES))
@pytest.mark.parametrize("shape,groups", [((2, 9, 11, 128, 48, 3, 3, 1, 1), 2), ((1, 17, 23, 256, 80, 3, 5, 2, 2), 2),
                                          ((3, 7, 7, 384, 144, 2, 2, 1, 0), 2), ((2, 9, 11, 192, 48, 3, 3, 1, 1), 1)])
def test_convolutions(gpu, oracle, kernels_of, variant, shape, groups):
    """Channels in whole blocks of 128 (a block holds one filter tap) and not; with and without filter sums."""
    import torch
    b, hi, wi, ci, co, hf, wf, stride, pad = shape
    rng = np.random.default_rng(9)
    image = rng.integers(0, 256, (b, hi, wi, ci), dtype=np.uint8)
    filters = rng.integers(-128, 128, (co, hf, wf, ci), dtype=np.int8)
    want = oracle.conv_direct(image, filters, stride, pad)
    dI, dF = torch.from_numpy(image).cuda(), torch.from_numpy(filters.view(np.uint8)).cuda()
    sums = torch.from_numpy(filters.reshape(co, -1).sum(axis=1, dtype=np.int32)).cuda()
    for given in (False, True):
        fn, extra = (gpu.mipgemm_conv_s8u8s32_with_sums, (sums,)) if given else (gpu.mipgemm_conv_s8u8s32, ())
        dO = torch.full(want.shape, 5, dtype=torch.int32, device="cuda")

        def call():
            fn(b, hi, wi, ci, co, hf, wf, stride, pad, dF, dI, dO, W.ACCUMULATE, *extra)
        with gpu.tuning(MIPGEMM_VARIANT=variant, MIPGEMM_SPLITK="1"):
            call()
            assert np.array_equal(dO.cpu().numpy(), want + 5), given
            assert _groups(kernels_of(call), variant) == groups
