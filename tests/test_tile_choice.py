"""The choice between the tile forms by predicted time: which form a product takes on either side of its lines, and the
results of calls as dispatched, in every order, signedness, output type and mode, beside the kernel that takes one
thread per element of C (itself pinned against the oracle)."""
import numpy as np
import pytest

import paper_2506_11728_amd as M


def _name(m, n, k, oa, ob, au=False):
    return M.mipgemm_variant_name(m, n, k, m if oa else k, oa, k if ob else n, ob, n, 0, au, False)


@pytest.mark.parametrize("shape,name", [
    # one round of 128 x 128 tiles, where 8192-element ones need a second for a few tiles
    ((512, 5760, 6400, 0, 1), "mfma_dma128_k128"),
    ((496, 4432, 3840, 0, 0), "mfma_dma128_k128_split"),
    # k of whole 64-deep blocks only: the 128-deep kernels are out
    ((496, 4432, 3904, 0, 0), "mfma_dma128"),
    # stays: two k-contiguous operands on 64 x 64 tiles, a short k on whole 128 x 128 ones, fewer than 200 tiles
    ((2160, 688, 6656, 0, 1), "mfma_dma64"),
    ((2304, 1536, 512, 0, 1), "mfma_dma128_k128"),
    # stays: whole 256 x 256 tiles in two rounds or less
    ((4608, 4608, 4096, 0, 1), "mfma_dma256_k128"),
])
def test_choice(shape, name):
    assert _name(*shape) == name


@pytest.mark.parametrize("m,n,k,ldc,mode,name", [
    # rows of C that end inside four words: added to by 64-deep tiles, unless k or the tiles are many; overwritten by 128-deep ones
    (2461, 1101, 1664, 1101, 1, "mfma_dma128x64"), (2461, 1101, 1664, 1101, 0, "mfma_dma128_k128_split"),
    (3152, 4321, 640, 4321, 1, "mfma_dma128"), (2816, 2753, 4096, 2753, 1, "mfma_dma128_k128_split"),
    # whole rows, at whatever alignment
    (2464, 1104, 1664, 1104, 1, "mfma_dma128_k128_split"), (3152, 4320, 640, 4324, 1, "mfma_dma128_k128_split"),
    (2816, 2752, 4096, 2753, 1, "mfma_dma128_k128_split")])
def test_choice_by_what_the_edge_of_c_costs(m, n, k, ldc, mode, name):
    assert M.mipgemm_variant_name_for_mode(m, n, k, k, 0, k, 1, ldc, 0, False, False, True, mode) == name


def test_pinned_ranges_keep_the_tiles_that_take_them():
    """A pinned number of k ranges names the 64-deep tiles it is for: forms that do not split k stay out."""
    with M.tuning(MIPGEMM_SPLITK="4"):
        assert _name(512, 5760, 6400, 0, 1) == "mfma_dma64x128"
        assert _name(496, 4432, 3840, 0, 0) == "mfma_dma64x128"


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(496, 1776, 640), (1376, 1584, 1152), (752, 2704, 1600), (416, 2048, 1664), (1371, 1583, 1094)],
                         ids=lambda s: "x".join(map(str, s)))
def test_results_as_dispatched(shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n, k = shape
    rng = np.random.default_rng(m)
    As = {o: torch.from_numpy(rng.integers(0, 256, (m, k) if o == 0 else (k, m), dtype=np.uint8)).cuda() for o in (0, 1)}
    Bs = {o: torch.from_numpy(rng.integers(0, 256, (k, n) if o == 0 else (n, k), dtype=np.uint8)).cuda() for o in (0, 1)}
    for oa in (0, 1):
        for ob in (0, 1):
            for entry in ("s8s8", "u8s8", "s8u8"):
                A = As[oa].view(torch.uint8 if entry[0] == "u" else torch.int8)
                B = Bs[ob].view(torch.uint8 if entry[2] == "u" else torch.int8)
                for out, mode in (("s32", 0), ("s32", 1), ("f32", 0), ("s8", 0)):
                    kind = {"s32": torch.int32, "f32": torch.float32, "s8": torch.int8}[out]
                    size = M.mipgemm_workspace_size if out == "s32" else M.mipgemm_workspace_size_f32
                    bytes_ = size(m, n, k, oa, ob, 0)
                    ws = torch.empty(max(bytes_, 16), dtype=torch.uint8, device="cuda")
                    scale = {} if out == "s32" else {"scale": 0.0005}
                    results = []
                    for variant in (None, "simple"):
                        C = torch.full((m, n), 7, dtype=kind, device="cuda")
                        with M.tuning(MIPGEMM_VARIANT=variant):
                            getattr(M, "mipgemm_" + entry + out)(m, n, k, A, A.shape[1], oa, B, B.shape[1], ob, C, n, 0, mode,
                                                                 workspace=ws, workspace_bytes=bytes_, **scale)
                        results.append(C)
                    assert torch.equal(*results), (shape, oa, ob, entry, out, mode)
