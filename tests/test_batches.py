"""Batches that share one operand and run as one product: that the rewritten product reads and writes, for every element of
C, what the batch does (on the CPU, every form up to a few rows, columns and problems), and the results of the entry
points on both sides of the rule, in every storage order, signedness and mode."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W

CHECK = r"""
#include "api_internal.h"
#include <cstdio>
#include <map>
#include <set>
#include <utility>
#include <vector>
using mip::Problem;
// offset in C -> the offsets in A and B whose products it sums; false where two elements of C are one
typedef std::map<int64_t, std::vector<std::pair<int64_t, int64_t>>> Sums;
static bool sums_of(const Problem &p, Sums *out) {
  for (int64_t z = 0; z < p.batch; ++z)
    for (int64_t i = 0; i < p.m; ++i)
      for (int64_t j = 0; j < p.n; ++j) {
        auto &sum = (*out)[z * p.c_sb + i * p.ldc + j];
        if (!sum.empty()) return false;
        for (int64_t q = 0; q < p.k; ++q)
          sum.emplace_back(z * p.a_sb + i * p.a_sm + q * p.a_sk, z * p.b_sb + q * p.b_sk + j * p.b_sn);
      }
  return true;
}
int main() {
  long forms = 0, rows[2] = {0, 0}, columns[2] = {0, 0}, wrong = 0;
  for (int64_t m = 1; m <= 3; ++m) for (int64_t n = 1; n <= 3; ++n) for (int64_t k = 1; k <= 3; ++k)
  for (int64_t batch = 1; batch <= 3; ++batch)
  for (int kc = 0; kc < 4; ++kc) for (int64_t pad = 0; pad < 3; ++pad) for (int64_t c_pad = 0; c_pad < 3; ++c_pad) {
    const bool a_kc = kc & 1, b_kc = kc & 2;
    // leading dimensions of one problem's matrix and of the whole batch's, a little more than either
    const std::set<int64_t> ldas = {(a_kc ? k : m) + pad, (a_kc ? k : m * batch) + pad}, ldbs = {(b_kc ? k : n) + pad, (b_kc ? k : n * batch) + pad},
                            ldcs = {n + c_pad, n * batch + c_pad};
    for (int64_t lda : ldas) for (int64_t ldb : ldbs) for (int64_t ldc : ldcs) {
      Problem p;
      p.m = m; p.n = n; p.k = k; p.batch = batch;
      p.a_sm = a_kc ? lda : 1; p.a_sk = a_kc ? 1 : lda; p.b_sn = b_kc ? ldb : 1; p.b_sk = b_kc ? 1 : ldb; p.ldc = ldc;
      // strides that continue the matrix one way or the other, and their neighbours
      const std::set<int64_t> as = {0, 1, m - 1, m, m + 1, m * lda - 1, m * lda, m * lda + 1, k * lda},
                              bs = {0, 1, n - 1, n, n + 1, n * ldb - 1, n * ldb, n * ldb + 1, k * ldb},
                              cs = {n - 1, n, n + 1, m * ldc - 1, m * ldc, m * ldc + 1};
      for (int64_t a : as) for (int64_t b : bs) for (int64_t c : cs) {
        p.a_sb = a; p.b_sb = b; p.c_sb = c;
        Problem q = p;
        mip::fold_batch(&q);
        ++forms;
        if (q.batch == p.batch && q.m == p.m && q.n == p.n) continue;
        Sums before, after;
        if (!sums_of(p, &before)) continue;  // (slices of C that overlap: not allowed)
        if (q.batch != 1 || !sums_of(q, &after) || before != after) ++wrong;
        if (q.m != p.m) ++rows[a_kc];
        else ++columns[b_kc];
      }
    }
  }
  std::printf("%d %d %d %d %d %ld", forms > 100000, rows[0] > 50, rows[1] > 50, columns[0] > 50, columns[1] > 50, wrong);
}
"""


def test_a_folded_batch_is_the_same_sums(tmp_path):
    from paper_2506_11728_amd import build
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("nothing to build it with")
    (tmp_path / "check.cpp").write_text(CHECK)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(build.HERE, "csrc"),
                    str(tmp_path / "check.cpp"), "-o", str(tmp_path / "check")], check=True, timeout=120)
    assert subprocess.run([str(tmp_path / "check")], capture_output=True, text=True, timeout=120).stdout == "1 1 1 1 1 0"


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_11728_amd as M
    M.load_library()
    return M


def _layout(batch, rows, cols, order, along, pad, off):
    """A batch of rows x cols matrices that are the row blocks (along = 0) or column blocks (1) of one matrix: leading dimension,
    stride between them (`off` elements more than that) and the index of every element (z, i, j) in the flat buffer."""
    whole = (rows * batch, cols) if along == 0 else (rows, cols * batch)
    ld = whole[1 - order] + pad
    stride = (cols if along else rows) * (1 if along != order else ld) + off
    z, i, j = np.ogrid[:batch, :rows, :cols]
    return ld, stride, z * stride + (i * ld + j if order == 0 else j * ld + i)


@pytest.mark.gpu
@pytest.mark.parametrize("off", ["none", "other", "C"])  # which operand's stride misses the rule by a few elements
@pytest.mark.parametrize("shape", [(48, 80, 192, 3, 0), (40, 24, 65, 5, 1), (1, 33, 130, 4, 3), (130, 1, 64, 2, 16)],
                         ids=lambda s: "x".join(map(str, s)))
def test_batches_that_share_an_operand(gpu, shape, off):
    import torch
    m, n, k, batch, pad = shape
    for at, (shared, oa, ob, oc, mode) in enumerate((s, a, b, c, d) for s in "AB" for a in (0, 1) for b in (0, 1) for c in (0, 1) for d in (0, 1)):
        signs = ("s8s8", "u8s8", "s8u8")[at % 3]
        rng = np.random.default_rng(at)

        def operand(rows, cols, order, share, along, unsigned):
            ld, stride, index = _layout(1 if share else batch, rows, cols, order, along, pad, 0 if share or off != "other" else 16)
            flat = rng.integers(0, 256, index.max() + 1, dtype=np.uint8)
            values = flat[index] if unsigned else flat[index].view(np.int8)
            return flat, ld, 0 if share else stride, np.broadcast_to(values, (batch, rows, cols)).astype(np.int64)
        A, lda, sa, va = operand(m, k, oa, shared == "A", 0, signs[0] == "u")
        B, ldb, sb, vb = operand(k, n, ob, shared == "B", 1, signs[2] == "u")
        # (C steps with the operand that is not shared; between the problems of a stacked C only the padding may be skipped)
        ldc, sc, index = _layout(batch, m, n, oc, 0 if shared == "B" else 1, pad + (4 if off == "C" else 0), 2 if off == "C" else 0)
        if off == "C":
            sc += index.max() + 1  # far enough apart for any order
            index = index + np.arange(batch)[:, None, None] * (index.max() + 1)
        C = rng.integers(-1000, 1000, index.max() + 9, dtype=np.int32)
        want = C.copy()
        want[index] = va @ vb + (C[index] if mode else 0)
        dA, dB, dC = (torch.from_numpy(x).cuda() for x in (A, B, C))
        getattr(gpu, "mipgemm_%ss32_batched" % signs)(m, n, k, dA, lda, oa, sa, dB, ldb, ob, sb, dC, ldc, oc, sc, batch, mode)
        assert np.array_equal(dC.cpu().numpy(), want), (shared, oa, ob, oc, mode, signs)  # what lies between the slices included


@pytest.mark.gpu
@pytest.mark.parametrize("apart,packed", [(0, True), (1, False)])
def test_a_folded_batch_is_packed(gpu, kernels_of, apart, packed):
    """Three unaligned products with one B: one product of three times the rows, packed into a workspace of its size."""
    import torch
    m, n, k, batch = 256, 641, 1024, 3
    rng = np.random.default_rng(5)
    A, B = rng.integers(-128, 128, (batch, m, k), dtype=np.int8), rng.integers(-128, 128, (k, n), dtype=np.int8)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    C = torch.full((batch, m * n + apart), 7, dtype=torch.int32, device="cuda")
    size = gpu.mipgemm_workspace_size(batch * m, n, k, 0, 0, 0)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    names = kernels_of(lambda: gpu.mipgemm_s8s8s32_batched(m, n, k, dA, k, 0, m * k, dB, n, 0, 0, C, n, 0, m * n + apart, batch, W.OVERWRITE,
                                                           workspace=ws, workspace_bytes=size))
    assert any("pack_kernel" in x for x in names) == packed, names
    got = C.cpu().numpy()
    assert np.array_equal(got[:, :m * n].reshape(batch, m, n), A.astype(np.float64) @ B.astype(np.float64))
    assert (got[:, m * n:] == 7).all()
