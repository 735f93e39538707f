// Shared between the files of the C-ABI layer.  Not installed.
#pragma once
#include "../../include/mipgemm.h"
#include "mip_internal.h"

namespace mip {

inline bool order_ok(int o) { return o == MIPGEMM_ROW_MAJOR || o == MIPGEMM_COL_MAJOR; }

// a strided batch of problems of one shape (count 1: a single problem)
struct Batch {
  int64_t count = 1;
  int64_t stride_a = 0, stride_b = 0, stride_c = 0;  // elements between consecutive problems
};

// Fills `out` and returns 0, or returns the negative argument number (numbered as in the
// single-problem GEMM entry points).
int validate_and_normalise(int a_unsigned, int b_unsigned, int64_t m, int64_t n, int64_t k,
                           const void *A, int64_t lda, int orderA, const void *B, int64_t ldb,
                           int orderB, void *C, int64_t ldc, int orderC, int mode,
                           void *workspace, size_t workspace_bytes, Problem *out);

// A batch that shares one operand and steps through the other and through C as one matrix would is one
// product with that many times the rows (or columns): it may be packed, and takes tiles by its whole size.
// (Three products of 1024 x 641 x 1024 with one unaligned B: 18.1 -> 9.5 us.)
inline void fold_batch(Problem *p) {
  const int64_t batch = p->batch;
  if (batch <= 1 || p->m == 0 || p->n == 0 || p->k == 0) return;
  if (p->b_sb == 0 && p->c_sb == p->m * p->ldc && p->m * batch <= MIPGEMM_MAX_DIM &&
      (p->a_sk == 1 ? p->a_sb == p->m * p->a_sm : p->a_sb == p->m && p->a_sk >= p->m * batch)) {
    p->m *= batch;
  } else if (p->a_sb == 0 && p->c_sb == p->n && p->ldc >= p->n * batch && p->n * batch <= MIPGEMM_MAX_DIM &&
             (p->b_sk == 1 ? p->b_sb == p->n * p->b_sn : p->b_sb == p->n && p->b_sk >= p->n * batch)) {
    p->n *= batch;
  } else {
    return;
  }
  p->batch = 1;
  p->a_sb = p->b_sb = p->c_sb = 0;
}

// Bytes of workspace with which this call would take the packed route (operands that the
// direct-to-LDS kernels cannot stream, and a product large enough for packing to pay), else 0.
size_t packed_route_bytes(const Problem &p);

// Enqueues the kernels of a plan.
hipError_t launch_plan(const Problem &p, const Plan &plan, hipStream_t s);

// Validates, plans and launches one GEMM call.  out_float: C holds floats and receives
// float(sum) * scale (the f32 entry points).
int run_gemm(int a_unsigned, int b_unsigned, int out_float, float scale, int64_t m, int64_t n,
             int64_t k, const void *A, int64_t lda, int orderA, const void *B, int64_t ldb,
             int orderB, void *C, int64_t ldc, int orderC, int mode, void *workspace,
             size_t workspace_bytes, void *stream, const Batch &batch = Batch(),
             const int32_t *ksum = nullptr);  // ksum: see Problem::ksum (pre-packed weights)

}  // namespace mip

// Every name that plan_name can give a plan with a kernel, for the tables that put a prefix before it.
#define MIP_FOR_EACH_VARIANT(X)                                                                    \
  X("simple") X("mfma_tile256") X("mfma_tile128") X("mfma_tile64") X("mfma_tile64x256")            \
  X("mfma_tile256x64") X("mfma_tile64x128") X("mfma_tile128x64") X("mfma_dma256") X("mfma_dma128") \
  X("mfma_dma64") X("mfma_dma64x256") X("mfma_dma256x64") X("mfma_dma64x128") X("mfma_dma128x64")  \
  X("mfma_dma256_k128") X("mfma_dma128_k128") X("mfma_dma256_k128_ragged")                         \
  X("mfma_dma128_k128_split") X("mfma_dma256x192_k128") X("mfma_dma192x256_k128")                  \
  X("mfma_dma192_k128") X("mfma_slab16") X("mfma_slab32") X("mfma_slab64")
