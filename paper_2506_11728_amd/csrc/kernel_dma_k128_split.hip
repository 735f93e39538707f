// The kernel with 128-deep k blocks (dma_k128.h) in its general form: ragged m and n on
// unpadded operands, on 256 x 256 or 128 x 128 tiles (those with a side of 192 have files of
// their own); on the latter k may be cut into ranges, for problems whose tiles are too few to occupy the device while k is long: every range of a
// tile is a workgroup of its own, and the ranges add their partial sums into C with integer
// atomics.
#include "dma_k128_general.h"

namespace mip {

bool dma_k128_split_eligible(const Problem &p, bool large) {
  if (p.conv || p.batch != 1 || p.k % KD2 || p.k < KD2) return false;
  const bool a_kc = p.a_sk == 1, b_kc = p.b_sk == 1;
  if (!a_kc && (p.a_sm != 1 || p.m % 16)) return false;  // a strided operand comes in 16-byte chunks
  if (!b_kc && (p.b_sn != 1 || p.n % 16)) return false;
  const int64_t lda = a_kc ? p.a_sm : p.a_sk;
  const int64_t ldb = b_kc ? p.b_sn : p.b_sk;
  if (lda % 16 || ldb % 16) return false;
  if (reinterpret_cast<uintptr_t>(p.A) % 16 || reinterpret_cast<uintptr_t>(p.B) % 16) return false;
  const int64_t side = large ? 256 : 128;
  if (side * lda >= ((int64_t)1 << 31) || side * ldb >= ((int64_t)1 << 31)) return false;
  if (((p.m + side - 1) / side) * ((p.n + side - 1) / side) > ((int64_t)1 << 30)) return false;
  return true;
}

hipError_t launch_dma_k128_split(const Problem &p, int splits, hipStream_t s, Shape shape) {
  switch (shape) {
    case SHAPE_256: return launch_general<256, 256>(p, 1, s);
    case SHAPE_256X192: return launch_dma_k128_256x192(p, s);
    case SHAPE_192X256: return launch_dma_k128_192x256(p, s);
    case SHAPE_192: return launch_dma_k128_192x192(p, s);
    default: return launch_general<128, 128>(p, splits, s);
  }
}

}  // namespace mip
