// Launcher of the kernel with 128-deep k blocks (dma_k128.h) in its general form, shared by the
// files that instantiate it, one per tile shape.
#pragma once
#include "dma_k128.h"

namespace mip {

namespace {

template <int BM, int BN>
hipError_t launch_general(const Problem &p, int splits, hipStream_t s) {
  DmaParams P;
  P.clocks = nullptr;
  P.A = static_cast<const uint8_t *>(p.A);
  P.B = static_cast<const uint8_t *>(p.B);
  P.C = p.C;
  P.lda = p.a_sk == 1 ? p.a_sm : p.a_sk;
  P.ldb = p.b_sk == 1 ? p.b_sn : p.b_sk;
  P.ldc = p.ldc;
  P.m = p.m;
  P.n = p.n;
  P.walk = tile_walk((p.m + BM - 1) / BM, (p.n + BN - 1) / BN);
  P.nkt = (int)(p.k / KD2);
  // k ranges on the small tile only, and only into an int32 C (float sums must not be combined
  // in arbitrary order, and an int8 C holds no partial sums)
  if (splits < 1 || BM != 128 || p.out_float) splits = 1;
  if (splits > P.nkt) splits = P.nkt;       // every range holds at least one block
  if (splits > 65535) splits = 65535;
  P.per_range = P.nkt / splits;
  P.longer = P.nkt % splits;
  P.atomic = splits > 1;
  P.accumulate = p.accumulate;
  P.out_float = p.out_float;
  P.scale = p.scale;
  P.ksum = nullptr;
  const int ntiles = P.walk.tiles_m * P.walk.tiles_n;
  P.first_round = (int)compute_units();
  // (the large tile's rows of an XCD's patch start apart, as in the form for whole tiles)
  P.stagger_ticks = BM != 128 && ntiles >= 2 * P.first_round ? STAGGER_TICKS : 0;
  if (P.atomic && !p.accumulate) {
    hipError_t e = launch_fill_zero(p, s);  // partial sums are added into C: start from zero
    if (e != hipSuccess) return e;
  }
  dim3 grid((unsigned)(((ntiles + 7) / 8) * 8), (unsigned)splits);
  const size_t lds = (size_t)Tile16<BM, BN>::LDS_BYTES;
  const bool a_kc = p.a_sk == 1, b_kc = p.b_sk == 1;
  const int uns = p.a_unsigned ? 1 : (p.b_unsigned ? 2 : 0);
  void (*kern)(DmaParams) = nullptr;
#define MIP_PICK(AK, BKC)                                                                     \
  kern = uns == 0 ? dma128_kernel<BM, BN, AK, BKC, 0, true, true>                             \
                  : (uns == 1 ? dma128_kernel<BM, BN, AK, BKC, 1, true, true>                 \
                              : dma128_kernel<BM, BN, AK, BKC, 2, true, true>)
  if (a_kc && b_kc) MIP_PICK(true, true);
  else if (a_kc) MIP_PICK(true, false);
  else if (b_kc) MIP_PICK(false, true);
  else MIP_PICK(false, false);
#undef MIP_PICK
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds);
  if (e != hipSuccess) return e;
  return launch_with(reinterpret_cast<const void *>(kern), grid, NTHREADS, lds, s, &P);
}

}  // namespace

}  // namespace mip
