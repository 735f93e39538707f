// The skinny-m kernel (m <= 64: a handful of tokens against a weight matrix).
//
// Such a GEMM is a stream of B through the chip, once: it is bound by memory, not
// by the matrix cores, and there are too few C tiles to give every compute unit
// one.  The tiled kernels answer that by splitting k over workgroups, which costs
// a zero-fill launch and atomic traffic on C.  Here a workgroup instead owns a
// narrow slab of B, 16, 32 or 64 columns wide and all of k deep, so that n / 16
// workgroups exist and nothing is shared between them: one launch, plain stores.
// Inside the workgroup the waves split k (wave w takes the 128-deep
// steps w, w + W, ...), each wave streams its steps through a private ring in LDS with
// direct loads and no workgroup barrier, and the partial sums meet in LDS at the end.  The
// micro-kernel is v_mfma_i32_16x16x64_i8: 16 rows of A are all a skinny problem has, and 16
// columns keep the slab narrow.
//
// What bounds it is how much of B is in flight and in what pieces: a step is 128 deep so that a
// k-contiguous B (and A) comes in whole 128-byte lines, and eight waves keep up to 128 KB of B
// per workgroup on its way.  Against four waves with 64-deep steps (half lines, at most 64 KB in
// flight), us: (1, 4096, 4096) 6.6 -> 6.0 a call, (16, 11008, 4096) 12.5 -> 10.2 (the kernel alone
// 12.3 -> 9.4: 4.9 TB/s), (1, 11008, 4096) 10.9 -> 9.5 (the kernel).  (Loading the fragments
// of a k-contiguous B straight into registers, half lines of sixteen columns at a time, takes
// twice as long: 10.2 -> 21.)
//
// Fragment layout of that instruction (as for the 32 x 32 x 32 form): lane l
// supplies, for row (A) or column (B) l % 16, the 16 bytes k = 16 * (l / 16) ..
// + 15 of the 64-deep half step; in the result lane l holds column l % 16, register v
// holds row 4 * (l / 16) + v.
//
// Preconditions, checked on the host (slab_eligible): 1 <= m <= 64, A stored with
// k contiguous, n a multiple of 16, k a multiple of 64, 16-byte aligned operand
// bases and leading dimensions.
#include "dma_common.h"

namespace mip {

namespace {

// Rings of a workgroup.  DEEP: eight waves (four where A or the slab is wide), together all of a
// compute unit's 160 KB of LDS.  HALF: eight waves and half of it, for more narrow slabs than there are
// compute units.  FEW: four waves, two or three workgroups to a compute unit, for more slabs than that
// with little k, where most of eight waves would have no step, or 64 columns wide.  (1, 32000, 768) on
// 64 columns 8.7 / 5.2 us cold / warm deep, 7.1 / 4.1 few; (4, 15472, 11008) on 16 columns 35.7 / 26.8
// half, 40.9 / 28.2 few.
enum Rings { DEEP, HALF, FEW };
constexpr int slab_waves(int mt, int nt, Rings rings) {
  return rings == FEW || (mt >= 4 && nt >= 2) || (mt == 2 && nt == 4) ? 4 : 8;
}
// steps of A and of B in flight per wave
constexpr int steps_of_a(int mt, int nt, Rings rings) {
  return rings != DEEP ? 2 : mt >= 4 ? (nt == 2 ? 3 : 2) : (nt == 1 ? (mt == 1 ? 4 : 3) : 2);
}
constexpr int steps_of_b(int mt, int nt, Rings rings) {
  return rings != DEEP ? (nt >= 4 ? 2 : (rings == FEW && mt == 1 ? 4 : 3))
         : mt >= 4     ? (nt == 1 ? 2 : 3)
                       : (nt >= 4 ? (mt == 2 ? 3 : 2) : (nt == 2 ? (mt == 2 ? 3 : 4) : (mt == 1 ? 6 : 4)));
}

struct SlabParams {
  const uint8_t *A, *B;
  int32_t *C;
  int64_t lda, ldb, ldc;
  int m;
  int nsteps;      // k / 128, rounded up
  int half_last;   // the last step is 64 deep
  int tiles;       // n / (16 * NT)
  int accumulate;  // C += instead of C =
  int out_float;   // dequantised output: float(sum) * scale
  float scale;
};

template <int N>
__device__ __forceinline__ void loads_landed() {  // all but the N newest direct loads
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// 16 k-contiguous rows of a step in LDS: row r at r * 128, its 16-byte chunk c at
// 16 * (c ^ ((r >> 1) & 7)).  Direct load q fetches eight rows, eight lanes to a row.
__device__ __forceinline__ int kc_chunk(int q, int lane) { return (lane & 7) ^ ((4 * q + (lane >> 4)) & 7); }

// MT: row blocks of 16 (m <= 16 * MT).  NT: column blocks of 16 per workgroup.
// B_KC: B stored with k contiguous (column-major).  UNS: 0 both signed, 1 A
// unsigned, 2 B unsigned.
template <int MT, int NT, bool B_KC, int UNS, Rings RINGS>
__global__ __launch_bounds__(64 * slab_waves(MT, NT, RINGS)) void slab_kernel(SlabParams P) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int W = slab_waves(MT, NT, RINGS), DA = steps_of_a(MT, NT, RINGS), DB = steps_of_b(MT, NT, RINGS);
  static_assert(DB >= DA, "the waits below");
  constexpr int NB = 2 * NT, NA = 2 * MT;           // direct loads of a step
  constexpr int B_STEP = NB * 1024, A_STEP = NA * 1024;  // its bytes
  constexpr int WAVE_BYTES = DB * B_STEP + DA * A_STEP;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // consecutive workgroup ids sit on different XCDs: give each XCD a contiguous run
  // of slabs, so that neighbours, which share cache lines of a row-major B, share an L2
  const int per_xcd = (P.tiles + 7) / 8;
  const int tile = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if ((int)(blockIdx.x / 8) >= per_xcd || tile >= P.tiles) return;
  const int64_t n0 = (int64_t)tile * 16 * NT;
  const int half_step = P.half_last ? P.nsteps - 1 : -1;

  uint8_t *ringB = smem + wave * WAVE_BYTES;
  uint8_t *ringA = ringB + DB * B_STEP;
  const uint32_t ldsB = lds_address(ringB), ldsA = lds_address(ringA);

  // Which 16 bytes each lane fetches.  A row-major B arrives as 128 k rows of 16 * NT bytes and is
  // turned by the transposing LDS read.
  uint32_t offA[NA], offB[NB];
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    int row = 8 * q + (lane >> 3);
    row = row < P.m ? row : P.m - 1;  // rows past m repeat the last one and are never stored
    offA[q] = (uint32_t)(row * P.lda + 16 * kc_chunk(q, lane));
  }
#pragma unroll
  for (int q = 0; q < NB; ++q)
    offB[q] = B_KC ? (uint32_t)((8 * q + (lane >> 3)) * P.ldb + 16 * kc_chunk(q, lane))
                   : (uint32_t)((q * (64 / NT) + lane / NT) * P.ldb + 16 * (lane % NT));
  const uint8_t *baseB = B_KC ? P.B + n0 * P.ldb : P.B + n0;
  const int64_t strideB = B_KC ? 128 : 128 * P.ldb;  // one step further down k

  const int cnt = (P.nsteps + W - 1 - wave) / W;  // steps wave, wave + W, ... below nsteps
  // (the second half of a 64-deep last step is fetched from the first: it exists, and is not used)
  auto issueB = [&](int i) __attribute__((always_inline)) {
    if (i < cnt) {
      const int step = wave + W * i;
      const uint8_t *g = wave_uniform(baseB + (int64_t)step * strideB);
      const uint32_t slot = ldsB + (i % DB) * B_STEP;
      if (step == half_step) {
#pragma unroll
        for (int q = 0; q < NB; ++q)
          dma16(B_KC ? offB[q] - (kc_chunk(q, lane) >= 4 ? 64 : 0) : offB[q >= NT ? q - NT : q], g, slot + q * 1024);
      } else {
#pragma unroll
        for (int q = 0; q < NB; ++q) dma16(offB[q], g, slot + q * 1024);
      }
    }
  };
  auto issueA = [&](int i) __attribute__((always_inline)) {
    if (i < cnt) {
      const int step = wave + W * i;
      const uint8_t *g = wave_uniform(P.A + (int64_t)step * 128);
      const uint32_t slot = ldsA + (i % DA) * A_STEP;
      if (step == half_step) {
#pragma unroll
        for (int q = 0; q < NA; ++q) dma16(offA[q] - (kc_chunk(q, lane) >= 4 ? 64 : 0), g, slot + q * 1024);
      } else {
#pragma unroll
        for (int q = 0; q < NA; ++q) dma16(offA[q], g, slot + q * 1024);
      }
    }
  };

  v4i acc[MT][NT];
  int sumA[MT], sumB[NT];  // k sums of the signed operand (unsigned-operand correction)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    sumA[mt] = 0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = v4i{0, 0, 0, 0};
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) sumB[nt] = 0;

  // The loads go out in one fixed interleaved order, B of step j + DB then A of
  // step j + DA, from j = -DB on.  Loads complete in order, so when step j is to
  // be used, everything issued after its A fragment, i.e. what the DA - 1 iterations since then
  // sent out, may still be in flight and nothing else (near the end fewer loads follow).
  for (int j = -(DB > DA ? DB : DA); j < 0; ++j) {
    if (j + DB >= 0) issueB(j + DB);
    if (j + DA >= 0) issueA(j + DA);
  }
  for (int j = 0; j < cnt; ++j) {
    if (j - 1 + DB < cnt && j - 1 + DA < cnt) loads_landed<(DA - 1) * (NB + NA)>();
    else if (j - 1 + DA < cnt) loads_landed<(DA - 1) * NA>();
    else loads_landed<0>();

    const uint8_t *sa = ringA + (j % DA) * A_STEP;
    const uint8_t *sb = ringB + (j % DB) * B_STEP;
    const bool half = wave + W * j == half_step;
    v4i fa[2][MT], fb[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kc = (lane & 15) * 128 + (((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) << 4);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) fa[h][mt] = *reinterpret_cast<const v4i *>(sa + mt * 2048 + kc);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        if (B_KC) {
          fb[h][nt] = *reinterpret_cast<const v4i *>(sb + nt * 2048 + kc);
        } else {
          // transposing read: in each group of 16 lanes, lane 2t + h names half h of the
          // 16-byte row t and lane i receives byte i of rows 0..7
          const int krow = 64 * h + 16 * (lane >> 4) + ((lane & 15) >> 1);
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const int off = (krow + 8 * r) * (16 * NT) + 16 * nt + 8 * (lane & 1);
            v2i t = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(v2i, sb + off));
            fb[h][nt][2 * r] = t[0];
            fb[h][nt][2 * r + 1] = t[1];
          }
        }
      }
    }
    // the fragments are in registers before the slots they came from are refilled
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issueB(j + DB);
    issueA(j + DA);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && half) break;
      if (UNS == 1) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) fa[h][mt] ^= (int)0x80808080u;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            sumB[nt] = __builtin_amdgcn_sdot4(fb[h][nt][r], 0x01010101, sumB[nt], false);
      }
      if (UNS == 2) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) fb[h][nt] ^= (int)0x80808080u;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            sumA[mt] = __builtin_amdgcn_sdot4(fa[h][mt][r], 0x01010101, sumA[mt], false);
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[h][mt], fb[h][nt], acc[mt][nt], 0, 0, 0);
    }
  }
  loads_landed<0>();

  // unsigned operand: sum (x - 128) y + 128 sum y, each wave for its own share of k
  if (UNS == 1) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      int t = sumB[nt];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);  // every lane: the sum of its own column l % 16
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt][nt] += 128 * t;
    }
  }
  if (UNS == 2) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      int t = sumA[mt];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);  // lane l: the sum of row l % 16
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = 128 * __shfl(t, 4 * (lane >> 4) + v);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt][v] += c;
      }
    }
  }

  // the waves' partial sums meet in LDS, over the rings, once every wave is done with them
  __syncthreads();
  v4i *red = reinterpret_cast<v4i *>(smem);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) red[((wave * MT + mt) * NT + nt) * 64 + lane] = acc[mt][nt];
  __syncthreads();
  const Finish fin{P.scale, P.out_float};
  constexpr int BLOCKS = MT * NT, MINE = (BLOCKS + W - 1) / W;  // blocks of 16 x 16: wave, wave + W, ...
  v4i sums[MINE];
#pragma unroll
  for (int i = 0; i < MINE; ++i) {
    const int b = wave + W * i;
    if (b < BLOCKS) {
      sums[i] = red[b * 64 + lane];
#pragma unroll
      for (int w = 1; w < W; ++w) sums[i] += red[(w * BLOCKS + b) * 64 + lane];
    }
  }
#pragma unroll
  for (int i = 0; i < MINE; ++i) {
    const int b = wave + W * i;
    if (b >= BLOCKS) break;
    const int mt = b / NT, nt = b % NT;
    int32_t *c = P.C + n0 + 16 * nt + (lane & 15);
    // (an accumulating call reads its four old words before the first store, not one behind each)
    int old[4] = {0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * mt + 4 * (lane >> 4) + v;
      if (P.accumulate && row < P.m) old[v] = c[row * P.ldc];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * mt + 4 * (lane >> 4) + v;
      if (row < P.m) c[row * P.ldc] = fin(sums[i][v], old[v], P.accumulate != 0);
    }
  }
}

template <int MT, int NT, Rings RINGS = DEEP>
void (*pick(bool b_kc, int uns))(SlabParams) {
  if (b_kc) return uns == 0 ? slab_kernel<MT, NT, true, 0, RINGS>
                            : (uns == 1 ? slab_kernel<MT, NT, true, 1, RINGS> : slab_kernel<MT, NT, true, 2, RINGS>);
  return uns == 0 ? slab_kernel<MT, NT, false, 0, RINGS>
                  : (uns == 1 ? slab_kernel<MT, NT, false, 1, RINGS> : slab_kernel<MT, NT, false, 2, RINGS>);
}

}  // namespace

bool slab_eligible(const Problem &p, int nt) {
  if (p.conv || p.batch != 1 || p.m < 1 || p.m > 64 || p.a_sk != 1) return false;
  if (p.out_float == 2) return false;  // (no int8 write-back here)
  if (nt != 1 && nt != 2 && nt != 4) return false;
  if (p.n % (16 * nt) || p.k % 64 || p.k < 64) return false;
  if (p.b_sk != 1 && p.b_sn != 1) return false;
  const int64_t lda = p.a_sm, ldb = p.b_sk == 1 ? p.b_sn : p.b_sk;
  if ((p.m > 1 && lda % 16) || ldb % 16) return false;  // a single row of A has no stride
  if (reinterpret_cast<uintptr_t>(p.A) % 16 || reinterpret_cast<uintptr_t>(p.B) % 16) return false;
  if ((p.m > 1 && 64 * lda >= ((int64_t)1 << 31)) || 128 * ldb >= ((int64_t)1 << 31)) return false;
  if (p.n / (16 * nt) >= ((int64_t)1 << 23)) return false;  // x 512 threads stays below 2^32
  return true;
}

hipError_t launch_slab(const Problem &p, int nt, hipStream_t s) {
  SlabParams P;
  P.A = static_cast<const uint8_t *>(p.A);
  P.B = static_cast<const uint8_t *>(p.B);
  P.C = p.C;
  P.lda = p.a_sm;
  const bool b_kc = p.b_sk == 1;
  P.ldb = b_kc ? p.b_sn : p.b_sk;
  P.ldc = p.ldc;
  P.m = (int)p.m;
  P.nsteps = (int)((p.k + 127) / 128);
  P.half_last = p.k % 128 != 0;
  P.tiles = (int)(p.n / (16 * nt));
  P.accumulate = p.accumulate;
  P.out_float = p.out_float;
  P.scale = p.scale;
  const int uns = p.a_unsigned ? 1 : (p.b_unsigned ? 2 : 0);
  const int mt = p.m <= 16 ? 1 : (p.m <= 32 ? 2 : 4);
  void (*kern)(SlabParams) = nullptr;
  const bool many = P.tiles > compute_units(), few_steps = P.nsteps <= 4;
  Rings rings = DEEP;
  if (nt == 1 && mt == 1) rings = few_steps || (many && P.nsteps < 16) ? FEW : (many ? HALF : DEEP);
  else if ((nt == 4 && mt == 1) || (nt == 1 && mt == 2)) rings = many || few_steps ? FEW : DEEP;
  if (rings == HALF) kern = pick<1, 1, HALF>(b_kc, uns);
  else if (rings == FEW && nt == 4) kern = pick<1, 4, FEW>(b_kc, uns);
  else if (rings == FEW) kern = mt == 1 ? pick<1, 1, FEW>(b_kc, uns) : pick<2, 1, FEW>(b_kc, uns);
  else if (nt == 1) kern = mt == 1 ? pick<1, 1>(b_kc, uns) : (mt == 2 ? pick<2, 1>(b_kc, uns) : pick<4, 1>(b_kc, uns));
  else if (nt == 2) kern = mt == 1 ? pick<1, 2>(b_kc, uns) : (mt == 2 ? pick<2, 2>(b_kc, uns) : pick<4, 2>(b_kc, uns));
  else kern = mt == 1 ? pick<1, 4>(b_kc, uns) : (mt == 2 ? pick<2, 4>(b_kc, uns) : pick<4, 4>(b_kc, uns));
  const int waves = slab_waves(mt, nt, rings);
  const size_t lds = (size_t)waves * 2048 * (steps_of_b(mt, nt, rings) * nt + steps_of_a(mt, nt, rings) * mt);
  {
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds);
    if (e != hipSuccess) return e;
  }
  dim3 grid((unsigned)(((P.tiles + 7) / 8) * 8));
  return launch_with(reinterpret_cast<const void *>(kern), grid, 64 * waves, lds, s, &P);
}

}  // namespace mip
