// Tiles whose waves split k between them: for a C of so few tiles that the chain of k blocks a
// workgroup goes through, and not the matrix cores, is what a product takes.
#pragma once
#include "dma_common.h"
#include "epilogue16.h"

namespace mip {

struct WaveTileParams {
  const uint8_t *A, *B;
  int32_t *C;
  int64_t m, n, k;
  int64_t lda, ldb, ldc;  // the one stride of each operand that is not 1
  TileWalk walk;
  int nsteps;      // k / 128, rounded up
  int half_last;   // the last step is 64 deep
  int accumulate;  // C += instead of C =
  int out_mode;    // 0 int32, 1 float(sum) * scale, 2 requantised int8
  float scale;
  const int32_t *ksum;  // not null: the k sums of the signed operand (see Problem::ksum)
  int64_t a_sb, b_sb, c_sb;
};
struct WaveConvParams : WaveTileParams {
  ConvGeom conv;
  // by the output positions of an image and of a row of one, the 64-channel blocks of a tap, and the taps of a filter row
  Divisor per_image, per_row, per_tap, per_filter_row;
};

// Where a wave's operands come from.  STREAMED: 16-byte aligned, k a multiple of 64, by direct loads into
// LDS.  GATHERED: the same with the lowered matrix of a convolution as A, channels a multiple of 64.
// STAGED: any alignment, through registers.
enum Source { STREAMED, GATHERED, STAGED };

// One operand of a wave's step: 16 * T rows (m or n), 128 of k, 2 * T pieces of 16 bytes per lane, piece q of
// the 64 lanes 1 KB of LDS.
//   KC: row r at r * 128, its 16-byte chunk c at 16 * (c ^ (r / 2 % 8)); piece q: rows 8 q .. + 7.
//   strided: k-row q at q * 16 T, its chunk c at 16 * (c ^ swz(q)).
template <int T, bool KC>
struct WaveOperand {
  static constexpr int LOADS = 2 * T, BYTES = LOADS * 1024;
  __device__ static __forceinline__ int row(int q, int lane) { return KC ? 8 * q + (lane >> 3) : q * (64 / T) + lane / T; }
  __device__ static __forceinline__ int swz(int row) {
    return KC ? (row >> 1) & 7 : (T == 4 ? 2 * ((row >> 2) & 1) : 0);
  }
  // the chunk of its row that a lane's piece q is: direct loads leave lane l's 16 bytes at 16 l
  __device__ static __forceinline__ int chunk(int q, int lane) { return (lane % (KC ? 8 : T)) ^ swz(row(q, lane)); }
  // source offset of a lane's piece q where `rows` rows exist: what lies beyond repeats something that does
  __device__ static __forceinline__ uint32_t source(int q, int lane, int rows, int64_t ld) {
    const int r = row(q, lane), c = chunk(q, lane);
    if (KC) return (uint32_t)((r < rows ? r : rows - 1) * ld + 16 * c);
    return (uint32_t)(r * ld + 16 * (16 * c < rows ? c : 0));
  }
  // fragment of v_mfma_i32_16x16x64_i8: row block t, 64-deep half h of the step
  __device__ static __forceinline__ v4i fragment(const uint8_t *s, int t, int h, int lane) {
    if (KC)
      return *reinterpret_cast<const v4i *>(s + t * 2048 + (lane & 15) * 128 +
                                            (((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) << 4));
    // transposing read: in each group of 16 lanes, lane 2 u + e names half e of the 16-byte row u
    // and lane i receives byte i of rows 0 .. 7
    const int krow = 64 * h + 16 * (lane >> 4) + ((lane & 15) >> 1);
    v4i f;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int q = krow + 8 * r;
      const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
          LDS_PTR(v2i, s + q * (16 * T) + ((t ^ swz(q)) << 4) + 8 * (lane & 1)));
      f[2 * r] = x[0];
      f[2 * r + 1] = x[1];
    }
    return f;
  }
};

// MT, NT: blocks of 16 rows and columns in a tile.  W: waves.
// UNS: 0 both operands signed, 1 A unsigned, 2 B unsigned.
// A workgroup of W waves has one tile of 16 MT x 16 NT; wave w takes steps w, w + W, ... of 128 k through LDS
// stages of its own, so that nothing but its own loads holds a wave up and the only barriers are those of the final
// sum over LDS.  What bounds it is the rate at which a compute unit takes direct loads, 63 bytes a clock (more of
// them per product the smaller the tile), and for a short k the latency of the first load and of the sum, some 3 us.
// (512, 512, 2048) on 64 x 64 tiles that share each block among four waves took 6.5 us and takes 4.2 on these.
template <int MT, int NT, int W, bool A_KC, bool B_KC, int UNS, Source SOURCE>
__global__ __launch_bounds__(64 * W) void wave_tile_kernel(std::conditional_t<SOURCE == GATHERED, WaveConvParams, WaveTileParams> P) {
  constexpr bool CONV = SOURCE == GATHERED, REGS = SOURCE == STAGED;
  static_assert(!CONV || (A_KC && B_KC && UNS == 1), "the lowered matrix is unsigned, it and the filters k-contiguous");
  using OA = WaveOperand<MT, A_KC>;
  using OB = WaveOperand<NT, B_KC>;
  constexpr int BM = 16 * MT, BN = 16 * NT, PITCH = BN + 4;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  fetch_arguments(P.walk, P.A, P.B, P.C, P.m, P.n, P.k, P.lda, P.ldb, P.ldc, P.nsteps, P.accumulate, P.out_mode,
                  P.scale, P.ksum);
  if constexpr (CONV)
    fetch_arguments(P.per_image.d, P.per_image.inv, P.per_row.inv, P.per_tap.inv, P.per_filter_row.inv, P.conv.hi,
                    P.conv.wi, P.conv.ci, P.conv.wf, P.conv.wo, P.conv.stride, P.conv.pad);
  else
    fetch_arguments(P.a_sb, P.b_sb, P.c_sb);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  int tm, tn;
  if (!tile_of_workgroup(P.walk, &tm, &tn)) return;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const uint8_t *A = P.A, *B = P.B;
  if (!CONV) {
    const int64_t z = blockIdx.z;
    A += z * P.a_sb + (A_KC ? m0 * P.lda : m0);
    B += z * P.b_sb;
  }
  B += B_KC ? n0 * P.ldb : n0;
  const int rows = (int)(P.m - m0 < BM ? P.m - m0 : BM), cols = (int)(P.n - n0 < BN ? P.n - n0 : BN);
  const int cnt = (P.nsteps + W - 1 - wave) / W;  // steps wave, wave + W, ... below nsteps
  const int64_t strideA = A_KC ? 128 : 128 * P.lda, strideB = B_KC ? 128 : 128 * P.ldb;
  const int half_step = !REGS && P.half_last ? P.nsteps - 1 : -1;

  uint32_t offA[OA::LOADS], offB[OB::LOADS];
  int conv_y[CONV ? OA::LOADS : 1], conv_x[CONV ? OA::LOADS : 1];
#pragma unroll
  for (int q = 0; q < OB::LOADS; ++q) offB[q] = OB::source(q, lane, cols, P.ldb);
#pragma unroll
  for (int q = 0; q < OA::LOADS; ++q) {
    if constexpr (CONV) {
      const ConvGeom &G = P.conv;
      int row = OA::row(q, lane);
      row = (int)m0 + (row < rows ? row : rows - 1);
      const int g = (int)divided((unsigned)row, P.per_image), r = row - g * (int)P.per_image.d;
      const int oy = (int)divided((unsigned)r, P.per_row), ox = r - oy * G.wo;
      conv_y[q] = oy * G.stride - G.pad;
      conv_x[q] = ox * G.stride - G.pad;
      offA[q] = (uint32_t)(((g * G.hi + conv_y[q]) * G.wi + conv_x[q]) * G.ci + 16 * (OA::chunk(q, lane) & 3));
    } else {
      offA[q] = OA::source(q, lane, rows, P.lda);
    }
  }

  uint8_t *const sa = smem + wave * (OA::BYTES + OB::BYTES), *const sb = sa + OA::BYTES;
  const uint32_t ldsA = lds_address(sa), ldsB = ldsA + OA::BYTES;
  v4i ra[REGS ? OA::LOADS : 1], rb[REGS ? OB::LOADS : 1];
  // Sends for step i of this wave.  Streamed: into its LDS, a 64-deep last step's second half fetched from its
  // first (it exists, and is not used).  Staged: into registers; a piece that k or n ends in, or that lies behind
  // the end, is fetched so far ahead of its place that it ends there, and shifted on its way into LDS.
  auto send = [&](int i) __attribute__((always_inline)) {
    const int step = wave + W * i;
    const uint8_t *gb = wave_uniform(B + step * strideB), *ga = CONV ? A : wave_uniform(A + step * strideA);
    if constexpr (REGS) {
      const int left = (int)(P.k - (int64_t)step * 128 < 128 ? P.k - (int64_t)step * 128 : 128);
      auto fetch = [&](auto operand, bool kc, const uint8_t *g, const uint32_t *off, int ext, int64_t ld, v4i *r) {
        using O = decltype(operand);
        if (left == 128 && (kc || ext % 16 == 0)) {
#pragma unroll
          for (int q = 0; q < O::LOADS; ++q) r[q] = load16(g + off[q]);
        } else {
#pragma unroll
          for (int q = 0; q < O::LOADS; ++q) {
            const int c = 16 * O::chunk(q, lane), row = O::row(q, lane);
            const int end = kc ? left : ext, back = c + 16 > end ? c + 16 - end : 0, have = kc ? ext : left;
            r[q] = load16(g + (row < have ? row : have - 1) * ld + (c - back));
          }
        }
      };
      fetch(OB{}, B_KC, gb, offB, cols, P.ldb, rb);
      fetch(OA{}, A_KC, ga, offA, rows, P.lda, ra);
    } else {
      const bool half = step == half_step;
#pragma unroll
      for (int q = 0; q < OB::LOADS; ++q) {
        uint32_t off = offB[q];
        if (half) off = B_KC ? off - (OB::chunk(q, lane) >= 4 ? 64 : 0) : offB[q >= NT ? q - NT : q];
        dma16(off, gb, ldsB + q * 1024);
      }
      if constexpr (CONV) {
        const ConvGeom &G = P.conv;
        int y[2], x[2], at[2];  // the tap of either half of the step
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const unsigned block = 2 * step + (half ? 0 : h), tap = divided(block, P.per_tap);
          y[h] = (int)divided(tap, P.per_filter_row);
          x[h] = (int)tap - y[h] * G.wf;
          at[h] = (y[h] * G.wi + x[h]) * G.ci + (int)(block * 64 - tap * (unsigned)G.ci);
        }
#pragma unroll
        for (int q = 0; q < OA::LOADS; ++q) {
          const bool second = OA::chunk(q, lane) >= 4;
          const int py = conv_y[q] + (second ? y[1] : y[0]), px = conv_x[q] + (second ? x[1] : x[0]);
          const bool inside = (unsigned)py < (unsigned)G.hi && (unsigned)px < (unsigned)G.wi;
          dma16_at(inside ? A + ((int)offA[q] + (second ? at[1] : at[0])) : outside_image, ldsA + q * 1024);
        }
      } else {
#pragma unroll
        for (int q = 0; q < OA::LOADS; ++q) {
          uint32_t off = offA[q];
          if (half) off = A_KC ? off - (OA::chunk(q, lane) >= 4 ? 64 : 0) : offA[q >= MT ? q - MT : q];
          dma16(off, ga, ldsA + q * 1024);
        }
      }
    }
  };
  // Step i of this wave in its LDS.
  auto arrive = [&](int i) __attribute__((always_inline)) {
    if constexpr (REGS) {
      const int64_t step = wave + W * i;
      const int left = (int)(P.k - step * 128 < 128 ? P.k - step * 128 : 128);
      auto place = [&](auto operand, bool kc, uint8_t *to, int ext, v4i *r) {
        using O = decltype(operand);
        if (left < 128 || (!kc && ext % 16 != 0)) {
#pragma unroll
          for (int q = 0; q < O::LOADS; ++q) {
            const int c = 16 * O::chunk(q, lane), end = kc ? left : ext;
            r[q] = c + 16 > end ? shifted_down(r[q], c + 16 - end) : r[q];
            if (!kc && O::row(q, lane) >= left) r[q] = v4i{0, 0, 0, 0};
          }
        }
#pragma unroll
        for (int q = 0; q < O::LOADS; ++q) *reinterpret_cast<v4i *>(to + q * 1024 + 16 * lane) = r[q];
      };
      place(OB{}, B_KC, sb, cols, rb);
      place(OA{}, A_KC, sa, rows, ra);
      asm volatile("" ::: "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
  };
  if (cnt > 0) send(0);

  v4i acc[MT][NT], accS[UNS == 1 ? NT : MT];  // accS: the signed operand's k sums, by a row (column) of ones
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = v4i{0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < (UNS == 1 ? NT : MT); ++i) accS[i] = v4i{0, 0, 0, 0};
  const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};

  for (int j = 0; j < cnt; ++j) {
    arrive(j);
    if (REGS && j + 1 < cnt) send(j + 1);  // (the registers are free, the LDS is not)
    v4i fa[2][MT], fb[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[h][i] = OA::fragment(sa, i, h, lane);
#pragma unroll
      for (int i = 0; i < NT; ++i) fb[h][i] = OB::fragment(sb, i, h, lane);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // in registers before the LDS is refilled
    if (!REGS && j + 1 < cnt) send(j + 1);
    const bool half = wave + W * j == half_step;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && half) break;
      if (UNS == 1) {
#pragma unroll
        for (int i = 0; i < MT; ++i) fa[h][i] ^= (int)0x80808080u;
        if (!P.ksum) {
#pragma unroll
          for (int i = 0; i < NT; ++i)
            accS[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[h][i], ones, accS[i], 0, 0, 0);
        }
      }
      if (UNS == 2) {
#pragma unroll
        for (int i = 0; i < NT; ++i) fb[h][i] ^= (int)0x80808080u;
        if (!P.ksum) {
#pragma unroll
          for (int i = 0; i < MT; ++i)
            accS[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, fa[h][i], accS[i], 0, 0, 0);
        }
      }
      // (B first: lane l of a result holds C row l % 16, its four registers columns 4 * (l / 16) .. + 3)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[h][t], fa[h][i], acc[i][t], 0, 0, 0);
    }
  }

  // the waves' partial sums meet in LDS, over the operands, once every wave is done with them
  const int active = P.nsteps < W ? P.nsteps : W;
  __syncthreads();
  int32_t *red = reinterpret_cast<int32_t *>(smem);
  if (wave < active) {
    int32_t *mine = red + wave * (BM * PITCH) + (lane & 15) * PITCH + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (UNS != 0) acc[i][t] += 128 * accS[UNS == 1 ? t : i];
        *reinterpret_cast<v4i *>(mine + i * 16 * PITCH + 16 * t) = acc[i][t];
      }
  }
  __syncthreads();
  constexpr int QUADS = BM * BN / 4, PASSES = (QUADS + 64 * W - 1) / (64 * W);
  int32_t *C = P.C + (int64_t)blockIdx.z * P.c_sb + m0 * P.ldc + n0;
  int8_t *Q = reinterpret_cast<int8_t *>(P.C) + m0 * P.ldc + n0;
  v4i sum[PASSES];
#pragma unroll
  for (int u = 0; u < PASSES; ++u) {
    const int at = tid + u * (64 * W), r = at / (BN / 4), c = 4 * (at % (BN / 4));
    const int32_t *from = red + (QUADS % (64 * W) == 0 || r < BM ? r * PITCH + c : 0);
    v4i part[W];
#pragma unroll
    for (int w = 0; w < W; ++w) part[w] = *reinterpret_cast<const v4i *>(from + (w < active ? w : 0) * (BM * PITCH));
    sum[u] = part[0];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      if (w < active) sum[u] += part[w];
    }
  }
#pragma unroll
  for (int u = 0; u < PASSES; ++u) {
    const int at = tid + u * (64 * W), r = at / (BN / 4), c = 4 * (at % (BN / 4));
    if (r >= rows || c >= cols) continue;
    int32_t *dst = C + r * P.ldc + c;
    const bool whole = c + 3 < cols;
    v4i old = {0, 0, 0, 0};
    if (P.accumulate) {
      if (whole) old = *reinterpret_cast<const v4i_dword_aligned *>(dst);
      else
        for (int e = 0; e < cols - c; ++e) old[e] = dst[e];
    }
    if (UNS != 0 && P.ksum) {
      if (UNS == 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c + e < cols) sum[u][e] += 128 * P.ksum[n0 + c + e];
      } else {
        sum[u] += 128 * P.ksum[m0 + r];
      }
    }
    if (P.out_mode == 2) {
      const int word = requantise(sum[u][0], P.scale) | requantise(sum[u][1], P.scale) << 8 |
                       requantise(sum[u][2], P.scale) << 16 | requantise(sum[u][3], P.scale) << 24;
      int8_t *d = Q + r * P.ldc + c;
      if (whole) reinterpret_cast<q8_word *>(d)->w = word;
      else
        for (int e = 0; e < cols - c; ++e) d[e] = (int8_t)(word >> (8 * e));
      continue;
    }
    const Finish fin = {P.scale, P.out_mode};
    v4i out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = fin(sum[u][e], old[e], P.accumulate != 0);
    if (whole) *reinterpret_cast<v4i_dword_aligned *>(dst) = out;
    else
      for (int e = 0; e < cols - c; ++e) dst[e] = out[e];
  }
}

// SOURCE: STREAMED (a convolution is gathered) or STAGED
template <int MT, int NT, int W, Source SOURCE>
hipError_t launch_wave_tile_for(const Problem &p, hipStream_t s) {
  constexpr int BM = 16 * MT, BN = 16 * NT;
  const bool a_kc = p.a_sk == 1, b_kc = p.b_sk == 1;
  WaveConvParams P;
  P.A = static_cast<const uint8_t *>(p.A);
  P.B = static_cast<const uint8_t *>(p.B);
  P.C = p.C;
  P.m = p.m;
  P.n = p.n;
  P.k = p.k;
  P.lda = a_kc ? p.a_sm : p.a_sk;
  P.ldb = b_kc ? p.b_sn : p.b_sk;
  P.ldc = p.ldc;
  P.walk = tile_walk((p.m + BM - 1) / BM, (p.n + BN - 1) / BN);
  P.nsteps = (int)((p.k + 127) / 128);
  P.half_last = p.k % 128 != 0;
  P.accumulate = p.accumulate;
  P.out_mode = p.out_float;
  P.scale = p.scale;
  const int uns = p.a_unsigned ? 1 : (p.b_unsigned ? 2 : 0);
  P.ksum = p.batch <= 1 ? p.ksum : nullptr;
  P.a_sb = p.a_sb;
  P.b_sb = p.b_sb;
  P.c_sb = p.c_sb;
  void (*kern)(WaveTileParams) = nullptr;
#define MIP_PICK(AK, BKC)                                                                      \
  kern = uns == 0 ? wave_tile_kernel<MT, NT, W, AK, BKC, 0, SOURCE>                            \
                  : (uns == 1 ? wave_tile_kernel<MT, NT, W, AK, BKC, 1, SOURCE>                \
                              : wave_tile_kernel<MT, NT, W, AK, BKC, 2, SOURCE>)
  if (a_kc && b_kc) MIP_PICK(true, true);
  else if (a_kc) MIP_PICK(true, false);
  else if (b_kc) MIP_PICK(false, true);
  else MIP_PICK(false, false);
  const void *kernel = reinterpret_cast<const void *>(kern);
  if constexpr (SOURCE == STREAMED) {
    if (p.conv) {
      const ConvGeom &g = *p.conv;
      P.conv = g;
      P.per_image = divisor((int64_t)g.ho * g.wo, p.m);
      P.per_row = divisor(g.wo, (int64_t)g.ho * g.wo);
      P.per_tap = divisor(g.ci / 64, p.k / 64 + 1);
      P.per_filter_row = divisor(g.wf, p.k / g.ci + 1);
      void (*gather)(WaveConvParams) = wave_tile_kernel<MT, NT, W, true, true, 1, GATHERED>;
      kernel = reinterpret_cast<const void *>(gather);
    }
  }
#undef MIP_PICK
  const size_t stages = (size_t)W * (MT + NT) * 2048, sums = (size_t)W * BM * (BN + 4) * 4;
  const size_t lds = stages > sums ? stages : sums;
  hipError_t e = allow_dynamic_lds(kernel, lds);
  if (e != hipSuccess) return e;
  const int64_t tiles = (int64_t)P.walk.tiles_m * P.walk.tiles_n;
  dim3 grid((unsigned)(((tiles + 7) / 8) * 8), 1, (unsigned)p.batch);
  return launch_with(kernel, grid, 64 * W, lds, s, &P);
}

}  // namespace mip
