// Weight pre-packing: the k x n 8-bit matrix B rewritten once with k contiguous
// (column-major, pitch ldp), the form in which the paper's packed buffer B_c
// feeds its micro-kernels (Section 4.1; Section 5: every MIP instruction wants k
// contiguous per operand register).  The GEMM kernels take either order as it is,
// so this is never needed for correctness; it pays when the same weights meet a
// few rows of activations many times, because the skinny-m kernel streams a
// k-contiguous B in whole 64-byte runs and a row-major one in 16-byte pieces.
//
// Pure data movement: a byte transpose of square tiles through LDS, or a re-pitching copy when B
// already is k-contiguous.  The same kernels pack both operands of a GEMM whose storage the
// direct-to-LDS kernels cannot stream (Section 4.1: Pack A, Pack B into the aligned buffers
// A_c, B_c): then the k tail up to the padded length is zeroed.  Loads are 16 bytes at whatever
// alignment, four of a thread in flight; stores are 16 bytes where the destination's alignment allows.
#include "dma_common.h"

namespace mip {

namespace {

// B(p, j) = B[p * ldb + j]  ->  P[j * ldp + p]
// One packing job: the k x n matrix at B (k_contiguous: column j at B + j * ldb; else row
// p at B + p * ldb) to P, column j at P + j * ldp, entries k .. kfill - 1 of every packed
// column written as zeros (kfill == k: none).
struct PackJob {
  int64_t k, kfill, n;
  const uint8_t *B;
  int64_t ldb;
  uint8_t *P;
  int64_t ldp;
  int k_contiguous, wide_store;
  Divisor tiles_n;      // transposing job: tiles along n
  int large;            // tiles of 128 x 128 instead of 64 x 64
  int lanes_per_column; // copying job: a power of two, at most 64
  unsigned blocks;      // workgroups this job is given
};

// The first `left` (may be <= 0 or > 16) of the 16 bytes at p, zeros behind them; `before`: how many bytes of the
// same run lie ahead of p.
__device__ __forceinline__ v4i load_piece(const uint8_t *p, int64_t left, int64_t before) {
  if (left >= 16) return load16(p);
  if (left <= 0) return v4i{0, 0, 0, 0};
  if (before + left >= 16) return shifted_down(load16(p - (16 - left)), (int)(16 - left));
  return load16_partial(p, (int)left);
}
__device__ __forceinline__ void store_piece(uint8_t *dst, v4i v, int64_t left, bool wide) {
  if (wide && left >= 16) {
    *reinterpret_cast<v4i *>(dst) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (e < left) dst[e] = (uint8_t)(v[e >> 2] >> (8 * (e & 3)));
  }
}

// block: this workgroup's number within the job.  A tile of E x E bytes is staged row by row (k), its
// 16-byte chunk c of k-row q at q * E + 16 * (c ^ swz(q)), and read back column by column with the
// transposing LDS read (see WaveOperand and Stage16 for the layout).  Sixteen single-byte LDS reads per
// piece, on 64 x 64 tiles with one load in flight, took 17.5 us for both operands of
// 4095 x 4097 x 4099; this takes 15.0.
template <int E>
__device__ __forceinline__ void pack_transpose_body(const PackJob &J, unsigned block, uint8_t *tile) {
  constexpr int CHUNKS = E / 16, PIECES = E * E / 16 / NTHREADS;  // per thread
  auto swz = [](int q) { return E == 64 ? 2 * ((q >> 2) & 1) : (2 * ((q >> 1) & 3)) ^ ((q >> 4) & 1); };
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const unsigned tile_k = divided(block, J.tiles_n);
  const int64_t p0 = (int64_t)tile_k * E, n0 = (int64_t)(block - tile_k * J.tiles_n.d) * E;
  v4i piece[PIECES];
#pragma unroll
  for (int u = 0; u < PIECES; ++u) {
    const int at = t + u * NTHREADS, q = at / CHUNKS, c = at % CHUNKS;
    const int64_t row = p0 + q, col = n0 + 16 * c;
    piece[u] = load_piece(J.B + (row < J.k ? row : 0) * J.ldb + col, row < J.k ? J.n - col : 0, col);
  }
#pragma unroll
  for (int u = 0; u < PIECES; ++u) {
    const int at = t + u * NTHREADS, q = at / CHUNKS, c = at % CHUNKS;
    *reinterpret_cast<v4i *>(tile + q * E + 16 * (c ^ swz(q))) = piece[u];
  }
  __syncthreads();
  // a group of sixteen lanes takes sixteen columns and sixteen k; the four groups of a wave are
  // neighbours along k, 64 consecutive bytes of a packed column
#pragma unroll
  for (int u = 0; u < PIECES; ++u) {
    const int unit = wave + 4 * u;                       // of CHUNKS column blocks by E / 64 quarters of k
    const int cb = unit % CHUNKS, k16 = 4 * (unit / CHUNKS) + (lane >> 4);
    v4i v;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int q = 16 * k16 + 8 * r + ((lane & 15) >> 1);
      const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
          LDS_PTR(v2i, tile + q * E + 16 * (cb ^ swz(q)) + 8 * (lane & 1)));
      v[2 * r] = x[0];
      v[2 * r + 1] = x[1];
    }
    const int64_t col = n0 + 16 * cb + (lane & 15), row = p0 + 16 * k16;
    if (col < J.n && row < J.kfill) store_piece(J.P + col * J.ldp + row, v, J.kfill - row, J.wide_store);
  }
}

// B already k-contiguous: column j moves from B + j * ldb to P + j * ldp.  lanes_per_column lanes share a
// column, so that no position is found by dividing a flat index.
__device__ __forceinline__ void pack_copy_body(const PackJob &J, unsigned block) {
  constexpr int FLY = 4;
  const int lanes = J.lanes_per_column, shift = __builtin_ctz(lanes);
  const int l = threadIdx.x & (lanes - 1);
  const int columns = NTHREADS >> shift;
  for (int64_t j = (int64_t)block * columns + (threadIdx.x >> shift); j < J.n; j += (int64_t)J.blocks * columns) {
    const uint8_t *src = J.B + j * J.ldb;
    uint8_t *dst = J.P + j * J.ldp;
    for (int64_t p0 = 16 * l; p0 < J.kfill; p0 += 16 * FLY * lanes) {
      v4i piece[FLY];
#pragma unroll
      for (int u = 0; u < FLY; ++u) {
        const int64_t p = p0 + u * 16 * lanes;
        piece[u] = load_piece(src + p, J.k - p, p);
      }
#pragma unroll
      for (int u = 0; u < FLY; ++u) {
        const int64_t p = p0 + u * 16 * lanes;
        if (p < J.kfill) store_piece(dst + p, piece[u], J.kfill - p, J.wide_store);
      }
    }
  }
}

// One or two jobs in one launch: the first a.blocks workgroups work on a, the rest on b
// (Pack A and Pack B of a GEMM are independent of each other).
__global__ __launch_bounds__(NTHREADS) void pack_kernel(PackJob a, PackJob b) {
  __shared__ __attribute__((aligned(16))) uint8_t tile[128 * 128];
  const bool first = blockIdx.x < a.blocks;  // workgroup-uniform
  const PackJob &J = first ? a : b;
  const unsigned block = first ? blockIdx.x : blockIdx.x - a.blocks;
  if (J.k_contiguous) pack_copy_body(J, block);
  else if (J.large) pack_transpose_body<128>(J, block, tile);
  else pack_transpose_body<64>(J, block, tile);
}

bool aligned16(const void *p, int64_t ld) {
  return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 16 == 0;
}

// false: the job is too large for one launch
bool make_job(int64_t k, int64_t kfill, int64_t n, const uint8_t *B, int64_t ldb, bool b_kc,
              uint8_t *P, int64_t ldp, PackJob *out) {
  PackJob J;
  J.k = k; J.kfill = kfill < k ? k : kfill; J.n = n;
  J.B = B; J.ldb = ldb; J.P = P; J.ldp = ldp;
  J.k_contiguous = b_kc;
  J.wide_store = aligned16(P, ldp);
  J.tiles_n = Divisor{1, 0};
  J.large = 0;
  J.lanes_per_column = 64;
  if (J.kfill == 0 || n == 0) {
    J.blocks = 0;
  } else if (b_kc) {
    while (J.lanes_per_column > 1 && J.lanes_per_column * 8 >= J.kfill) J.lanes_per_column /= 2;
    const int64_t columns = NTHREADS / J.lanes_per_column, blocks = (n + columns - 1) / columns;
    J.blocks = (unsigned)(blocks < 256 * 64 ? blocks : 256 * 64);
  } else {
    // (128 x 128 tiles, whole cache lines on both sides, where there are enough of them)
    auto tiles = [&](int64_t e, int64_t *along_n) {
      *along_n = (n + e - 1) / e;
      return (J.kfill + e - 1) / e * *along_n;
    };
    int64_t tiles_n, count = tiles(128, &tiles_n);
    J.large = count >= 256;
    if (!J.large) count = tiles(64, &tiles_n);
    if (count > 0x3fffffff) return false;
    J.tiles_n = divisor(tiles_n, count);
    J.blocks = (unsigned)count;
  }
  *out = J;
  return true;
}

// One wave per column of a k-contiguous matrix: the sum of its k bytes read as signed 8-bit
// values.  WIDE: k a multiple of 16 and every column 16-byte aligned.
template <bool WIDE>
__global__ __launch_bounds__(256) void column_sums_kernel(const uint8_t *P, int64_t ldp, int64_t k,
                                                          int64_t n, int32_t *sums) {
  const int lane = threadIdx.x & 63;
  const int64_t col = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= n) return;
  int sum = 0;
  if (WIDE) {
    const v4i *src = reinterpret_cast<const v4i *>(P + col * ldp);
    for (int64_t c = lane; c < k / 16; c += 64) {
      const v4i v = src[c];
#pragma unroll
      for (int e = 0; e < 4; ++e) sum = __builtin_amdgcn_sdot4(v[e], 0x01010101, sum, false);
    }
  } else {
    const int8_t *src = reinterpret_cast<const int8_t *>(P + col * ldp);
    for (int64_t c = lane; c < k; c += 64) sum += src[c];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) sums[col] = sum;
}

}  // namespace

hipError_t launch_column_sums(int64_t k, int64_t n, const uint8_t *P, int64_t ldp, int32_t *sums,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if ((n + 3) / 4 > 0x7fffffff) return hipErrorInvalidValue;
  const bool wide = k % 16 == 0 && ldp % 16 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
  const dim3 grid((unsigned)((n + 3) / 4));
  if (wide) hipLaunchKernelGGL(column_sums_kernel<true>, grid, dim3(256), 0, s, P, ldp, k, n, sums);
  else hipLaunchKernelGGL(column_sums_kernel<false>, grid, dim3(256), 0, s, P, ldp, k, n, sums);
  return hipGetLastError();
}

hipError_t launch_pack_b(int64_t k, int64_t n, const uint8_t *B, int64_t ldb, bool b_kc, uint8_t *P,
                         int64_t ldp, hipStream_t s, int64_t kfill) {
  PackJob J, none = {};
  if (!make_job(k, kfill, n, B, ldb, b_kc, P, ldp, &J)) return hipErrorInvalidValue;
  if (J.blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_kernel, dim3(J.blocks), dim3(256), 0, s, J, none);
  return hipGetLastError();
}

hipError_t launch_pack_pair(int64_t k, int64_t kfill, int64_t m, const uint8_t *A, int64_t lda,
                            bool a_kc, uint8_t *Ap, int64_t n, const uint8_t *B, int64_t ldb,
                            bool b_kc, uint8_t *Bp, int64_t ldp, hipStream_t s) {
  PackJob a, b;
  if (!make_job(k, kfill, m, A, lda, a_kc, Ap, ldp, &a) || !make_job(k, kfill, n, B, ldb, b_kc, Bp, ldp, &b))
    return hipErrorInvalidValue;
  if (a.blocks + b.blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_kernel, dim3(a.blocks + b.blocks), dim3(256), 0, s, a, b);
  return hipGetLastError();
}

}  // namespace mip
