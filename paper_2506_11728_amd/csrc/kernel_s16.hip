// 16-bit operands on the 8-bit matrix instructions.
//
// gfx950 has no integer matrix instruction for 16-bit operands (the paper's ISA table lists
// (i32, i16, i16) forms for other machines: vpdpwssd, smopa), so an int16 x int16 -> int32
// product is built from int8 products.  With x' = x - 128, every int16 splits exactly into two
// SIGNED bytes, x' = 256 h + l with h = x >> 8 (arithmetic) and l = (x & 255) - 128, and
//     sum_p a b = sum_p a' b' + 128 (sum_p a + sum_p b) - 16384 k,
//     sum_p a' b' = 65536 sum_p ah bh + 256 sum_p (ah bl + al bh) + sum_p al bl,
// all modulo 2^32.
//
// One kernel does all of it.  The 16-bit operands are staged in LDS as they are stored, a wave
// splits each fragment into its two byte planes on the way from LDS to the matrix instructions
// (eight byte permutes and four sign flips for sixteen k of sixteen rows), keeps the three sums
// of byte products in registers and puts them together in the write-back.  Both planes of a
// fragment meet both planes of the other operand's, so a byte of operand feeds twice the
// matrix instructions it would in an 8-bit product: a 128 x 128 tile has the operand traffic of
// a 256 x 256 one there.
// What bounds it: a 64-deep block of a 128 x 128 tile takes 1024 clocks of matrix instructions and as
// many of LDS traffic per compute unit, and about 900 of ordinary vector instructions (splits, sums,
// addresses) per SIMD; together, with a barrier per block, they take about 2000.
// (Splitting into planes in memory first, three 8-bit products and a pass that combined them were
// nine launches and five passes over C-sized data: (1024, 3072, 768) 43 us, this kernel 16.5 us
// (17.7 under a profiler, 18 in a graph); 64 x 64 of wave tile instead of 64 x 32, one wave to a SIMD: 19 us.)
#include <cstring>

#include "dma_common.h"
#include "tuning.h"

namespace mip {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));  // sums modulo 2^32
typedef v4u v4u_dword_aligned __attribute__((aligned(4)));
struct __attribute__((packed, aligned(2))) s16x8 { short v[8]; };

constexpr int KB = 64;        // k per staged block: 128 bytes
constexpr int STAGES = 3;

// what a chunk beyond the end of k is fetched from (device memory, always zero)
static __device__ v4i g_zero_chunk;

struct S16Params {
  const uint8_t *A, *B;
  uint32_t *C;
  int64_t lda, ldb;  // bytes: the one stride of each operand that is not one element
  int64_t ldc;
  int64_t m, n, k;
  TileWalk walk;
  int nkt;        // blocks of 64 k, the last one filled up with zeros
  int splits;     // ranges of k, one per blockIdx.y
  int per_range, longer;  // their blocks; the first `longer` have one more
  int accumulate;
  int wide_offsets;  // rows of a tile reach further than 32-bit offsets do
  // splits > 1: `splits` slots of partial sums per tile and one zeroed counter per tile; null: the
  // ranges add into C, which holds zeros (or what the call accumulates into) before the launch
  int32_t *slots;
  unsigned *tickets;
};

// One R x 64 block of an operand in LDS.
//   KC (k contiguous in memory): R rows of 128 bytes; 16-byte chunk c of row r sits at
//     r*128 + 16*(c ^ ((r >> 1) & 7)): the sixteen rows that one 16-byte read of a lane group
//     touches lie in all banks.
//   strided (the index runs contiguously): 64 k-rows of 2 R bytes; chunk c of k-row q sits at
//     q*2R + 16*(c ^ 2 f(q)): the eight k-rows (four of each of two lane groups) that half a
//     transposing read touches, 32 bytes of each, lie in all banks.
// NT: threads of the workgroup.
template <int R, bool KC, int NT>
struct StageS16 {
  static constexpr int BYTES = R * 2 * KB;
  static constexpr int LOADS = BYTES / 16 / NT;
  static constexpr int ROW_CHUNKS = R / 8;
  __device__ static __forceinline__ int swz(int q) {
    return R == 128 ? 2 * ((q & 3) | ((q >> 3) & 1) << 2) : 2 * (((q >> 1) & 1) | ((q >> 3) & 1) << 1);
  }
  // direct load i of this thread: row a (KC) or k-row a, 16-byte chunk g of it
  __device__ static __forceinline__ void chunk_of(int i, int tid, int &a, int &g) {
    const int q = tid + NT * i;
    if (KC) { a = q >> 3; g = (q & 7) ^ ((a >> 1) & 7); }
    else { a = q / ROW_CHUNKS; g = (q % ROW_CHUNKS) ^ swz(a); }
  }
  // The chunk's offset from the block's origin.  `extent` rows (KC) or elements of a k-row
  // (strided; a multiple of 8) exist from the tile's origin on; what would lie beyond is
  // fetched from a place that exists, and what it feeds never reaches C.
  __device__ static __forceinline__ int64_t global_offset(int i, int tid, int64_t ld, int extent) {
    int a, g;
    chunk_of(i, tid, a, g);
    if (KC) a = a < extent ? a : extent - 1;
    else g = 8 * g < extent ? g : 0;
    return a * ld + 16 * g;
  }
  // does the chunk hold anything when only `left` k of the block exist (KC: a multiple of 8)
  __device__ static __forceinline__ bool inside_k(int i, int tid, int left) {
    int a, g;
    chunk_of(i, tid, a, g);
    return (KC ? 8 * g : a) < left;
  }
  // Fragment F of the block, its rows 16 F .. + 15: lane l gets, of row 16 F + l % 16, the eight k
  // from 8 (l / 16) on and the eight from 32 + 8 (l / 16) on, as 32 bytes.  (Any order of k will
  // do that both operands share; in this one a read's lanes never meet in a bank, whichever
  // sixteen of them the hardware serves at a time.)  Its LDS address is (lane_base ^ turn(F)) +
  // shift(F) from the stage on, the first part per lane, the others the same in a wave.
  __device__ static __forceinline__ uint32_t lane_base(int lane) {
    if (KC) return (uint32_t)((lane & 15) * 128 + (((lane >> 4) ^ ((lane >> 1) & 7)) << 4));
    // ds_read_b64_tr_b16: inside each group of 16 lanes, lane 4t+h supplies the address of
    // quarter h of the 32 bytes of k-row t, and lane i receives element i of k-rows 0..3
    const int s = lane & 15, q = 8 * (lane >> 4) + (s >> 2);
    return (uint32_t)(q * (2 * R) + ((((s & 3) >> 1) ^ swz(q)) << 4) + 8 * (s & 1));
  }
  __device__ static __forceinline__ uint32_t turn(int F) { return KC ? 0u : 32u * (uint32_t)F; }
  __device__ static __forceinline__ uint32_t shift(int F) { return KC ? 2048u * (uint32_t)F : 0u; }
  // at: (lane_base ^ turn) + shift + the stage's place in LDS
  __device__ static __forceinline__ void fragment(const uint8_t *smem, uint32_t at, v4i (&raw)[2]) {
    if (KC) {
      raw[0] = *reinterpret_cast<const v4i *>(smem + at);
      raw[1] = *reinterpret_cast<const v4i *>(smem + (at ^ 64u));  // chunk 4 + l / 16 (rows are 128-byte aligned)
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const s16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            LDS_PTR(s16x4, smem + at + ((t >> 1) * 32 + (t & 1) * 4) * (2 * R)));
        const v2i w = __builtin_bit_cast(v2i, h);
        raw[t >> 1][2 * (t & 1)] = w[0];
        raw[t >> 1][2 * (t & 1) + 1] = w[1];
      }
    }
  }
};

// WR x WC waves over a tile of C, each on FM x FN blocks of 16 x 16.  Fragments of block t + 1 are
// read and split while block t is multiplied; loads run two blocks further ahead.  Two waves to
// a SIMD: one alone issues an ordinary vector instruction only every eight clocks.
// STAGED: operands at any alignment, through registers: a block is loaded into them a step before it is stored to its
// LDS stage; a 16-byte piece that an operand's edge cuts is fetched so far ahead that it ends there, and shifted
// on its way.
template <int WR, int WC, int FM, int FN, bool A_KC, bool B_KC, bool STAGED>
__global__ __launch_bounds__(64 * WR * WC, 2) void s16_kernel(S16Params P) {
  constexpr int NT = 64 * WR * WC, WM = 16 * FM, WN = 16 * FN, BM = WR * WM, BN = WC * WN;
  using SA = StageS16<BM, A_KC, NT>;
  using SB = StageS16<BN, B_KC, NT>;
  constexpr int STAGE = SA::BYTES + SB::BYTES, LOADS = SA::LOADS + SB::LOADS;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WC, wn = wave % WC;
  fetch_arguments(P.walk, P.A, P.B, P.C, P.lda, P.ldb, P.ldc, P.m, P.n, P.k, P.nkt, P.splits, P.per_range, P.longer,
                  P.accumulate, P.wide_offsets, P.slots);
  int tm, tn;
  if (!tile_of_workgroup(P.walk, &tm, &tn)) return;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int block0 = first_of_range(blockIdx.y, P.per_range, P.longer);
  const int nkt = P.per_range + ((int)blockIdx.y < P.longer);

  const int rows_a = (int)(P.m - m0 < BM ? P.m - m0 : BM), rows_b = (int)(P.n - n0 < BN ? P.n - n0 : BN);
  uint32_t offA[SA::LOADS], offB[SB::LOADS];
#pragma unroll
  for (int i = 0; i < SA::LOADS; ++i) offA[i] = (uint32_t)SA::global_offset(i, tid, P.lda, rows_a);
#pragma unroll
  for (int i = 0; i < SB::LOADS; ++i) offB[i] = (uint32_t)SB::global_offset(i, tid, P.ldb, rows_b);
  const int64_t stepA = A_KC ? 2 * KB : KB * P.lda, stepB = B_KC ? 2 * KB : KB * P.ldb;
  const uint8_t *gA = P.A + (A_KC ? m0 * P.lda : 2 * m0) + block0 * stepA;  // of the next block to load
  const uint8_t *gB = P.B + (B_KC ? n0 * P.ldb : 2 * n0) + block0 * stepB;
  const uint32_t lds0 = lds_address(smem) + wave * 1024;
  // the block that has to be fetched chunk by chunk: the last one of k when k ends inside it
  const int ragged = P.k % KB ? P.nkt - 1 - block0 : -1;

  v4i pieces[STAGED ? LOADS : 1];
  auto load = [&](int t) {  // into the registers, blocks in order
    const int left = t == ragged ? (int)(P.k % KB) : KB;
    auto fetch = [&](auto stage, bool kc, const uint8_t *g, int64_t ld, int extent, v4i *to) {
      using S = decltype(stage);
#pragma unroll
      for (int i = 0; i < S::LOADS; ++i) {
        int a, c;
        S::chunk_of(i, tid, a, c);
        const int end = 2 * (kc ? left : extent), have = kc ? extent : left;
        const int back = 16 * c + 16 > end ? 16 * c + 16 - end : 0;
        to[i] = load16(g + (a < have ? a : have - 1) * ld + (16 * c - back));
      }
    };
    fetch(SA{}, A_KC, gA, P.lda, rows_a, pieces);
    fetch(SB{}, B_KC, gB, P.ldb, rows_b, pieces + SA::LOADS);
    gA += stepA;
    gB += stepB;
  };
  auto place = [&](int t) {  // what was loaded last, block t, into its stage
    const int left = t == ragged ? (int)(P.k % KB) : KB;
    uint8_t *to = smem + (t % STAGES) * STAGE + 16 * tid;
    auto put = [&](auto stage, bool kc, int extent, const v4i *from, uint8_t *at) {
      using S = decltype(stage);
#pragma unroll
      for (int i = 0; i < S::LOADS; ++i) {
        int a, c;
        S::chunk_of(i, tid, a, c);
        const int end = 2 * (kc ? left : extent);
        v4i v = 16 * c + 16 > end ? shifted_down(from[i], 16 * c + 16 - end) : from[i];
        if (!kc && a >= left) v = v4i{0, 0, 0, 0};
        *reinterpret_cast<v4i *>(at + i * (16 * NT)) = v;
      }
    };
    put(SA{}, A_KC, rows_a, pieces, to);
    put(SB{}, B_KC, rows_b, pieces + SA::LOADS, to + SA::BYTES);
  };
  auto issue = [&](int t) {  // blocks in order
    const uint32_t to = lds0 + (uint32_t)(t % STAGES) * STAGE;
    if (t == ragged || P.wide_offsets) {
      const int left = t == ragged ? (int)(P.k % KB) : KB;
      const uint8_t *zero = reinterpret_cast<const uint8_t *>(&g_zero_chunk);
#pragma unroll
      for (int i = 0; i < SA::LOADS; ++i)
        dma16_at(SA::inside_k(i, tid, left) ? gA + SA::global_offset(i, tid, P.lda, rows_a) : zero, to + i * (16 * NT));
#pragma unroll
      for (int i = 0; i < SB::LOADS; ++i)
        dma16_at(SB::inside_k(i, tid, left) ? gB + SB::global_offset(i, tid, P.ldb, rows_b) : zero,
                 to + SA::BYTES + i * (16 * NT));
    } else {
#pragma unroll
      for (int i = 0; i < SA::LOADS; ++i) dma16(offA[i], gA, to + i * (16 * NT));
#pragma unroll
      for (int i = 0; i < SB::LOADS; ++i) dma16(offB[i], gB, to + SA::BYTES + i * (16 * NT));
    }
    gA += stepA;
    gB += stepB;
  };

  v4i hh[FM][FN], mid[FM][FN], ll[FM][FN];

  // WC waves share every row of A and WR every column of B; each sums its part of them over k.  A
  // wave takes its fragments in an order that puts its own part first (block i of its registers
  // is block i ^ flip of its sub-tile), so which fragments are summed is known at compile time.
  constexpr int SUMS_A = FM / WC, SUMS_B = FN / WR;
  static_assert(SUMS_A * WC == FM && SUMS_B * WR == FN, "every row and column is summed by one wave");
  const int flipA = wn * SUMS_A, flipB = wm * SUMS_B;
  int sum[SUMS_A + SUMS_B];  // of B's first
#pragma unroll
  for (int i = 0; i < SUMS_A + SUMS_B; ++i) sum[i] = 0;

  v4i hiA[FM], loA[FM], hiB[2][FN], loB[2][FN];
  v4i raw[FM + FN][2];
  const uint32_t laneA = SA::lane_base(lane), laneB = SB::lane_base(lane);
  // f: B's fragments, then A's.  (The scalar part is hidden from the compiler, which would
  // otherwise keep one vector register per fragment for the invariant part of the address.)
  auto read = [&](uint32_t stage, int f) {
    if (f < FN) {
      const int F = wn * FN + (f ^ flipB);
      uint32_t turn = SB::turn(F), rest = stage + SA::BYTES + SB::shift(F);
      if (!B_KC) asm volatile("" : "+s"(turn));
      asm volatile("" : "+s"(rest));
      SB::fragment(smem, (laneB ^ turn) + rest, raw[f]);
    } else {
      const int F = wm * FM + ((f - FN) ^ flipA);
      uint32_t turn = SA::turn(F), rest = stage + SA::shift(F);
      if (!A_KC) asm volatile("" : "+s"(turn));
      asm volatile("" : "+s"(rest));
      SA::fragment(smem, (laneA ^ turn) + rest, raw[f]);
    }
  };
  // A quarter of a fragment's split: sixteen of its bytes.  Inline assembly, as the matrix
  // instructions are, because that stays where it is put: the compiler would gather the work
  // where the operands arrive, or behind the next barrier, where the results are used.
  auto split = [&](int set, int f, int e) {
    int h, l;
    asm volatile(
        "v_perm_b32 %0, %3, %2, %4\n\t"
        "v_perm_b32 %1, %3, %2, %5\n\t"
        "v_xor_b32 %1, %6, %1"
        : "=&v"(h), "=&v"(l)
        : "v"(raw[f][e >> 1][2 * (e & 1)]), "v"(raw[f][e >> 1][2 * (e & 1) + 1]), "s"(0x07050301), "s"(0x06040200),
          "s"(0x80808080));
    if (f < FN) { hiB[set][f][e] = h; loB[set][f][e] = l; } else { hiA[f - FN][e] = h; loA[f - FN][e] = l; }
  };
  // the same quarter's part of the sum over k, where this wave sums the fragment
  auto add_up = [&](int f, int e) {
    if (f < FN ? f >= SUMS_B : f - FN >= SUMS_A) return;
    asm volatile(
        "v_dot2c_i32_i16 %0, %3, %1\n\t"
        "v_dot2c_i32_i16 %0, %3, %2"
        : "+v"(sum[f < FN ? f : SUMS_B + f - FN])
        : "v"(raw[f][e >> 1][2 * (e & 1)]), "v"(raw[f][e >> 1][2 * (e & 1) + 1]), "s"(0x00010001));
  };

  // prologue: the first blocks on their way, block 0 in registers
#pragma unroll
  for (int t = 0; t < STAGES; ++t)
    if (t < nkt) {
      if constexpr (STAGED) {
        if (t > 0) place(t - 1);
        load(t);
      } else {
        issue(t);
      }
    }
  if (STAGED && nkt < STAGES) place(nkt - 1);
  // (zeroed here, while the loads fly, and not right before the matrix instructions, which are
  // hidden from the compiler's wait states)
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      hh[i][j] = mid[i][j] = ll[i][j] = v4i{0, 0, 0, 0};
      asm volatile("" : "+a"(hh[i][j]), "+a"(mid[i][j]), "+a"(ll[i][j]));
    }
  if (STAGED) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else if (nkt >= STAGES) publish_barrier<(STAGES - 1) * LOADS>();
  else publish_barrier<0>();
  auto first = [&](int set) {  // set is a constant at both calls
#pragma unroll
    for (int f = 0; f < FM + FN; ++f) read(0, f);
#pragma unroll
    for (int f = 0; f < FM + FN; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        split(set, f, e);
        add_up(f, e);
      }
  };

  // The matrix instructions are inline assembly with the accumulators bound to the accumulation
  // registers: the register allocator otherwise moves some of the 96 (48) to and fro inside the
  // loop.  The compiler therefore inserts no wait states for them: an operand is written long
  // before its first use (the s_nop before the first and the last block see to the rest), and
  // the two that share an accumulator are five apart.
  auto mfma = [&](v4i &acc, const v4i &b, const v4i &a) {
    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
  };
  // instruction q of the four that multiply the planes of block (i, j), row by row of the
  // blocks, odd rows backwards so that only one operand changes from one block to the next; the
  // fourth is that of the block before
  constexpr int GROUPS = FM * FN;
  auto multiply = [&](int cur, int g, int q) {
    const int at = q == 3 ? g - 1 : g;
    if (at < 0 || at >= GROUPS) return;
    const int i = at / FN, j = (i & 1) ? FN - 1 - at % FN : at % FN;
    if (q == 0) mfma(hh[i][j], hiB[cur][j], hiA[i]);
    else if (q == 1) mfma(mid[i][j], loB[cur][j], hiA[i]);
    else if (q == 2) mfma(ll[i][j], loB[cur][j], loA[i]);
    else mfma(mid[i][j], hiB[cur][j], loA[i]);
  };

  // Block t is in registers, its B fragments in set `cur`.  At the barrier every wave has read block
  // t, so its stage takes block t + STAGES, and block t + 1 has landed.  A wave issues one
  // instruction in four clocks and a matrix instruction occupies the pipe for sixteen: beside
  // each there is room for three others, a quarter of a split or the reads of a fragment.
  // B's fragments of block t + 1 go into the other set from early on, A's into the registers of
  // the fragment whose row of blocks is done (two sets of both do not fit 128 registers, which is
  // what two waves to a SIMD leave beside the accumulators).
  auto step = [&](int t, auto cur_tag) {
    constexpr int cur = decltype(cur_tag)::value;
    if (STAGED) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else if (t + STAGES <= nkt) publish_barrier<(STAGES - 2) * LOADS>();
    else publish_barrier<0>();
    if constexpr (STAGED) {
      // (the stage that block t - 1 left a step ago)
      if (t + STAGES - 1 < nkt) place(t + STAGES - 1);
      if (t + STAGES < nkt) load(t + STAGES);
    } else if (t + STAGES < nkt) {
      issue(t + STAGES);
    }
    const uint32_t stage = (uint32_t)((t + 1) % STAGES) * STAGE;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g <= GROUPS + 1; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        multiply(cur, g, q);
#pragma unroll
        for (int f = 0; f < FM + FN; ++f) {
          const int at = f < FN ? (f + 1) * (GROUPS / 4) : FN * (f - FN + 1) + 1;  // group of the split
          if (q == 0 && (at > 2 ? at - 2 : 0) == g) read(stage, f);
          if (at == g) {
            split(cur ^ 1, f, q);
            add_up(f, q);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  // Steps come in pairs, one per fragment set, and the last block, which has no next one to
  // read, is always in set 0; with an even number of blocks, block 0 goes ahead in set 1.  (One
  // way out of the loop: where two ways meet, the accumulators are moved between registers.)
  int t = 0;
  if (nkt % 2 == 0) {
    first(1);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7" ::: "memory");
    step(0, std::integral_constant<int, 1>{});
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    t = 1;
  } else {
    first(0);
  }
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7" ::: "memory");
  for (; t + 1 < nkt; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    step(t + 1, std::integral_constant<int, 1>{});
  }
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7" ::: "memory");
#pragma unroll
  for (int g = 0; g <= GROUPS; ++g)
#pragma unroll
    for (int q = 0; q < 4; ++q) multiply(0, g, q);
  __builtin_amdgcn_sched_barrier(0);
  // the last results leave the pipe before anything reads them
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  publish_barrier<0>();  // no wave reads the stages any more: their LDS is reused from here on

  // Corrections, shared by the workgroup: BM words for the rows of the tile, BN for its columns.
  uint32_t *const rows = reinterpret_cast<uint32_t *>(smem), *const cols = rows + BM;
  constexpr int PITCH = WN + 4;  // words of a row of a wave's write-back patch
  uint32_t *const patch = cols + BN + wave * (16 * PITCH);
#pragma unroll
  for (int f = 0; f < SUMS_A + SUMS_B; ++f) {
    int total = sum[f] + __shfl_xor(sum[f], 16);
    total += __shfl_xor(total, 32);
    if (lane < 16) {
      if (f < SUMS_B) cols[wn * WN + 16 * (f ^ flipB) + lane] = 128u * (uint32_t)total;
      else rows[wm * WM + 16 * ((f - SUMS_B) ^ flipA) + lane] = 128u * (uint32_t)total - 16384u * KB * (uint32_t)nkt;
    }
  }
  __syncthreads();
  v4u acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
      acc[i][j] = (__builtin_bit_cast(v4u, hh[i][j]) << 16) + (__builtin_bit_cast(v4u, mid[i][j]) << 8) +
                  __builtin_bit_cast(v4u, ll[i][j]);

  if (__builtin_expect(P.splits > 1 && P.slots, 0)) {
    // Partial sums of a range of k: into the range's slot, with this range's corrections in
    // them; the workgroup that draws the tile's last ticket adds the other slots to its own
    // registers.  Slot accesses are device-scope, the ticket is drawn after the stores
    // are acknowledged and the other slots are read after it has come back.
    const int64_t tile = (int64_t)tm * P.walk.tiles_n + tn;
    int32_t *slots = P.slots + tile * P.splits * (int64_t)(BM * BN) + wave * (WM * WN);
    unsigned *ticket = P.tickets + tile;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const uint32_t r = rows[wm * WM + 16 * (i ^ flipA) + (lane & 15)];
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const v4u c = *reinterpret_cast<const v4u *>(cols + wn * WN + 16 * (j ^ flipB) + 4 * (lane >> 4));
        acc[i][j] += c + r;
      }
    }
    v4i *mine = reinterpret_cast<v4i *>(slots + (int64_t)blockIdx.y * (BM * BN)) + lane;
#pragma unroll
    for (int b = 0; b < FM * FN; ++b) store16_device_scope(mine + b * 64, __builtin_bit_cast(v4i, acc[b / FN][b % FN]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int *word = reinterpret_cast<int *>(smem);
    if (tid == 0) *word = atomicAdd(ticket, 1u) == (unsigned)(P.splits - 1) ? 1 : 0;
    __syncthreads();
    if (!*word) return;
    for (int r = 0; r < P.splits; ++r) {
      if (r == (int)blockIdx.y) continue;
      const v4i *other = reinterpret_cast<const v4i *>(slots + (int64_t)r * (BM * BN)) + lane;
#pragma unroll
      for (int b = 0; b < FM * FN; b += 4) {
        v4i v[4];
        load_slot_quad(other + b * 64, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[(b + e) / FN][(b + e) % FN] += __builtin_bit_cast(v4u, v[e]);
      }
    }
    if (tid == 0) atomicExch(ticket, 0u);  // every range has drawn: the counter is free again
    __syncthreads();
    // the corrections are in the sums
    for (int x = tid; x < BM + BN; x += NT) rows[x] = 0;
    __syncthreads();
  }

  if (__builtin_expect(P.splits > 1 && !P.slots, 0)) {
    // The range's sums into C, in any order the same bits.  Turned through the wave's patch as
    // below, so that an instruction adds to whole rows of the sub-tile: whole cache lines.
    static_assert(WN == 32, "two rows of the sub-tile to an instruction");
    const int64_t mw = m0 + wm * WM, col = n0 + wn * WN + (lane & 31);
    const uint32_t colc = cols[wn * WN + (lane & 31)];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row0 = 16 * (i ^ flipA);
      if (mw + row0 >= P.m) continue;  // wave-uniform
#pragma unroll
      for (int j = 0; j < FN; ++j)
        *reinterpret_cast<v4u *>(patch + (lane & 15) * PITCH + 16 * (j ^ flipB) + 4 * (lane >> 4)) = acc[i][j];
      // same wave wrote and reads: LDS operations of a wave complete in order
      asm volatile("" ::: "memory");
#pragma unroll 1
      for (int p = 0; p < 8; ++p) {
        const int r = 2 * p + (lane >> 5);
        const int64_t row = mw + row0 + r;
        const uint32_t val = patch[r * PITCH + (lane & 31)] + colc + rows[wm * WM + row0 + r];
        if (row < P.m && col < P.n)
          __hip_atomic_fetch_add(P.C + row * P.ldc + col, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    return;
  }

  // Sixteen rows at a time turned through the wave's patch, so that a store covers whole rows of
  // the sub-tile (non-temporal: C is not read again here).
  constexpr int LANES_PER_ROW = WN / 4, ROWS_PER_PASS = 64 / LANES_PER_ROW, PASSES = 16 / ROWS_PER_PASS;
  const int r0 = lane / LANES_PER_ROW, c0 = 4 * (lane % LANES_PER_ROW);
  const int64_t mw = m0 + wm * WM, nw = n0 + wn * WN;
  const v4u colc = *reinterpret_cast<const v4u *>(cols + wn * WN + c0);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row0 = 16 * (i ^ flipA);
    if (mw + row0 >= P.m) continue;  // wave-uniform
#pragma unroll
    for (int j = 0; j < FN; ++j)
      *reinterpret_cast<v4u *>(patch + (lane & 15) * PITCH + 16 * (j ^ flipB) + 4 * (lane >> 4)) = acc[i][j];
    // same wave wrote and reads: LDS operations of a wave complete in order
    v4u val[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int row = p * ROWS_PER_PASS + r0;
      val[p] = *reinterpret_cast<const v4u *>(patch + row * PITCH + c0) + colc + rows[wm * WM + row0 + row];
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int64_t row = mw + row0 + p * ROWS_PER_PASS + r0, col = nw + c0;
      if (row >= P.m) continue;
      uint32_t *dst = P.C + row * P.ldc + col;
      if (col + 3 < P.n) {
        if (P.accumulate) val[p] += __builtin_nontemporal_load(reinterpret_cast<const v4u_dword_aligned *>(dst));
        __builtin_nontemporal_store(val[p], reinterpret_cast<v4u_dword_aligned *>(dst));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < P.n) dst[e] = val[p][e] + (P.accumulate ? dst[e] : 0u);
      }
    }
  }
}

// Operands that cannot be fetched 16 bytes at a time, rewritten k-contiguous: row r of P (pitch
// kp elements, a multiple of 64) holds the k elements of row r of X, then zeros.  Both operands
// in one launch; 64 rows x 64 k at a time per workgroup, turned through LDS where X is strided.
struct Pack16Job {
  const int16_t *X;
  int64_t s_r, s_k, rows;
  int16_t *P;
  int64_t blocks;  // of 64 x 64 in this job
};
constexpr int64_t PACK_GRID = 1 << 22;  // workgroups at most: x 256 threads stays below 2^32

__global__ __launch_bounds__(256) void pack16_kernel(Pack16Job a, Pack16Job b, int64_t k, int64_t kp) {
  __shared__ short tile[64][66];
  const int tid = threadIdx.x;
  for (int64_t block = blockIdx.x; block < a.blocks + b.blocks; block += gridDim.x) {
    const bool first = block < a.blocks;
    const Pack16Job J = first ? a : b;
    const int64_t id = first ? block : block - a.blocks;
    const int64_t kts = kp / KB;
    const int64_t r0 = id / kts * 64, p0 = id % kts * KB;
    if (J.s_k != 1) {
      const int64_t r = r0 + (tid & 63);
#pragma unroll
      for (int e = 0; e < KB / 4; ++e) {
        const int q = 4 * e + (tid >> 6);
        tile[q][tid & 63] = r < J.rows && p0 + q < k ? J.X[r * J.s_r + (p0 + q) * J.s_k] : (short)0;
      }
      __syncthreads();
    }
    // eight k of one row per thread, twice: eight threads write the 128 bytes of a row
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t row = r0 + h * 32 + (tid >> 3), p = p0 + 8 * (tid & 7);
      if (row >= J.rows) continue;
      union { short e[8]; v4i v; } out;
      if (J.s_k != 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) out.e[e] = tile[8 * (tid & 7) + e][h * 32 + (tid >> 3)];
      } else if (p + 8 <= k) {
        const s16x8 x = *reinterpret_cast<const s16x8 *>(J.X + row * J.s_r + p);
#pragma unroll
        for (int e = 0; e < 8; ++e) out.e[e] = x.v[e];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) out.e[e] = p + e < k ? J.X[row * J.s_r + p + e] : (short)0;
      }
      *reinterpret_cast<v4i *>(J.P + row * kp + p) = out.v;
    }
    if (J.s_k != 1) __syncthreads();  // the next block's loads overwrite the tile
  }
}

// Can the kernel fetch the operand 16 bytes at a time as it is stored?
bool streamable(const int16_t *X, int64_t s_r, int64_t s_k, int64_t rows, int64_t k) {
  if (reinterpret_cast<uintptr_t>(X) % 16) return false;
  if (s_k == 1) return s_r % 8 == 0 && k % 8 == 0;
  return s_k % 8 == 0 && rows % 8 == 0;
}

template <int WR, int WC, int FM, int FN, bool STAGED = false>
hipError_t launch_tiles(S16Params P, bool a_kc, bool b_kc, hipStream_t s) {
  constexpr int BM = 16 * FM * WR, BN = 16 * FN * WC;
  const int64_t tiles = (int64_t)P.walk.tiles_m * P.walk.tiles_n;
  if (tiles > ((int64_t)1 << 30)) return hipErrorInvalidValue;
  auto far = [](int64_t ld, int rows) { return (int64_t)(rows - 1) * ld + 2 * KB >= ((int64_t)1 << 32); };
  P.per_range = P.nkt / P.splits;
  P.longer = P.nkt % P.splits;
  P.wide_offsets = far(P.lda, a_kc ? BM : KB) || far(P.ldb, b_kc ? BN : KB);
  void (*kern)(S16Params) =
      a_kc ? (b_kc ? s16_kernel<WR, WC, FM, FN, true, true, STAGED> : s16_kernel<WR, WC, FM, FN, true, false, STAGED>)
           : (b_kc ? s16_kernel<WR, WC, FM, FN, false, true, STAGED> : s16_kernel<WR, WC, FM, FN, false, false, STAGED>);
  const size_t lds = (size_t)STAGES * (BM + BN) * 2 * KB;
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds);
  if (e != hipSuccess) return e;
  return launch_with(reinterpret_cast<const void *>(kern), dim3((unsigned)((tiles + 7) / 8 * 8), (unsigned)P.splits), 64 * WR * WC,
                     lds, s, &P);
}

}  // namespace

hipError_t launch_s16(const S16Problem &p, hipStream_t s) {
  const int64_t kp = (p.k + KB - 1) / KB * KB;
  S16Params P;
  P.C = reinterpret_cast<uint32_t *>(p.C);
  P.ldc = p.ldc;
  P.m = p.m;
  P.n = p.n;
  P.k = p.k;
  P.accumulate = p.accumulate;
  const int16_t *X[2] = {p.A, p.B};
  int64_t s_r[2] = {p.a_sm, p.b_sn}, s_k[2] = {p.a_sk, p.b_sk};
  const int64_t rows[2] = {p.m, p.n};
  uint8_t *ws = static_cast<uint8_t *>(p.ws), *const end = ws + p.ws_bytes;
  const int64_t cus = compute_units();
  auto tiles = [&](int64_t side) { return ((p.m + side - 1) / side) * ((p.n + side - 1) / side); };
  // Operands that cannot be streamed are read at their own alignment where that takes less than a launch that
  // rewrites them and one more pass over them: 64 x 64 tiles each read theirs again, so up to a product of
  // tiles and k.  Over 160 drawn products 0.78 of the time; us, rewritten and as they are: (128, 204, 64) 8.8 and 4.9,
  // (799, 757, 602) 17.6 and 13.1, (512, 1603, 1792) 27.2 and 27.0, but (682, 2790, 2848) 54 and 60,
  // (2965, 1216, 2153) 58 and 74.  One or two tiles under a very long k pay more for a block through registers than the
  // rewriting costs: over 5000 products, those of one tile, k = 4096 to 8192, 1.01 of the time overwriting and 0.88
  // accumulating, up to 16384 1.07 and 0.97; (10, 10, 14213) 21.9 and 28.2, accumulating (14, 15, 14340) 21.4 and 27.4.
  bool staged = !streamable(X[0], s_r[0], s_k[0], rows[0], p.k) || !streamable(X[1], s_r[1], s_k[1], rows[1], p.k);
  for (int i = 0; i < 2; ++i) staged = staged && (s_k[i] == 1 ? p.k : rows[i]) >= 8;
  staged = staged && (!std::strcmp(tuning().variant, "s16_staged") ||
                      (!*tuning().variant && tuning().splitk == 0 && (double)tiles(64) * (double)p.k <= 1600.0 * (double)cus &&
                       p.k <= (p.accumulate ? 8192 : 4096) * tiles(64)));
  // what cannot be streamed is rewritten into the front of the workspace first
  Pack16Job job[2] = {};
  for (int i = 0; i < 2 && !staged; ++i) {
    if (streamable(X[i], s_r[i], s_k[i], rows[i], p.k)) continue;
    const size_t bytes = (size_t)((rows[i] * kp * 2 + 255) / 256 * 256);
    if (bytes > (size_t)(end - ws)) return hipErrorInvalidValue;
    job[i] = {X[i], s_r[i], s_k[i], rows[i], reinterpret_cast<int16_t *>(ws), (rows[i] + 63) / 64 * (kp / KB)};
    X[i] = job[i].P;
    s_r[i] = kp;
    s_k[i] = 1;
    ws += bytes;
  }
  if (const int64_t blocks = job[0].blocks + job[1].blocks) {
    const unsigned grid = (unsigned)(blocks < PACK_GRID ? blocks : PACK_GRID);
    hipLaunchKernelGGL(pack16_kernel, dim3(grid), dim3(256), 0, s, job[0], job[1], p.k, kp);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // (a packed row is zero from k on; with both packed no block ends early)
    if (job[0].blocks && job[1].blocks) P.k = kp;
  }
  const bool a_kc = s_k[0] == 1, b_kc = s_k[1] == 1;
  P.A = reinterpret_cast<const uint8_t *>(X[0]);
  P.B = reinterpret_cast<const uint8_t *>(X[1]);
  P.lda = 2 * (a_kc ? s_r[0] : s_k[0]);
  P.ldb = 2 * (b_kc ? s_r[1] : s_k[1]);
  P.nkt = (int)(kp / KB);
  P.splits = 1;
  P.slots = nullptr;
  P.tickets = nullptr;

  // Tiles.  One 128 x 128 workgroup has a compute unit to itself, three 64 x 64 ones share it: the
  // large tile only where its rounds are nearly full.  Measured, us, 128 against 64: 2048^2 x 512
  // (256 tiles of 128: one round) 14.0 and 15.3, 4096^2 x 1024 (four rounds) 84 and 91; but
  // (1024, 3072, 768) (three quarters of a round) 17.0 and 15.7, 2304^2 x 1024 (1.27) 40 and 34,
  // 3000^2 x 1000 (2.25) 68 and 58.  A fourth or fifth stage changes neither.
  bool large = 10 * tiles(128) >= 9 * cus * ((tiles(128) + cus - 1) / cus);
  if (!std::strcmp(tuning().variant, "s16_128")) large = true;  // pinned by tests and tuning runs
  if (!std::strcmp(tuning().variant, "s16_64") || staged) large = false;
  const int64_t side = large ? 128 : 64, count = tiles(side);
  P.walk = tile_walk((p.m + side - 1) / side, (p.n + side - 1) / side);
  // Ranges of k, where that gives a compute unit at most three workgroups (a wave alone on its SIMD
  // issues at half rate): at most four, eight of few tiles, sixteen of very few with a very long k,
  // each of enough blocks to pay for the exchange.  Measured through slots, us, with 1 / 2 / 4 / 8 / 16
  // ranges of k = 4096: 16 tiles 31 / 19 / 13.3 / 11.9 / 14.2, 64 tiles 31 / 20 / 15.1 / 15.4 / 19,
  // 128 tiles 32 / 20 / 18 / 21 / 31, 192 tiles 32 / 26 / 23 / 27 / 43; of k = 1024: 64 tiles 10.8 / 9.4 /
  // 9.4, 128 tiles 10.9 / 10.0 / 10.1, 192 tiles 11.0 / 11.3 / 11.2; of k = 16384: 16 tiles
  // 112 / 60 / 34 / 21.9 / 19.5.
  const int64_t most = count > 32 ? 4 : (count > 16 || P.nkt < 256 ? 8 : 16);
  int64_t splits = large ? 1 : 3 * cus / count, blocks = count / 16 > 4 ? count / 16 : 4;
  if (splits > most) splits = most;
  if (count > 16 && P.nkt < 12) splits = 1;
  if (tuning().splitk > 0) { splits = tuning().splitk; blocks = 4; }
  if (splits > P.nkt / blocks) splits = P.nkt / blocks;
  if (splits > 1024) splits = 1024;
  if (splits > 1) {
    // The ranges meet in slots, where the workspace has room for at least half of them.  (A captured
    // call, whose counters are never handed out again, does as well without.)
    const int64_t room = (end - ws) / (count * side * side * 4), fit = room < splits ? room : splits;
    // (Accumulating into C from operands read as they are: without slots, which cost 0.84 of the time of rewritten operands
    // over 2494 products where adding takes 0.77; (72, 151, 1289) 9.2 rewritten, 14.3 through slots.)
    if (!(staged && p.accumulate) && fit > 1 && 2 * fit >= splits && !being_captured(s) &&
        splitk_tickets(count, s, nullptr, &P.tickets) == hipSuccess) {
      P.slots = reinterpret_cast<int32_t *>(ws);
      splits = fit;
    } else if (!p.accumulate) {
      // Otherwise they add into C, which an overwriting call has zeroed first: 2 us more, which a
      // short k does not save.  Measured, us, k whole and in the ranges chosen above: k = 512 16 tiles
      // 7.5 and 7.7; k = 1024 16 tiles 10.6 and 7.7, 64 tiles 10.7 and 9.5, 128 tiles 10.8 and 11.5;
      // k = 2048 128 tiles 17.7 and 14.1, 192 tiles 17.8 and 17.9; k = 4096 192 tiles 32 and 26.
      if (P.nkt < 12 + count / 8 && tuning().splitk == 0) {
        splits = 1;
      } else {
        Problem z;
        z.m = p.m; z.n = p.n; z.k = 0; z.C = p.C; z.ldc = p.ldc;
        const hipError_t e = launch_fill_zero(z, s);
        if (e != hipSuccess) return e;
      }
    }
    P.splits = (int)splits;
  }
  if (staged) return launch_tiles<2, 2, 2, 2, true>(P, a_kc, b_kc, s);
  return large ? launch_tiles<2, 4, 4, 2>(P, a_kc, b_kc, s) : launch_tiles<2, 2, 2, 2>(P, a_kc, b_kc, s);
}

}  // namespace mip
