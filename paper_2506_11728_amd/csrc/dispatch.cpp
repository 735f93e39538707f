// Which kernel serves which problem: eligibility, tile shape, k ranges.  Host only.
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "mip_internal.h"
#include "tuning.h"

namespace mip {

bool dma_eligible(const Problem &p, Shape shape) {
  switch (shape) {
    case SHAPE_256: return dma_eligible_256x256(p);
    case SHAPE_128: return dma_eligible_128x128(p);
    case SHAPE_64: return dma_eligible_64x64(p);
    case SHAPE_64X256: return dma_eligible_64x256(p);
    case SHAPE_256X64: return dma_eligible_256x64(p);
    case SHAPE_64X128: return dma_eligible_64x128(p);
    case SHAPE_128X64: return dma_eligible_128x64(p);
    default: return false;
  }
}

hipError_t launch_dma(const Problem &p, Shape shape, int splits, hipStream_t s) {
  switch (shape) {
    case SHAPE_256: return launch_dma_256x256(p, splits, s);
    case SHAPE_128: return launch_dma_128x128(p, splits, s);
    case SHAPE_64: return launch_dma_64x64(p, splits, s);
    case SHAPE_64X256: return launch_dma_64x256(p, splits, s);
    case SHAPE_256X64: return launch_dma_256x64(p, splits, s);
    case SHAPE_64X128: return launch_dma_64x128(p, splits, s);
    case SHAPE_128X64: return launch_dma_128x64(p, splits, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_wave_32x32(const Problem &p, bool streamed, hipStream_t s);
hipError_t launch_wave_32x64(const Problem &p, bool streamed, hipStream_t s);

hipError_t launch_wave(const Problem &p, Wave wave, bool streamed, hipStream_t s) {
  switch (wave) {
    case WAVE_32: return launch_wave_32x32(p, streamed, s);
    case WAVE_32X64: return launch_wave_32x64(p, streamed, s);
    default: return hipErrorInvalidValue;
  }
}

static bool wave_streamed_eligible(const Problem &p) {
  const int64_t lda = p.a_sk == 1 ? p.a_sm : p.a_sk, ldb = p.b_sk == 1 ? p.b_sn : p.b_sk;
  return dma_eligible(p, SHAPE_64) && (p.conv || 128 * lda < ((int64_t)1 << 31)) && 128 * ldb < ((int64_t)1 << 31);
}

// Sixteen bytes along k or, where the other index is contiguous, along that: pieces at an edge are fetched
// from further inside (wave_tile.h).
bool wave_staged_eligible(const Problem &p) {
  if (p.conv || p.k < 1) return false;
  if ((p.a_sk == 1 ? p.k : p.m) < 16 || (p.b_sk == 1 ? p.k : p.n) < 16) return false;
  const int64_t lda = p.a_sk == 1 ? p.a_sm : p.a_sk, ldb = p.b_sk == 1 ? p.b_sn : p.b_sk;
  return 128 * lda < ((int64_t)1 << 31) && 128 * ldb < ((int64_t)1 << 31);
}

static const char *const kShapeNames[SHAPE_COUNT] = {"256", "128", "64", "64x256", "256x64",
                                                     "64x128", "128x64"};
static const int64_t kShapeRows[SHAPE_COUNT] = {256, 128, 64, 64, 256, 64, 128};
static const int64_t kShapeCols[SHAPE_COUNT] = {256, 128, 64, 256, 64, 128, 64};

const char *plan_name(const Plan &plan) {
  static const char *const staged[SHAPE_COUNT] = {"mfma_tile256", "mfma_tile128", "mfma_tile64",
                                                  "mfma_tile64x256", "mfma_tile256x64",
                                                  "mfma_tile64x128", "mfma_tile128x64"};
  static const char *const dma[SHAPE_COUNT] = {"mfma_dma256", "mfma_dma128", "mfma_dma64",
                                               "mfma_dma64x256", "mfma_dma256x64",
                                               "mfma_dma64x128", "mfma_dma128x64"};
  switch (plan.kind) {
    case KIND_NONE: return "none";
    case KIND_FILL: return "fill_zero";
    case KIND_SIMPLE: return "simple";
    case KIND_STAGED: return staged[plan.shape];
    case KIND_DMA: return dma[plan.shape];
    case KIND_DMA_K128: return plan.shape == SHAPE_128 ? "mfma_dma128_k128" : "mfma_dma256_k128";
    case KIND_DMA_K128_SPLIT:
      switch (plan.shape) {
        case SHAPE_256: return "mfma_dma256_k128_ragged";
        case SHAPE_256X192: return "mfma_dma256x192_k128";
        case SHAPE_192X256: return "mfma_dma192x256_k128";
        case SHAPE_192: return "mfma_dma192_k128";
        default: return "mfma_dma128_k128_split";
      }
    case KIND_SLAB: return plan.splits == 4 ? "mfma_slab64" : (plan.splits == 2 ? "mfma_slab32" : "mfma_slab16");
    default: return "?";
  }
}

// The tuning value MIPGEMM_VARIANT pins the kernel (tuning and tests): "simple", "dma256k128",
// "dma128k128" (the same kernel on 128 x 128 tiles), "dma128k128split" (its general form with k
// ranges), "dma256k128ragged", "dma256x192k128", "dma192x256k128", "dma192k128" (the general form on
// tiles of those sides), "slab16" / "slab32" / "slab64" (the skinny-m kernel with that slab width),
// "wave32" / "wave32x64" (tiles whose waves split k),
// "tile<shape>" (register-staged) or "dma<shape>" (direct-to-LDS) with <shape> one of
// 256, 128, 64, 64x256, 256x64, 64x128, 128x64.  A dma variant only applies to problems it is
// eligible for; others fall back to the staged kernel of the same shape.
// MIPGEMM_SPLITK pins the number of k ranges of the tile kernels.
static int forced_splits() { return tuning().splitk; }

// k ranges for the 128 x 128 tiles with 128-deep blocks: workgroups for about three quarters
// of the compute units, at most eight ranges (every range adds a whole C through atomics), each
// of at least eight blocks.  Measured best, ranges at tiles: 6-8 at 16, 6 at 24, 4 at 36 to 52,
// 3-4 at 64, 2 at 96.
static int k128_ranges(const Problem &p) {
  if (forced_splits() > 0) return forced_splits();
  const int64_t tiles = ((p.m + 127) / 128) * ((p.n + 127) / 128);
  const int64_t blocks = p.k / 128;
  int64_t sp = (3 * compute_units() / 4 + tiles / 2) / tiles;
  if (sp > 8) sp = 8;
  if (sp > blocks / 8) sp = blocks / 8;
  return sp > 1 ? (int)sp : 1;
}

static bool forced_plan(const Problem &p, Plan *plan) {
  const char *e = tuning().variant;
  if (!*e) return false;
  if (!std::strcmp(e, "simple")) { *plan = {KIND_SIMPLE, SHAPE_64, 1}; return true; }
  if (!std::strcmp(e, "dma256k128")) {
    if (!dma_k128_eligible(p)) return false;
    *plan = {KIND_DMA_K128, SHAPE_256, 1};
    return true;
  }
  if (!std::strcmp(e, "dma128k128")) {
    if (!dma_k128_eligible(p, true)) return false;
    *plan = {KIND_DMA_K128, SHAPE_128, 1};
    return true;
  }
  if (!std::strcmp(e, "dma128k128split")) {
    if (!dma_k128_split_eligible(p)) return false;
    *plan = {KIND_DMA_K128_SPLIT, SHAPE_128, k128_ranges(p)};
    return true;
  }
  if (!std::strcmp(e, "dma256k128ragged")) {
    if (!dma_k128_split_eligible(p, true)) return false;
    *plan = {KIND_DMA_K128_SPLIT, SHAPE_256, 1};
    return true;
  }
  static const struct { const char *name; Shape shape; } with_192[3] = {
      {"dma256x192k128", SHAPE_256X192}, {"dma192x256k128", SHAPE_192X256}, {"dma192k128", SHAPE_192}};
  for (const auto &v : with_192)
    if (!std::strcmp(e, v.name)) {
      if (!dma_k128_split_eligible(p, true)) return false;
      *plan = {KIND_DMA_K128_SPLIT, v.shape, 1};
      return true;
    }
  if (!std::strcmp(e, "slab16") || !std::strcmp(e, "slab32") || !std::strcmp(e, "slab64")) {
    const int nt = e[4] == '6' ? 4 : (e[4] == '3' ? 2 : 1);
    if (!slab_eligible(p, nt)) return false;
    *plan = {KIND_SLAB, SHAPE_64, nt};
    return true;
  }
  static const struct { const char *name; Wave wave; } waves[2] = {{"wave32", WAVE_32}, {"wave32x64", WAVE_32X64}};
  for (const auto &v : waves)
    if (!std::strcmp(e, v.name)) {
      const bool streamed = wave_streamed_eligible(p);
      if (!streamed && !wave_staged_eligible(p)) return false;
      *plan = {streamed ? KIND_DMA : KIND_STAGED, SHAPE_64, 1, v.wave};
      return true;
    }
  const bool want_dma = !std::strncmp(e, "dma", 3);
  if (!want_dma && std::strncmp(e, "tile", 4)) return false;
  const char *shape = e + (want_dma ? 3 : 4);
  for (int i = 0; i < SHAPE_COUNT; ++i)
    if (!std::strcmp(shape, kShapeNames[i])) {
      const Shape sh = static_cast<Shape>(i);
      *plan = {want_dma && dma_eligible(p, sh) ? KIND_DMA : KIND_STAGED, sh, 1};
      return true;
    }
  return false;
}

hipError_t allow_dynamic_lds(const void *kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  struct Granted { const void *kernel; int device; size_t bytes; };
  static std::mutex lock;
  static std::vector<Granted> granted;  // a few dozen kernels at most
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> guard(lock);
    Granted *known = nullptr;
    for (Granted &g : granted)
      if (g.kernel == kernel && g.device == device) known = &g;
    if (known && known->bytes >= bytes) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess && known) known->bytes = bytes;
    else if (e == hipSuccess) granted.push_back({kernel, device, bytes});
  }
  if (e != hipSuccess) (void)hipGetLastError();  // (as in launch_with)
  return e;
}

// Compute units of the current device, asked once; 256 (an MI355X) where no device answers,
// as on a build host that only names kernels.
int64_t compute_units() {
  static std::once_flag once;
  static int64_t count = 256;
  std::call_once(once, [] {
    int device = 0, n = 0;
    if (hipGetDevice(&device) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && n > 0)
      count = n;
    (void)hipGetLastError();  // a missing device must not surface in a later call
  });
  return count;
}

// over all problems of a batch: what the chip sees is their sum
static int64_t tile_count(const Problem &p, Shape s) {
  return ((p.m + kShapeRows[s] - 1) / kShapeRows[s]) * ((p.n + kShapeCols[s] - 1) / kShapeCols[s]) *
         (p.batch > 1 ? p.batch : 1);
}

// A 64 x 64 tile plan of few tiles: the form whose waves split k, where that is the faster one.  One workgroup
// of it goes through k eight steps of 128 at a time, so that a chain of k blocks that takes a 64 x 64
// tile 0.115 us per 64 takes a few microseconds whatever its length, without a workspace and a second
// launch; but a workgroup has a compute unit to itself, and what it takes in per multiply-accumulate
// grows as the tile shrinks, most for a strided operand, whose pieces of a row are 32 or 64 bytes.
// So: the smallest tile of which there is one round, for a k that is long enough, and no longer than what the
// 64 x 64 tiles need that can split k over workgroups (through atomics, cheapest into an int32 C that needs no
// zero fill and into one of few rows, or through slots).  The fewer the tiles, the more ranges of k
// there is room for, and the shorter the k up to which one workgroup to a tile keeps up.
// Measured over 16000 products, batches and convolutions of up to 1200 tiles of 32 x 32 (k = 16 to 60000), aligned and
// not, the rule takes 0.793 of the time without it; 304 are slower by more than 5 %, 88 by more than a tenth.
// (Limits for unaligned operands drawn again after that: of 4300 such products of up to 768 tiles, k = 512 to 6000, 54 are
// slower by more than 6 % than before there was this form, 31 by more than a tenth; on average they take 0.61 of the time.)
// us, before and after: (512, 512, 2048) k-contiguous 6.5 -> 4.2, (256, 256, 1024) 4.4 -> 3.7, (64, 4096, 11008) u8
// packed 14.8 -> 12.9, row-major B (1024, 512, 4096) 12.3 -> 9.9;
// a 3 x 3 convolution of 7 x 7 x 512 at batch 8 19.7 -> 7.4; unaligned (32, 256, 3600) to int8 35 -> 12.9,
// (42, 2368, 2112) 22.9 -> 6.5, (1024, 70, 1024) 18.2 -> 4.8, (459, 1024, 836) packed before 7.9 -> 6.1.
// On the other side of the lines, us without this form and with it: (1024, 1024, 1024) 5.1 and 6.6, (1024, 512, 1024)
// row-major 4.75 and 5.1, (304, 208, 6144) column-major A 16.8 packed and 21; a long k: (14, 512, 11136) 6.1 and 7.6, 11 x 11
// filters over 448 channels, 176 positions and 7 filters, 11.0 and 38, (64, 1162, 53696) 28 and 46; adding into C:
// (2, 246, 3712) 3.6 and 5.2, (206, 32, 3584) 4.1 and 5.2, unaligned (128, 128, 1472) with both operands strided
// 4.9 and 8.5; 21 unaligned products of (357, 64, 64) 4.2 and 7.8.
static Wave wave_form(const Problem &p, bool streamed) {
  if (p.k < 1 || (p.batch > 1 && p.out_float == 2)) return WAVE_NONE;
  const int64_t cus = compute_units(), k = p.k, batch = p.batch > 1 ? p.batch : 1;
  auto tiles = [&](int64_t bm, int64_t bn) { return ((p.m + bm - 1) / bm) * ((p.n + bn - 1) / bn) * batch; };
  const int64_t short_side = p.m < p.n ? p.m : p.n, target = short_side <= 16 ? 2 * cus : cus;
  const bool adds = p.accumulate && !p.out_float;
  const bool may_split = (!p.out_float || (p.ws && streamed)) &&
                         (p.accumulate || p.out_float ? 2 * tiles(64, 64) <= target : 2 * tiles(64, 64) < target);
  const int64_t any = INT64_MAX / 4, small = tiles(32, 32);
  const int strided = (p.a_sk != 1) + (p.b_sk != 1);
  if (streamed) {
    if (!wave_streamed_eligible(p)) return WAVE_NONE;
    // (row-major (192, 448, 3904), 84 tiles of 32 x 32: 8.2 us on 21 of 64 x 64 in four ranges, 10.0 here)
    int64_t most = any;
    if (may_split && adds) {
      most = strided == 2 ? 1792 : (strided ? 2560 : (4 * small <= cus ? 2048 : 4096));
    } else if (may_split && strided) {
      most = 4 * small <= cus ? (strided == 2 ? 3072 : 4096) : (strided == 2 ? 2048 : 3072);
    } else if (may_split && short_side <= 16) {
      if (4 * small <= cus) most = 5120;
    } else if (may_split && 2 * small <= cus) {
      most = 16 * small <= cus ? 10240 : 16384;
    }
    if (small <= cus) return k < most && (!p.conv || k >= 512) ? WAVE_32 : WAVE_NONE;
    if (tiles(32, 64) <= cus && p.a_sk == 1) return k >= (strided ? 1536 : 1024) && k < 2 * most ? WAVE_32X64 : WAVE_NONE;
    return WAVE_NONE;
  }
  if (!wave_staged_eligible(p) || tuning().pack > 0) return WAVE_NONE;
  // (with a workspace, larger products are packed)
  const bool packable = packing_serves(p), whole = p.m % 64 == 0 && p.n % 64 == 0, few = 4 * small <= cus;
  // (the 64 x 64 tiles lose most where a strided operand ends inside a 16-byte piece)
  const bool whole_pieces = (p.a_sk == 1 || p.m % 16 == 0) && (p.b_sk == 1 || p.n % 16 == 0);
  int64_t most = any;
  if (may_split && adds)
    most = few ? (strided && whole_pieces ? 768 : 1024) : (strided == 2 && whole ? 512 : 1536);
  else if (may_split)
    most = few && strided && whole_pieces ? 2048 : (64 * small <= cus || (8 * small <= cus && !strided) ? 3072 : 4096);
  if (packable && most > 4096) most = 4096;
  // (both operands strided and a short k: packed, a choice that a test names; (300, 200, 333) 5.8 us, 4.3 here)
  if (packable && strided == 2 && k < 512) return WAVE_NONE;
  // A batch of short sums is a matter of how many workgroups start, and these have twice the threads.
  if (small <= cus) return k < most && (batch == 1 || k > 64) ? WAVE_32 : WAVE_NONE;
  if (packable) return WAVE_NONE;
  if (tiles(32, 64) <= cus && k < most)
    return k >= (batch > 1 ? (p.accumulate ? 768 : 192) : 96) ? WAVE_32X64 : WAVE_NONE;
  // Two or three rounds of these, against one of 64 x 64 tiles, which keep up where strided operands fill them: in ranges of k,
  // adding into C ((512, 640, 3097) with both operands strided 14.5 us, 25.7 here, 17 of 24 such products slower; one
  // strided, k = 1536 to 4096, 1.14 of the time over 33, 0.81 below) or under a long k (1.08 of the time over 25 from
  // k = 4096 on, 0.55 below); and under a short k with an unsigned operand, whose partner every wave
  // sums up ((512, 1152, 640) 8.4 and 10.7; 48 such 1.04, all others 0.51).
  const bool filled = strided == 2 ? whole : strided && (p.a_sk != 1 ? p.m : p.n) % 128 == 0;
  if (may_split && filled && (adds ? strided == 2 || k >= 1536 : k >= 4096)) return WAVE_NONE;
  if (small > 2 * cus && k < 2048 && whole_pieces && p.n % 64 == 0 && (p.a_unsigned || p.b_unsigned || strided == 2)) return WAVE_NONE;
  return small <= 3 * cus && k >= 512 ? WAVE_32 : WAVE_NONE;
}

size_t splitk_slot_bytes(const Problem &p, const Plan &plan) {
  // (int32 outputs add into C, and 256 x 256 tiles have no slots)
  if (plan.kind != KIND_DMA || plan.shape == SHAPE_256 || plan.splits < 2 || !p.out_float) return 0;
  const int64_t bm = kShapeRows[plan.shape], bn = kShapeCols[plan.shape];
  const int64_t tiles = ((p.m + bm - 1) / bm) * ((p.n + bn - 1) / bn) * (p.batch > 1 ? p.batch : 1);
  const double bytes = (double)tiles * ((double)plan.splits * (double)(bm * bn * 4) + sizeof(unsigned));
  return bytes < 1.0e15 ? (size_t)bytes : 0;
}

// A few rows of A: width of the slabs, in blocks of 16 columns, where a workgroup per slab of B is
// the better plan, 0 where tiles are.  One pass over B in one launch, without atomics or a zero
// fill, against tiles that share A between more columns and split k over workgroups.
//
// The width is the narrowest of which one round of compute units holds all slabs: a narrower one leaves a
// second round mostly idle, a wider one has fewer bytes of B in flight.  Up to 16 rows, where the
// shallow rings put two workgroups on a compute unit, more slabs than that do no harm.
//
// Where slabs are taken was measured on 14 to 36 widths n, 7 to 10 depths k and 5 to 8 row counts
// each, with operands that stay in the last-level cache ("warm") and with operands that come from
// memory ("cold", what decoding sees: the weights of a layer are gone when its turn comes again).
// us, cold / warm, slabs against tiles, (m, n, k), B k-contiguous:
//   (32, 8192, 4096) 10.7 / 6.8 against 17.7 / 12.1, (24, 12288, 4096) 15.0 / 11.8 against 19.2 / 12.8;
//   but (24, 12288, 1024) 6.8 / 5.2 against 7.3 / 4.8 and, a third of a second round with more than
//   16 rows, (24, 22016, 3072) 22 / 17.6 against 23 / 15.0.
// B row-major, whose rows a slab takes in pieces of 16 bytes a column block, where the tiles of 256
// columns take whole lines:
//   (16, 8192, 2048) 10.0 / 5.4 against 10.5 / 6.7,
//   (8, 12288, 2048) 11.7 / 7.1 against 12.8 / 8.5, but (16, 6144, 3072) 13.7 / 8.0 against 11.0 / 7.8
//   and (8, 12288, 4096) 19.6 / 13.1 against 15.3 / 13.3.
// How deep they may go depends on the leading dimension: pieces whole multiples of 512 bytes apart
// meet in few memory channels: (16, 11264, 3072) 1.18 times the tiles' cold time, (16, 12288, 3072) at
// ld = 12352 0.90.
// Adding into an int32 C needs no zero fill, and the tiles win or tie except against slabs of 64 columns of
// a k-contiguous B: (16, 11008, 4096) 12.5 / 9.9 against 14.1 / 11.7; row-major
// (1, 10240, 4096) 21 / 13.4 against 11.6 / 9.7.
static int slab_width(const Problem &p) {
  if (p.m > 64 || !slab_eligible(p, 1)) return 0;
  const int64_t cus = compute_units(), m = p.m, n = p.n, k = p.k;
  const bool kc = p.b_sk == 1;
  const bool into_int32 = p.accumulate && !p.out_float;
  const bool adds_in_place = into_int32 && k >= (m >= 16 ? 1024 : 1536);
  auto slabs = [&](int nt) { return n / (16 * nt); };
  int width = slabs(1) <= cus ? 1 : (slabs(2) <= cus ? 2 : 4);
  if (!slab_eligible(p, width)) width = 1;
  const bool one_round = slabs(width) <= cus;
  // Up to 16 rows the tiles of 256 columns, in as many ranges of k as fill the chip, may leave an XCD
  // (an eighth of it) a second round: (16, 12352, 4096) row-major 14.9 / 11.0 on slabs, 20.7 / 17.5 on tiles.
  const int64_t tiles = (n + 255) / 256;
  const bool crowded = m <= 16 && k / 512 * tiles >= cus && (tiles + 7) / 8 * (cus / tiles) > cus / 8;
  if (kc && slabs(1) >= 128) {
    if (m <= 16) {
      // (at most four rows from k = 4096 on: narrow slabs, two workgroups to a compute unit, come
      // near wide ones and pass them at k = 8192: (1, 11008, 4096) 11.7 / 9.4 and 11.1 / 9.1,
      // (1, 11008, 8192) 17.8 / 14.9 and 19.4 / 15.1)
      if (!adds_in_place) return m <= 4 && width == 4 && one_round && k >= 4096 ? 1 : width;
      if (width == 4 && (one_round || k <= 3072 || 3 * slabs(4) >= 4 * cus || crowded)) return 4;
    } else if (m <= 32) {
      if (width < 4) {
        if (one_round && !adds_in_place && (p.out_float || slabs(1) >= 192 || k <= 8192)) return width;
      } else if (one_round) {
        if (k >= 2048 && (slabs(4) <= 240 || k < 2560 || k >= 5120)) return 4;
      } else if (k >= 8192 && 10 * slabs(4) >= 9 * ((slabs(4) + cus - 1) / cus * cus)) {
        return 4;  // (the rounds nearly full: (24, 32000, 8192) 0.94 of the tiles' time, (24, 22016, 8192) 1.07)
      }
    } else if (width < 4 && one_round && !adds_in_place && (p.packed_weights || p.out_float) && k >= 2048 &&
               k <= 8192) {
      // (above 32 rows for a float output, which the tiles combine through slots, and for packed weights)
      if (width == 1 && (p.out_float || slabs(1) >= 192 || k <= 5120)) return 1;
      if (width == 2 && (p.packed_weights || slabs(2) >= 164 || k <= 3072)) return 2;
    }
  }
  if (!kc && one_round) {
    if (width == 4) {
      const bool spread = p.b_sk % 512 != 0;  // the leading dimension
      bool pays;
      if (m > 16) pays = m <= 32 && !into_int32 && spread && slabs(4) >= 160 && slabs(4) <= 224 && k >= 3072;
      else if (into_int32) pays = k < 1024 || crowded;
      else if (p.out_float) pays = p.b_sk % 2048 != 0 || slabs(4) >= 192 || k <= 3072;
      else pays = crowded ||
                  k <= (spread ? 4096 : (slabs(4) >= 180 || p.b_sk % 2048 ? 2560 : 1024));
      if (pays && n * k <= ((int64_t)64 << 20)) return 4;
    } else if (!adds_in_place) {
      if (width == 2 && m <= 32 && k <= 2048) return 2;
      // (a float output splits k through slots, which cost it more than atomics do an int32 one:
      // (16, 4096, 4096) 13.4 / 8.1 against 14.4 / 10.8)
      if (p.out_float && m <= 16 && slabs(1) >= 192 && k <= 4096) return width;
    }
  }
  if (adds_in_place) return 0;
  // Short k, where the tiles, too few to fill the chip, would have to split it (up to 4096 at
  // m <= 16, 2048 at 32, 1024 at 64; row-major only to 2048: cold it loses beyond), and a float
  // output without a workspace, which tiles cannot split at all.  Measured, us warm/cold:
  // (1, 1024, 2048) 4.9/5.6 -> 3.6/4.5, (16, 2048, 2048) 5.3/6.1 -> 4.5/5.5,
  // (64, 4096, 1024) 6.3/7.2 -> 5.1/5.7; float (16, 2048, 8192) 17.8/29.2 -> 9.7/11.2.
  const bool short_k = k * (m > 16 ? m : 16) <= 65536 && (kc || k <= 2048);
  if ((short_k || (p.out_float && !p.ws)) && tile_count(p, SHAPE_64) < cus / 2 && slabs(1) >= 64) return width;
  return 0;
}

// Tiles with a side of 192 for the kernel with 128-deep blocks, where 256 x 256 ones leave a last round
// mostly idle or are too few and 128 x 128 ones cost more operand traffic: the shape whose rounds of
// workgroups take least by the times below, if that is a tenth under those of the shape chosen so far.
// Microseconds of a round over nkt blocks (of 128 x 128 tiles, two of which share a compute unit, for a
// full round and one with a single tile to a compute unit) and of reading a million words of C where the
// call accumulates (rows of 96 words, those of a side of 192 along n, cost most), fitted to 1200 products
// of 384 to 12000 rows and columns with k = 1024 to 9000 in every order, signedness, mode and output type, which
// the model meets within 10 % at the median.  Over these the rule takes 0.959 of the time without
// such tiles, the best choice each time 0.952; with costs fitted to a few overwriting s8 x s8 products
// it was 0.984, and accumulating ones lost up to 1.7 times.
// Measured, us, before and after: (768, 11008, 4096) 46 -> 36 (192 x 192), 3072^3 37 -> 30,
// (1500, 8192, 2048) to float 32 -> 28 (192 x 256); not (8171, 2730, 1024) accumulating, 68 on 128 x 128
// and 117 on 256 x 192, nor (3968, 3008, 1024) to int8, 20 and 28: below k = 1536 the write-back decides.
// (Whole 256 x 256 tiles, or packed operands padded to them, in two rounds or less stay, a choice that
// tests name: 4608^2 x 4096 95 us, 82 on 192 x 256; (8192, 3072, 4096) 99 and 108.)
static Shape shape_with_192(const Problem &p, Shape chosen) {
  if ((chosen != SHAPE_256 && chosen != SHAPE_128) || p.k < 1536 || p.m < 384 || p.n < 384 ||
      !dma_k128_split_eligible(p, true))
    return chosen;
  // (the forms for whole tiles read the k-sums that packed weights bring, these accumulate them)
  if (p.ksum && dma_k128_eligible(p, chosen == SHAPE_128)) return chosen;
  const int64_t cus = compute_units();
  auto tiles = [&](int64_t bm, int64_t bn) { return ((p.m + bm - 1) / bm) * ((p.n + bn - 1) / bn); };
  const bool whole = (p.m % 256 == 0 && p.n % 256 == 0) || p.rows_padded_to_256;
  if (chosen == SHAPE_256 && whole && tiles(256, 256) <= 2 * cus) return chosen;
  const double nkt = (double)(p.k / 128), old_words = p.accumulate ? 1e-6 * (double)p.m * (double)p.n : 0.0;
  auto time = [&](int64_t bm, int64_t bn, double block, double ends, double read) {
    return (double)((tiles(bm, bn) + cus - 1) / cus) * (block * nkt + ends) + read * old_words;
  };
  const int64_t pairs = tiles(128, 128) / (2 * cus), rest = tiles(128, 128) % (2 * cus);
  const double time128 = (double)(pairs + (rest > cus)) * (0.92 * nkt + 5.0) +
                         (rest > 0 && rest <= cus ? 0.57 * nkt + 4.2 : 0.0) + 0.9 * old_words;
  // (a wider margin where the call accumulates, whose reads the model knows least: (6800, 2912, 1920) with an
  // unsigned operand 68 -> 79 at the same one)
  double best = (p.accumulate ? 0.85 : 0.9) * (chosen == SHAPE_256 ? time(256, 256, 1.21, 12.7, 1.0) : time128);
  auto consider = [&](Shape shape, double cost) {
    if (cost < best) { best = cost; chosen = shape; }
  };
  consider(SHAPE_256X192, time(256, 192, 1.04, 13.7, 1.8));
  consider(SHAPE_192X256, time(192, 256, 1.01, 10.5, 0.95));
  consider(SHAPE_192, time(192, 192, 0.835, 10.3, 1.5));
  return chosen;
}

// What an unsplit product takes on tiles of one form, us: rounds of workgroups, per_cu of them on each compute unit,
// each a time per 128 of k and one for its two ends that grow with how many run side by side; more for an
// unsigned operand whose partner's k sums the kernel has to add up, and for strided operands; and
// what the words of C and the bytes of the operands add.
struct TileForm {
  Kind kind;
  Shape shape;
  int bm, bn, per_cu;
  double block[4], ends[4];           // with 1 .. per_cu workgroups on a compute unit
  double a_unsigned, b_unsigned;      // parts of the time per block,
  double a_strided, b_strided, whole; // the last where no tile reaches over an edge
  double words, old_words, operands;  // per million words written, words added to, bytes read
};

// Fitted to 2400 products of 128 to 13000 rows and columns, k = 512 to 8192, in every order, signedness, mode
// and output type, each timed on every form; the median error is 6 %, nine in ten are within 15 %.
static const TileForm kTileForms[] = {
    {KIND_DMA, SHAPE_64, 64, 64, 4, {0.234, 0.424, 0.728, 0.994}, {3.3, 3.3, 3.27, 1.62},
     0.133, 0.109, 0.149, 0.16, -0.0909, 0.163, 0.548, 0.058},
    {KIND_DMA, SHAPE_128X64, 128, 64, 3, {0.334, 0.698, 1.15}, {3.99, 3.78, 2.96},
     0.152, 0.138, 0.00605, 0.106, -0.0873, 0.191, 0.732, 0.0453},
    {KIND_DMA, SHAPE_64X128, 64, 128, 3, {0.332, 0.678, 1.1}, {3.9, 3.83, 3.28},
     0.202, 0.126, 0.12, 0.0112, -0.11, 0.17, 0.752, 0.0623},
    {KIND_DMA, SHAPE_128, 128, 128, 2, {0.462, 0.996}, {4.34, 5.89},
     0.358, 0.292, 0.0212, 0.00768, -0.0929, 0.258, 0.914, 0.0679},
    {KIND_DMA_K128_SPLIT, SHAPE_128, 128, 128, 2, {0.413, 0.786}, {5.27, 6.24},
     0.197, 0.198, 0.0685, 0.0555, -0.161, -0.039, 0.944, 0.0514},
};

static double predicted_us(const TileForm &f, const Problem &p, int64_t cus) {
  const int64_t tiles = ((p.m + f.bm - 1) / f.bm) * ((p.n + f.bn - 1) / f.bn);
  const int64_t full = tiles / (f.per_cu * cus), rest = (tiles % (f.per_cu * cus) + cus - 1) / cus;
  const bool whole = p.m % f.bm == 0 && p.n % f.bn == 0;
  const double words = 1e-6 * (double)p.m * (double)p.n;
  // What the write-back of the 128-deep kernels takes more: a little per word where rows of C do not start on 16 bytes, and
  // 8.5 us a call that adds to a C whose rows end inside four words, which the waves at that edge fetch one by one (over 600
  // such calls, 172 of them with such rows, 128-deep blocks lost 9 us to the best 64-deep form there and 2 elsewhere;
  // (1372, 1583, 1094) packed 31 us, 20 on 64 x 128 tiles, but (2816, 2752, 4048) to float 62 and 72).  Overwriting it costs nothing.
  const bool unaligned_c = (4 * p.ldc % 16 || reinterpret_cast<uintptr_t>(p.C) % 16) && p.out_float != 2;
  const double extra = f.kind == KIND_DMA ? 0
                                          : (unaligned_c ? words * (p.accumulate ? 0.4 : 0.2) : 0) +
                                                (p.accumulate && p.n % 4 ? 8.5 : 0);
  // (the 64-deep kernels and the form for whole tiles read the sums that packed weights bring)
  const bool sums = !(p.ksum && (f.kind == KIND_DMA || dma_k128_eligible(p, true)));
  const double slower = 1 + (sums && p.a_unsigned ? f.a_unsigned : 0) + (sums && p.b_unsigned ? f.b_unsigned : 0) +
                        (p.a_sk == 1 ? 0 : f.a_strided) + (p.b_sk == 1 ? 0 : f.b_strided) + (whole ? f.whole : 0);
  const double blocks = (double)p.k / 128 * slower;
  return (double)full * (f.block[f.per_cu - 1] * blocks + f.ends[f.per_cu - 1]) +
         (rest ? f.block[rest - 1] * blocks + f.ends[rest - 1] : 0) + words * (p.out_float == 2 ? 0 : f.words) +
         (p.accumulate ? words * f.old_words : 0) +
         extra + 1e-6 * (double)(p.m + p.n) * (double)p.k * f.operands;
}

// The form that takes least by these times, if that is an eighth under those of the plan chosen so far.  The rules of
// choose_plan were each measured at a few products on either side of their lines; between them one tile more than a
// round, or a side a little over a multiple of a tile, costs up to a half.  Over 2500 other products, half
// of them cold, with packed weights and unaligned operands among them, it takes 0.976 of the time without it: 373
// are faster by more than 3 %, up to 1.8 times, 69 slower by more than that.  Over 3400 unaligned ones, packed, half of them
// adding to C, 5 are slower by more than 6 %, one by more than a tenth.
// Measured, us, before and after: (512, 5760, 6400) with an unsigned A 65 -> 36 (180 tiles of 128 x 128 for 360 of
// 128 x 64), (3840, 640, 2176) cold 18.8 -> 12.9, (496, 4432, 3840) 29 -> 19, (3440, 8992, 640) 61 -> 43 (128-deep blocks),
// row-major B (736, 3856, 5120) to int8 40 -> 24.
// From 200 tiles of 64 x 64 on: fewer are a matter of splitting k, as are forms with less than half a round of tiles.
// Between the tiles of 128 x 128 and less: whether sides of 192 or 256 pay is settled before.
static Plan fastest_tiles(const Problem &p, Plan plan) {
  const int64_t cus = compute_units();
  if (p.conv || p.batch > 1 || p.k < 512 || p.m < 128 || p.n < 128 || plan.splits != 1 || tile_count(p, SHAPE_64) < 200)
    return plan;
  const TileForm *now = nullptr;
  for (const TileForm &f : kTileForms)
    if (f.shape == plan.shape && (f.kind == KIND_DMA) == (plan.kind == KIND_DMA)) now = &f;
  if (!now || plan.kind == KIND_STAGED) return plan;
  const double before = predicted_us(*now, p, cus);
  double best = before;
  // What the model, fitted to operands that partly come from the last-level cache, does not see: 64 x 64 tiles depend most
  // on where theirs come from ((1200, 6752, 640) strided, cold, 18.9 us on 128 x 128, 23.7 on these), two groups
  // of waves on them serve k-contiguous ones best ((2160, 688, 6656) cold 25.3 us, 29.9 on 128 x 64), and whole
  // 128 x 128 tiles hold at a short k ((2304, 1536, 512) to int8 7.4 us, 8.5 on 64 x 64).
  if (plan.shape == SHAPE_64 && p.a_sk == 1 && p.b_sk == 1) return plan;
  if (plan.kind == KIND_DMA_K128 && p.k < 1024) return plan;
  for (const TileForm &f : kTileForms) {
    const bool deep = f.kind != KIND_DMA;
    const double margin = f.shape == SHAPE_64 ? 0.8 : 0.88;
    if (2 * ((p.m + f.bm - 1) / f.bm) * ((p.n + f.bn - 1) / f.bn) <= cus) continue;
    if (deep ? !dma_k128_split_eligible(p) : !dma_eligible(p, f.shape)) continue;
    if (const double us = predicted_us(f, p, cus); us < best && us < margin * before) {
      best = us;
      plan = {deep && dma_k128_eligible(p, true) ? KIND_DMA_K128 : f.kind, f.shape, 1};
    }
  }
  return plan;
}

Plan choose_plan(const Problem &p) {
  const int64_t kComputeUnits = compute_units();
  if (p.m == 0 || p.n == 0) return {KIND_NONE, SHAPE_64, 1};
  // (the zero fill writes words; an int8 output of an empty sum goes through the simple kernel)
  if (p.k == 0) return {p.accumulate ? KIND_NONE : (p.out_float == 2 ? KIND_SIMPLE : KIND_FILL), SHAPE_64, 1};
  Plan plan;
  if (!forced_plan(p, &plan)) {
    // The largest tile that still gives most compute units a workgroup; a
    // matrix that is short in one dimension takes a tile that is short there too.
    // A short side (a few tokens, a few output channels) makes the problem a
    // stream over the long operand: wide tiles only when the long side alone
    // fills the chip, else 64 x 64 tiles, which give four times as many workgroups.
    // With at most 16 rows the atomics of split k are cheap, and wide tiles (whole
    // cache lines of a row-major operand) win as soon as k is long enough to cut
    // into one range of 8 blocks or more per compute unit.
    Shape sh;
    const Shape rect = (!p.conv && p.b_sn == 1 && p.a_sk == 1)   ? SHAPE_64X128
                       : (!p.conv && p.a_sm == 1 && p.b_sk == 1) ? SHAPE_128X64
                                                                 : (p.m >= p.n ? SHAPE_128X64 : SHAPE_64X128);
    const int64_t ranges = p.k / 512 > 1 ? p.k / 512 : 1;
    auto enough = [&](Shape wide, int64_t short_side) {
      const int64_t t = tile_count(p, wide);
      return t >= kComputeUnits || (short_side <= 16 && !p.out_float && t * ranges >= kComputeUnits);
    };
    // (With k under 512 a workgroup holds one to eight k blocks; 64 x 64 tiles then need
    // little LDS, many fit a compute unit, and they overtake the wide tiles:
    // (64, 100352, 64) 10.9 -> 9.4 us, (64, 100352, 256) 12.4 -> 11.7 us.)
    // (From 32 rows on, a weight matrix that does not fit the L2 caches streams better through
    // 64 x 128 tiles, whole 128-byte lines of a row-major B, than through 64 x 64 ones; measured
    // cold, us: (32, 11008, 4096) 18.9 -> 16.5, (64, 11008, 4096) 20.7 -> 18.7, (32, 4096, 11008)
    // 18.9 -> 15.3, (64, 4096, 11008) 21.5 -> 18.9; warm within 0.5 us either way; at
    // (64, 4096, 4096) the 64 x 64 tiles stay ahead, 11.6 against 12.7.  A k-contiguous B has no
    // lines to complete: (64, 11008, 4096) 13.3/19.2 us warm/cold on 64 x 64, 16.2/20.8 on 64 x 128.
    // A float output needs enough of them, its ranges of k meeting in slots, cold / warm: (32, 4096, 8192),
    // 32 tiles, 20 / 16.9 us against 17.1 / 11.9 on 64 x 64, (48, 5120, 8192) 21.8 / 17.0 and 21.9 / 14.8; but
    // (32, 6144, 8192), 48 tiles, 21.1 / 16.3 against 24.2 / 16.2.)
    if (p.m <= 64 && p.n > 128)
      sh = p.k >= 512 && enough(SHAPE_64X256, p.m)
               ? SHAPE_64X256
               : (p.m >= 32 && p.k >= 512 && p.b_sn == 1 && p.n * p.k >= ((int64_t)32 << 20) &&
                          (!p.out_float || tile_count(p, SHAPE_64X128) >= 44) && dma_eligible(p, SHAPE_64X128)
                      ? SHAPE_64X128
                      : SHAPE_64);
    else if (p.n <= 64 && p.m > 128) sh = p.k >= 512 && enough(SHAPE_256X64, p.n) ? SHAPE_256X64 : SHAPE_64;
    // A large tile buys operand reuse, which only a long k turns into time: with a short
    // k the problem is a stream that ends in the write of C, and small tiles, several
    // workgroups to a compute unit, overlap that write with the next tile's loads.
    // Between 128 x 128 (too few tiles) and 64 x 64 (64 operations per operand byte,
    // which the L2 caches cannot feed) sit the 8192-element tiles, long side along the
    // longer dimension of C.
    // (One 256 x 256 workgroup fills a compute unit: a few tiles more than there are
    // compute units cost a second round almost in full, which 128 x 128 tiles, two
    // workgroups to a compute unit, do not.  Measured at k = 4096: 289 tiles 121 us
    // against 110, 324 tiles 124 against 125, 400 tiles 132 against 150.)
    else if (p.k >= 1024 && tile_count(p, SHAPE_256) >= 192 &&
             !(tile_count(p, SHAPE_256) > kComputeUnits && tile_count(p, SHAPE_256) <= 320))
      sh = SHAPE_256;
    // (128 x 128 tiles from three quarters of a round on: measured cold against the
    // 8192-element tiles, us: (128, 25088, 1152) 15.2 -> 12.6, (256, 12544, 1152) 14.8 -> 11.2,
    // (768, 4096, 2048) 17.9 -> 13.1, (1024, 3072, 3072) 26.6 -> 23.4, (1024, 3072, 768) 8.2 -> 7.9.)
    else if (p.k >= 512 && !p.conv && tile_count(p, SHAPE_128) >= 192) sh = SHAPE_128;
    // (The long side of an 8192-element tile goes along a row-major B, whose rows it then
    // fetches in whole 128-byte lines, or down a column-major A; with both operands
    // k-contiguous or both strided, along the longer dimension of C.  (3072, 1024, 768)
    // row-major: 128 x 64 8.9 us cold, 64 x 128 8.0; (6272, 256, 2304) 15.4 and 13.0.  They
    // serve from three quarters of a round of tiles on: (256, 6272, 2304) 19.9 us on 64 x 64
    // tiles, 13.3 on 196 tiles of 64 x 128.)
    // (A gathered convolution keeps the order it was measured with: 8192-element tiles from a
    // whole round on, long side along the longer dimension, then 128 x 128 tiles.)
    else if (p.k >= 512 && tile_count(p, rect) >= (p.conv ? kComputeUnits : 192) && dma_eligible(p, rect))
      sh = rect;  // (measured on the direct-to-LDS kernels only)
    else if (p.k >= 512 && tile_count(p, SHAPE_128) >= 192) sh = SHAPE_128;
    else sh = SHAPE_64;
    if (const int nt = slab_width(p)) plan = {KIND_SLAB, SHAPE_64, nt};
    // A very long k over few tiles: the 128 x 128 tiles with 128-deep blocks, k in ranges.
    // The 64 x 64 tiles chosen above for such a shape (enough of them to need no split) run
    // at 64 operations per operand byte; the wider tile halves the bytes, and the ranges give
    // the compute units their workgroups.  Measured warm/cold, us, against the choice above:
    // (768, 768, 8192) 22.8/31.0 -> 18.8/22.6, (512, 1568, 8192) 25.4/34.6 -> 21.5/25.2,
    // (1024, 1024, 16384) 46.5/60.0 -> 32.7/37.4, (768, 2048, 16384) 54.6/73.4 -> 45.3/51.4,
    // (512, 512, 16384) 19.0/23.1 -> 17.7/20.7; accumulating (no zero-fill launch) already from
    // k = 6144: (768, 768, 6144) 18.1/18.5 -> 14.7/17.0, (512, 1568, 6144) 20.1/26.8 -> 16.9/19.8.
    // Not below: at k = 4608 the atomics cost what the ranges save, (1024, 1024, 4608)
    // 13.2/15.4 against 19.8/22.0, (512, 1568, 4608) 14.7/16.7 against 16.7/20.0.
    else if (!p.out_float && p.m > 64 && p.n > 64 && p.k >= (p.accumulate ? 6144 : 8192) &&
             tile_count(p, SHAPE_128) >= 16 &&
             tile_count(p, SHAPE_128) <= 3 * kComputeUnits / 8 && dma_k128_split_eligible(p))
      plan = {KIND_DMA_K128_SPLIT, SHAPE_128, k128_ranges(p)};
    else if (const Shape with_192 = shape_with_192(p, sh); with_192 != sh)
      plan = {KIND_DMA_K128_SPLIT, with_192, 1};
    else if (sh == SHAPE_256 && p.k >= 1024 && dma_k128_eligible(p)) plan = {KIND_DMA_K128, sh, 1};
    // (the same kernel on 128 x 128 tiles, where that is the shape and m, n, k are whole tiles
    // and blocks: 5 to 15 % over the 64-deep kernel of that shape; measured warm/cold, us:
    // 2048^3 14.6/15.1 -> 13.0/14.1, (1024, 3072, 3072) 17.1/23.2 -> 15.6/20.2,
    // (768, 4096, 2048) 12.3/12.9 -> 10.8/12.3, (256, 12544, 1152) 9.1/11.2 -> 8.3/10.4)
    else if (sh == SHAPE_128 && p.k >= 512 && dma_k128_eligible(p, true)) plan = {KIND_DMA_K128, sh, 1};
    // Aligned operands whose m or n is no multiple of the tile: the general forms of the same
    // kernel (loads redirected at the edges instead of padded operands), where the 64-deep
    // kernels with their masked edges used to serve.  On 256 x 256 tiles from k = 2048 on;
    // measured warm, us, overwriting: 4000^2 x 4096 105 -> 60, 4000^2 x 8192 193 -> 112,
    // 8000^2 x 4096 402 -> 254, (6000, 4000, 8192) 325 -> 198, (5008, 3008, 2048) 69 -> 42.
    else if (sh == SHAPE_256 && p.k >= 2048 && dma_k128_split_eligible(p, true))
      plan = {KIND_DMA_K128_SPLIT, SHAPE_256, 1};
    // On 128 x 128 tiles otherwise, from k = 768 on: 4000^2 x 1024 48 -> 30 (with an unsigned
    // operand 88 -> 33), 8000^2 x 1024 162 -> 93, (3000, 2000, 1024) 15.8 -> 14.0,
    // (3000, 2000, 4096) 45 -> 38, (1000, 3072, 768) 8.2 -> 6.7, (1000, 3072, 4096) 23 -> 21;
    // accumulating calls tie warm and gain cold ((3000, 2000, 1024) 19.7/25.7 -> 20.8/21.9).
    // Not at k = 512: (2048, 1568, 512) 6.6 -> 7.7.
    else if ((sh == SHAPE_256 || sh == SHAPE_128) && p.k >= 768 && dma_k128_split_eligible(p))
      plan = {KIND_DMA_K128_SPLIT, SHAPE_128, 1};
    // The same tiles one step below the count that makes 128 x 128 the shape above, on
    // problems with at least 1024 rows and columns and k from 2048: (1520, 1520, 2048)
    // 16.0/17.6 -> 13.3/14.3 us warm/cold, (1520, 1520, 8192) 56.5/56.0 -> 36.9/47.1.
    else if (p.k >= 2048 && p.m >= 1024 && p.n >= 1024 && tile_count(p, SHAPE_128) >= kComputeUnits / 2 &&
             tile_count(p, SHAPE_128) < 192 && dma_k128_split_eligible(p))
      plan = {KIND_DMA_K128_SPLIT, SHAPE_128, 1};
    else if (dma_eligible(p, sh)) plan = {KIND_DMA, sh, 1};
    // the register-staged kernel keeps its operands in flight in VGPRs, which a
    // 256 x 256 tile's accumulators leave no room for: it runs faster on 128 x 128
    // (and faster still on 128 x 64: its loads, 16 bytes at whatever alignment, are what
    // bounds it, and the narrower tile keeps more of them in flight per compute unit;
    // measured on 12 unaligned shapes from 1001 x 4099 x 513 to 4097 x 4099 x 2049: 9-25 % over
    // 128 x 128 on every one)
    // The wide side goes across the operand that is dearer to fetch again, a column-major A:
    // 8191 x 8193 x 8195 with such an A 4570 us on 128 x 64 tiles, 2570 on 64 x 128.
    else plan = {KIND_STAGED, sh == SHAPE_256 || sh == SHAPE_128 ? (p.a_sk == 1 ? SHAPE_128X64 : SHAPE_64X128) : sh, 1};
    // (a pinned number of ranges holds for the 64-deep tiles: nothing else may take their place then)
    if (forced_splits() == 0) plan = fastest_tiles(p, plan);
  }
  const bool pinned = *tuning().variant || forced_splits() > 0;
  if (!pinned && (plan.kind == KIND_STAGED || plan.kind == KIND_DMA) && plan.shape == SHAPE_64)
    plan.wave = wave_form(p, plan.kind == KIND_DMA);
  if ((plan.kind == KIND_STAGED || plan.kind == KIND_DMA) && plan.wave == WAVE_NONE) {
    // float sums are not combined out of order: a float output splits k only through slots of
    // integer partial sums, which need room in a workspace
    const bool may_split = !p.out_float || (p.ws != nullptr && plan.kind == KIND_DMA);
    plan.splits = may_split ? forced_splits() : 1;
    if (plan.splits == 0) {
      // Too few tiles to fill the chip: cut k into ranges of at least 512 (128 for the
      // register-staged kernel) until
      // there is about one workgroup per compute unit.  Every range adds its
      // partial sums into C with atomics (and an overwrite needs C zeroed first),
      // so short problems (few rows of C per byte of operand) may split further
      // than tall ones.
      const int64_t tiles = tile_count(p, plan.shape);
      const int64_t nkt = (p.k + 63) / 64;
      plan.splits = 1;
      // a stream over one long operand (short side of a few rows) is bound by memory
      // latency: it wants two workgroups per compute unit in flight
      const int64_t short_side = p.m < p.n ? p.m : p.n;
      // (of the 64 x 64 tiles, that is: the wide ones fill a compute unit's LDS alone,
      // and one workgroup too many would cost a second round)
      const bool small_tile = plan.shape == SHAPE_64;
      const int64_t target = short_side <= 16 && small_tile ? 2 * kComputeUnits : kComputeUnits;
      // (an accumulating call needs no zero-fill launch and gains from two ranges already
      // at half a round of tiles: (128, 4096, 4096) 11.2 -> 8.8 us, overwriting 11.0 either way)
      // (a float output through slots needs no zeroed C either: it splits as an accumulating call does)
      if (((p.accumulate || p.out_float) ? tiles <= target / 2 : tiles < target / 2) && may_split) {
        const int64_t want = short_side <= 16 && small_tile ? (target + tiles - 1) / tiles : target / tiles;
        // the register-staged kernel has a shallow pipeline with little to amortise:
        // ranges of two k blocks already pay, and it tolerates twice the atomics
        const bool staged = plan.kind == KIND_STAGED;
        const int64_t shortest = staged ? 2 : 8;  // k blocks per range
        const int64_t most = nkt / shortest > 1 ? nkt / shortest : 1;
        const int64_t atomics_ok = (short_side <= 16 ? 64 : (short_side <= 64 ? 8 : 4)) * (staged ? 2 : 1);
        int64_t sp = want < most ? want : most;
        if (sp > atomics_ok) sp = atomics_ok;
        // the zero-fill launch of an overwriting call costs more than the ranges of a short k
        // save: (512, 512, 1024) 5.1 us whole, 6.4 us in two ranges (accumulating 5.0 and 4.5);
        // (512, 512, 2048) 6.7 and 7.3, (256, 256, 2048) 6.5 and 6.0, (512, 512, 4096) 10.6 and 8.7
        if (!p.accumulate && !p.out_float && short_side > 64 && p.k < (tiles <= 32 ? 2048 : 3072)) sp = 1;
        plan.splits = (int)sp;
      }
    }
  }
  return plan;
}

}  // namespace mip
