// Helpers shared by the kernels that stream operands global -> LDS directly.
#pragma once
#include <type_traits>

#include "epilogue.h"
#include "lds_layout.h"
#include "mip_internal.h"

namespace mip {

// One wave-wide direct load: lane l's 16 bytes from sbase + voff land in LDS at
// lds_addr + 16 * l.  Written as inline assembly so that the compiler's
// automatic wait-count insertion, which would drain every outstanding load
// before any LDS read, stays out of the pipeline; the kernel places its own
// s_waitcnt vmcnt before the barrier that publishes a stage.  M0 carries the
// LDS base and needs one wait state before the load reads it.  M0 is reserved
// in this compiler: the register allocator never holds a value in it, and naming
// it on the clobber list only draws a "reserved register" warning.  The compiler
// sets M0 itself, right before use, for dynamically indexed register arrays and
// message sends; the kernels that call this keep every register array fully
// unrolled and send no messages, so nothing of the compiler's lives in M0 here.
__device__ __forceinline__ void dma16(uint32_t voff, const uint8_t *sbase, uint32_t lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(voff), "s"(sbase), "s"(lds_addr)
      :);
}

// The same with a full 64-bit address per lane (lanes may point anywhere).
__device__ __forceinline__ void dma16_at(const uint8_t *addr, uint32_t lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, off"
      :
      : "v"(addr), "s"(lds_addr)
      :);
}

// A pointer that is the same in every lane, said so that it stays in SGPRs (the
// direct loads need a scalar base).
__device__ __forceinline__ const uint8_t *wave_uniform(const uint8_t *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
}

// what a filter tap outside the image contributes
static __device__ __attribute__((aligned(16))) const uint8_t outside_image[16] = {};

// "my loads of the next block have landed (N newer loads may still fly), my LDS
// reads are complete; meet the other waves": after this the next stage is
// visible to the whole workgroup and the stage read two steps ago may be refilled.
template <int N>
__device__ __forceinline__ void publish_barrier() {
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const uint8_t *p) {
  return (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const uint8_t *)p);
}

// Kernel arguments fetched here, together: left to the compiler, each is loaded in the block that first
// needs it, and a workgroup waits for three or four such loads (about 500 clocks each) one after the
// other before its first operand load.
template <typename T>
__device__ __forceinline__ void fetch_argument(const T &x) {
  asm volatile("" ::"s"(x));
}
__device__ __forceinline__ void fetch_argument(const TileWalk &w) {
  asm volatile("" ::"s"(w.tiles_m), "s"(w.tiles_n), "s"(w.group.d), "s"(w.group.inv), "s"(w.last.d), "s"(w.last.inv));
}
template <typename... T>
__device__ __forceinline__ void fetch_arguments(const T &...x) {
  (fetch_argument(x), ...);
}

// n / d, d and the range of n known to the host (one multiplication on the scalar unit, where the
// compiler's division takes some forty dependent instructions, a third of a microsecond or more at the start of a
// workgroup, before its first load).
__device__ __forceinline__ unsigned divided(unsigned n, Divisor d) {
  if (__builtin_expect(d.inv != 0, 1)) return __umulhi(n, d.inv);
  return d.d == 1 ? n : n / d.d;
}

// First block of range y of those that k is cut into: `per` blocks each, one more in the first `longer`.
__device__ __forceinline__ int first_of_range(int y, int per, int longer) { return y * per + (y < longer ? y : longer); }

// Workgroup -> tile.  Consecutive workgroup ids land on different XCDs (8 of
// them, each with its own L2), so every XCD gets a contiguous run of tiles, and
// the tiles are walked in groups of 8 tile-rows so that the workgroups resident
// on one XCD share A row-panels and B column-panels.  Returns false for the
// padding workgroups at the end of the grid.
__device__ __forceinline__ bool tile_of_workgroup(const TileWalk &w, int *tm, int *tn) {
  const int ntiles = w.tiles_m * w.tiles_n;
  const int per_xcd = (ntiles + 7) / 8;
  const int lid = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (blockIdx.x / 8 >= per_xcd || lid >= ntiles) return false;
  constexpr int GROUP = 8;
  const int group = (int)divided((unsigned)lid, w.group), at = lid - group * (int)w.group.d;
  const int first_m = group * GROUP;
  const bool whole = w.tiles_m - first_m >= GROUP;
  *tn = whole ? at / GROUP : (int)divided((unsigned)at, w.last);
  *tm = first_m + at - *tn * (whole ? GROUP : (int)w.last.d);
  return true;
}

}  // namespace mip
