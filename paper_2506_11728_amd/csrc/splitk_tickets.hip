// The counters of split k through partial-sum slots (combine_k_ranges in epilogue.h): one
// 32-bit ticket counter per tile, zero whenever no call is using it.  They live in a static
// device array, zero from the moment the code object is loaded, because a caller's workspace
// arrives with unknown contents and zeroing it would cost the very launch this scheme saves.
// Every call takes the next `count` counters of the ring, so calls in flight at the same
// time (other streams, other threads) work on different counters; a range is handed out again
// only after the whole ring has gone round.  A call that is being captured keeps its counters for
// every replay of the graph, at any later time, beside calls that would have drawn the same ones
// since: its counters come from an array of their own and are never handed out again.  Once
// that is used up they lie in the call's workspace, where a kernel of the call zeroes them (1.5 us).
#include <atomic>
#include <mutex>

#include "mip_internal.h"

namespace mip {

namespace {

constexpr int64_t TICKETS = 1 << 20;   // 4 MiB per device
constexpr int64_t CAPTURED = 1 << 20;  // as much again, for some ten thousand captured calls
static __device__ unsigned g_tickets[TICKETS], g_captured[CAPTURED];

constexpr int MAX_DEVICES = 64;
struct PerDevice {
  std::once_flag once;
  unsigned *ring = nullptr, *captured = nullptr;
  hipError_t status = hipErrorNotInitialized;
  std::atomic<uint64_t> cursor{0}, captured_cursor{0};
};
PerDevice g_device[MAX_DEVICES];

}  // namespace

bool being_captured(hipStream_t s) {
  // (the null stream cannot be, and asking about it is an error while another stream is)
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (s == nullptr) return false;
  if (hipStreamIsCapturing(s, &status) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return status != hipStreamCaptureStatusNone;
}

hipError_t splitk_tickets(int64_t count, hipStream_t s, unsigned *own, unsigned **out) {
  if (count < 1 || count > TICKETS / 4) return hipErrorInvalidValue;
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
  PerDevice &d = g_device[device];
  std::call_once(d.once, [&d] {
    void *ring = nullptr, *captured = nullptr;
    d.status = hipGetSymbolAddress(&ring, HIP_SYMBOL(g_tickets));
    if (d.status == hipSuccess) d.status = hipGetSymbolAddress(&captured, HIP_SYMBOL(g_captured));
    d.ring = static_cast<unsigned *>(ring);
    d.captured = static_cast<unsigned *>(captured);
  });
  if (d.status != hipSuccess) return d.status;
  if (being_captured(s)) {
    uint64_t at = d.captured_cursor.load(std::memory_order_relaxed);
    while (at + (uint64_t)count <= (uint64_t)CAPTURED)
      if (d.captured_cursor.compare_exchange_weak(at, at + (uint64_t)count, std::memory_order_relaxed)) {
        *out = d.captured + at;
        return hipSuccess;
      }
    if (!own) return hipErrorOutOfMemory;
    Problem z;
    z.m = 1; z.n = count; z.k = 0; z.C = reinterpret_cast<int32_t *>(own); z.ldc = count;
    *out = own;
    return launch_fill_zero(z, s);
  }
  // the next `count` counters that do not straddle the end of the ring
  uint64_t at = d.cursor.load(std::memory_order_relaxed), first;
  do {
    first = at + (uint64_t)count > (uint64_t)TICKETS ? 0 : at;
  } while (!d.cursor.compare_exchange_weak(at, first + (uint64_t)count, std::memory_order_relaxed));
  *out = d.ring + first;
  return hipSuccess;
}

}  // namespace mip
