// Instantiations of the tiles whose waves split k, 64 x 64.
#include "wave_tile.h"

namespace mip {

hipError_t launch_wave_64x64(const Problem &p, bool streamed, hipStream_t s) {
  return streamed ? launch_wave_tile_for<4, 4, 8, STREAMED>(p, s) : hipErrorInvalidValue;
}

}  // namespace mip
