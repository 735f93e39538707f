// Instantiations of the tiles whose waves split k, 32 x 32.
#include "wave_tile.h"

namespace mip {

hipError_t launch_wave_32x32(const Problem &p, bool streamed, hipStream_t s) {
  return streamed ? launch_wave_tile_for<2, 2, 8, STREAMED>(p, s) : launch_wave_tile_for<2, 2, 8, STAGED>(p, s);
}

}  // namespace mip
