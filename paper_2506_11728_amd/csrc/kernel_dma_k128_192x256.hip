// The general form of the kernel with 128-deep k blocks on 192 x 256 tiles.
#include "dma_k128_general.h"

namespace mip {

hipError_t launch_dma_k128_192x256(const Problem &p, hipStream_t s) { return launch_general<192, 256>(p, 1, s); }

}  // namespace mip
