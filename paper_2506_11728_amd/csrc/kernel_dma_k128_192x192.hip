// The general form of the kernel with 128-deep k blocks on 192 x 192 tiles.
#include "dma_k128_general.h"

namespace mip {

hipError_t launch_dma_k128_192x192(const Problem &p, hipStream_t s) { return launch_general<192, 192>(p, 1, s); }

}  // namespace mip
