// The tiled 4-bit GEMM (gemm_packed_kernel.h): its 256 x 192 tile, 64 x 192 per wavefront.
#include "gemm_packed_kernel.h"

namespace relax {

hipError_t launch_packed_256x192(const GemmArgs &a, int splits, hipStream_t stream) { return packed::launch_packed<4, 12>(a, splits, stream); }

}  // namespace relax
