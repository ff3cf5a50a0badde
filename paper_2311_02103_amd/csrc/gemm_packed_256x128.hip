// The tiled 4-bit GEMM (gemm_packed_kernel.h): its 256 x 128 tile, 64 x 128 per wavefront.
#include "gemm_packed_kernel.h"

namespace relax {

hipError_t launch_packed_256x128(const GemmArgs &a, int splits, hipStream_t stream) { return packed::launch_packed<4, 8>(a, splits, stream); }

}  // namespace relax
