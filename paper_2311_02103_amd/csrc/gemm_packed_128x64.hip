// The tiled 4-bit GEMM (gemm_packed_kernel.h): its 128 x 64 tile, 32 x 64 per wavefront.
#include "gemm_packed_kernel.h"

namespace relax {

hipError_t launch_packed_128x64(const GemmArgs &a, int splits, hipStream_t stream) { return packed::launch_packed<2, 4>(a, splits, stream); }

}  // namespace relax
