// The streaming few-row matmul on one weight format: a code object of its own so that the formats compile side by side.
#include "fewrow_kernel.h"

namespace relax {
namespace fewrow {
hipError_t launch_f16(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream) { return launch_nb<F_F16>(nb, uw, a, lds_bytes, wait, stream); }
}  // namespace fewrow
}  // namespace relax
