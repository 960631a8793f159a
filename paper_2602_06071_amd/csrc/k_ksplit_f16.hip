// The K-split matrix-core kernel of the column layout, half instantiations.
#include "k_ksplit_kernel.h"

namespace fs {

hipError_t launch_ksplit_f16(const mm::Plan& pl, const mm::MfmaArgs& a, dim3 grid, hipStream_t st) {
  return launch_ksplit<f16>(pl, a, grid, st);
}

}  // namespace fs
