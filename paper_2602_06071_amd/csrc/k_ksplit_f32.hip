// The K-split matrix-core kernel of the column layout, fp32 instantiations.
#include "k_ksplit_kernel.h"

namespace fs {

hipError_t launch_ksplit_f32(const mm::Plan& pl, const mm::MfmaArgs& a, dim3 grid, hipStream_t st) {
  return launch_ksplit<float>(pl, a, grid, st);
}

}  // namespace fs
