// Joint launches of fp32 GEMMs that bind different kernels.
#include "go_kernel_u.h"
const void* gdy::joint_f32(int family) {
  return family == 1 ? reinterpret_cast<const void*>(&go_gemm_joint<DT_F32>) : nullptr;
}
