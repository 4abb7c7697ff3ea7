// Joint launches of fp16 GEMMs that bind different kernels.
#include "go_kernel_u.h"
const void* gdy::joint_f16(int family) {
  return family == 1   ? reinterpret_cast<const void*>(&go_gemm_joint<DT_F16>)
         : family == 2 ? reinterpret_cast<const void*>(&go_gemm_p_joint<DT_F16>)
                       : nullptr;
}
