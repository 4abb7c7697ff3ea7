// Joint launches of OCP e4m3 GEMMs that bind different kernels.
#include "go_kernel_u.h"
const void* gdy::joint_fp8(int family) {
  return family == 1   ? reinterpret_cast<const void*>(&go_gemm_joint<DT_FP8>)
         : family == 2 ? reinterpret_cast<const void*>(&go_gemm_p_joint<DT_FP8>)
                       : nullptr;
}
