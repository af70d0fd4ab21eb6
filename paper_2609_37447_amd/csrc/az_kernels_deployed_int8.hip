// int8 instantiations of the deployed-network kernel (az_dep_kernel.h),
// one translation unit per element format so that they compile in parallel.
#include "az_dep_kernel.h"

hipError_t az_launch_deployed_int8(const AzDevNet& n, int boards, const float* planes,
                                  const uint8_t* legal, int B, float* policy, float* value, float* wdl,
                                  hipStream_t s) {
  (void)hipGetLastError();
  if (n.filters != DF || B <= 0) return hipErrorInvalidValue;
  switch (boards) {
    case 0:  // a wave per board
      hipLaunchKernelGGL((az_dep_kernel1<MK_I8>), dim3(B), dim3(64), 0, s, n, planes, legal, policy, value, wdl);
      return hipGetLastError();
    case 1: return launch_dep<MK_I8, 1, 5, 12>(n, planes, legal, B, policy, value, wdl, s);
    case 2: return launch_dep<MK_I8, 2, 5, 8>(n, planes, legal, B, policy, value, wdl, s);
    default: return hipErrorInvalidValue;
  }
}
