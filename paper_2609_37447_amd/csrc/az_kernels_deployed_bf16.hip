// bf16 instantiations of the deployed-network kernel (az_dep_kernel.h),
// one translation unit per element format so that they compile in parallel.
#include "az_dep_kernel.h"

hipError_t az_launch_deployed_bf16(const AzDevNet& n, int boards, const float* planes,
                                  const uint8_t* legal, int B, float* policy, float* value, float* wdl,
                                  hipStream_t s) {
  switch (boards) {
    case 1: return launch_dep<MK_BF16, 1, 3, 12>(n, planes, legal, B, policy, value, wdl, s);
    case 2: return launch_dep<MK_BF16, 2, 3, 8>(n, planes, legal, B, policy, value, wdl, s);
    default: return hipErrorInvalidValue;
  }
}
