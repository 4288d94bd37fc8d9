// The prefill kernels with workgroups of four waves, one per block (see prefill_shape for the calls that take them).
#include "ra_prefill.h"

namespace ra {

hipError_t prefill_four_config()
{
    hipError_t e = hipSuccess;
#define RA_PF_CONFIG(DD, V)                                                                                                  \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_kernel<DD, 4, V>, hipFuncAttributeMaxDynamicSharedMemorySize, PfRing<DD, 4>::kBytes);
    RA_PF_CONFIG(128, false) RA_PF_CONFIG(128, true) RA_PF_CONFIG(64, false) RA_PF_CONFIG(64, true)
#undef RA_PF_CONFIG
    return e;
}

hipError_t launch_prefill_four(const PrefillLaunch &a, bool votes, unsigned workgroups, hipStream_t s)
{
#define RA_PF_LAUNCH(DD, V)                                                                                                  \
    hipLaunchKernelGGL((prefill_kernel<DD, 4, V>), dim3(workgroups), dim3(64 * 4), (PfRing<DD, 4>::kBytes), s, a.cu, a.num_prompts, a.limit, a.G, \
                       a.Hkv, a.units_shift, a)
    if (a.D == 128) {
        if (votes) RA_PF_LAUNCH(128, true);
        else RA_PF_LAUNCH(128, false);
    } else {
        if (votes) RA_PF_LAUNCH(64, true);
        else RA_PF_LAUNCH(64, false);
    }
#undef RA_PF_LAUNCH
    return hipGetLastError();
}

} // namespace ra
