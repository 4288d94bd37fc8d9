// The prefill kernel with workgroups of four waves, one per block (see prefill_shape for the calls that take it).
#include "ra_prefill.h"

namespace ra {

hipError_t prefill_four_config()
{
    const hipError_t e = hipFuncSetAttribute((const void *)prefill_kernel<128, false, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, PfRing<128, 4>::kBytes);
    return e != hipSuccess ? e : hipFuncSetAttribute((const void *)prefill_kernel<64, false, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, PfRing<64, 4>::kBytes);
}

hipError_t launch_prefill_four(const PrefillLaunch &a, unsigned workgroups, hipStream_t s)
{
#define RA_PF_LAUNCH(DD)                                                                                                     \
    hipLaunchKernelGGL((prefill_kernel<DD, false, 4>), dim3(workgroups), dim3(64 * 4), (PfRing<DD, 4>::kBytes), s, a.cu, a.num_prompts, a.limit, a.G, \
                       a.Hkv, a.units_shift, a)
    if (a.D == 128) RA_PF_LAUNCH(128);
    else RA_PF_LAUNCH(64);
#undef RA_PF_LAUNCH
    return hipGetLastError();
}

} // namespace ra
