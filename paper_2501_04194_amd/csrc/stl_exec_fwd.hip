// Generic executor, forward kernels.
#include "stl_exec.h"

namespace stlmi {

hipError_t launch_exec_fwd(bool full, const DevPlan& plan, const Batch& bt, const KArgs& ka, int grid, int nt,
                      size_t lds_bytes, hipStream_t s)
{
    if (!ka.garena && !full) {
        hipLaunchKernelGGL((stl_exec_kernel<false, false, false>), dim3(grid), dim3(nt), lds_bytes, s, plan, bt, ka);     // (ka.nt = nt)
        return hipGetLastError();
    }
    if (!ka.garena) {
        hipLaunchKernelGGL((stl_exec_kernel<false, false, true>), dim3(grid), dim3(nt), lds_bytes, s, plan, bt, ka);     // (ka.nt = nt)
        return hipGetLastError();
    }
    if (!full) {
        hipLaunchKernelGGL((stl_exec_kernel<false, true, false>), dim3(grid), dim3(nt), lds_bytes, s, plan, bt, ka);     // (ka.nt = nt)
        return hipGetLastError();
    }
    hipLaunchKernelGGL((stl_exec_kernel<false, true, true>), dim3(grid), dim3(nt), lds_bytes, s, plan, bt, ka);     // (ka.nt = nt)
    return hipGetLastError();
}

hipError_t set_max_lds_exec_fwd(int bytes)
{
    hipError_t e = hipSuccess;
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)stl_exec_kernel<false, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)stl_exec_kernel<false, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)stl_exec_kernel<false, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)stl_exec_kernel<false, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    return e;
}

}  // namespace stlmi
