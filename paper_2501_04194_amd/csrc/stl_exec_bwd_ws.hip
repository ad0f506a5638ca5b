// Generic executor, backward kernels with slots in the workspace.
#include "stl_exec.h"

namespace stlmi {

hipError_t launch_exec_bwd_ws(bool full, const DevPlan& plan, const Batch& bt, const KArgs& ka, int grid, int nt,
                      size_t lds_bytes, hipStream_t s)
{
    if (!full) {
        hipLaunchKernelGGL((stl_exec_kernel<true, true, false>), dim3(grid), dim3(nt), lds_bytes, s, plan, bt, ka);     // (ka.nt = nt)
        return hipGetLastError();
    }
    hipLaunchKernelGGL((stl_exec_kernel<true, true, true>), dim3(grid), dim3(nt), lds_bytes, s, plan, bt, ka);     // (ka.nt = nt)
    return hipGetLastError();
}

hipError_t set_max_lds_exec_bwd_ws(int bytes)
{
    hipError_t e = hipSuccess;
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)stl_exec_kernel<true, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)stl_exec_kernel<true, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    return e;
}

}  // namespace stlmi
