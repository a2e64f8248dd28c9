// The g-SpMM kernels for rows whose vectors overlap (four fp32 or eight bf16
// columns; spmm.hip hands such calls over).
#include "spmm_kernels.h"

namespace gnnk {

hipError_t launch_spmm_ov(const EngineArgs& a, int dtype, bool maxmin, int opk, int spec, int gc, dim3 grid,
                          dim3 block, hipStream_t s) {
    const int ext = ext_of(a.flags);
    if (maxmin) {
        if (dtype == 0) launch_cmp_ov<float, 4, true>(a, opk, spec, gc, grid, block, s);
        else launch_cmp_ov<bf16_t, 8, true>(a, opk, spec, gc, grid, block, s);
    } else {
        if (dtype == 0) launch_sum_ov<float, 4, true>(a, opk, ext, spec, gc, grid, block, s);
        else launch_sum_ov<bf16_t, 8, true>(a, opk, ext, spec, gc, grid, block, s);
    }
    return hipGetLastError();
}

// (max and min combine with exact vectors)
hipError_t launch_spmm_combine_ov(const EngineArgs& a, int dtype, dim3 grid, dim3 block, hipStream_t s) {
    if (dtype == 0) hipLaunchKernelGGL((spmm_sum_combine_kernel<float, 4, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((spmm_sum_combine_kernel<bf16_t, 8, true>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace gnnk
