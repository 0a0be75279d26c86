// Launchers of the step kernels of one method, main build (512 threads per node).
#include "step_resident_kernels.h"
#include "verify_generic.h"

namespace mdsd {

template <int DT>
static void launch_of(int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    if (nit == 4)
        launch_step_nit<kRRS, DT, 4>(masked, grid, st, P);
    else if (nit == 8)
        launch_step_nit<kRRS, DT, 8>(masked, grid, st, P);
    else if (nit == 16)
        launch_step_nit<kRRS, DT, 16>(masked, grid, st, P);
    else
        hipLaunchKernelGGL((step_streamed_kernel<DT, kRRS>), grid, dim3(kWG), 0, st, P);
}

void launch_step_rrs(int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    (dtype == MDSD_FP32 ? launch_of<0> : launch_of<1>)(nit, masked, grid, st, P);
}

}  // namespace mdsd
