// Draft kernels for logit rows in registers, 1024 threads per node (see launch_wide.h).
#define MDSD_WG 1024
#define MDSD_NS mdsd_wide
#define MDSD_MAX_SLABS 512
#include "draft_kernel.h"

#include "launch_wide.h"

namespace mdsd_wide {

template <int DT, int METHOD, int NIT>
static void launch_nit(dim3 grid, hipStream_t st, const Params& P)
{
    if (P.masked)
        hipLaunchKernelGGL((draft_kernel<DT, true, METHOD, NIT, true>), grid, dim3(kWG), 0, st, P);
    else
        hipLaunchKernelGGL((draft_kernel<DT, true, METHOD, NIT, false>), grid, dim3(kWG), 0, st, P);
}

template <int METHOD>
static void launch_method(int dtype, int nit, dim3 grid, hipStream_t st, const Params& P)
{
    if (dtype == MDSD_FP32)
        nit == 4 ? launch_nit<0, METHOD, 4>(grid, st, P) : launch_nit<0, METHOD, 8>(grid, st, P);
    else
        launch_nit<1, METHOD, 4>(grid, st, P);
}

void launch_draft(int method, int dtype, int nit, dim3 grid, hipStream_t st, const Params& P)
{
    if (method == kSpecHub)
        launch_method<kSpecHub>(dtype, nit, grid, st, P);
    else if (method == kRRS)
        launch_method<kRRS>(dtype, nit, grid, st, P);
    else
        launch_method<kRRSw>(dtype, nit, grid, st, P);
}

}  // namespace mdsd_wide
