// Step kernels of one method, 1024 threads per node (see launch_wide.h).
#define MDSD_WG 1024
#define MDSD_NS mdsd_wide
#define MDSD_MAX_SLABS 512
#include "step_resident_kernels.h"

#include "launch_wide.h"

namespace mdsd_wide {

template <int DT>
static void launch_of(int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    switch (nit) {
    case 4: launch_step_nit<kRRS, DT, 4>(masked, grid, st, P); break;
    case 8: launch_step_nit<kRRS, DT, 8>(masked, grid, st, P); break;
    case 16: launch_step_nit<kRRS, DT, 16>(masked, grid, st, P); break;
    default: launch_step_nit<kRRS, DT, 20>(masked, grid, st, P); break;
    }
}

void launch_step_rrs(int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    (dtype == MDSD_FP32 ? launch_of<0> : launch_of<1>)(nit, masked, grid, st, P);
}

}  // namespace mdsd_wide
