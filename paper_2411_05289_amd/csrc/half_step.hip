// The step kernels once more for 256 threads per node (see half_verify.hip).
#define MDSD_WG 256
#define MDSD_NS mdsd_half
#define MDSD_MAX_SLABS 64
#include "step_resident_kernels.h"

#include "launch_half.h"

namespace mdsd_half {

template <int METHOD, int DT>
static void launch_of(int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    nit == 4   ? launch_step_nit<METHOD, DT, 4>(masked, grid, st, P)
    : nit == 8 ? launch_step_nit<METHOD, DT, 8>(masked, grid, st, P)
               : launch_step_nit<METHOD, DT, 16>(masked, grid, st, P);
}

template <int METHOD>
static void launch_t(int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    (dtype == MDSD_FP32 ? launch_of<METHOD, 0> : launch_of<METHOD, 1>)(nit, masked, grid, st, P);
}

void launch_step(int method, int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    (method == kSpecHub ? launch_t<kSpecHub> : method == kRRS ? launch_t<kRRS> : launch_t<kRRSw>)(dtype, nit, masked, grid,
                                                                                                 st, P);
}

}  // namespace mdsd_half
