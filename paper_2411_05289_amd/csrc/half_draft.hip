// The draft kernels for logit rows in registers once more, 256 threads per node (see half_verify.hip).
#define MDSD_WG 256
#define MDSD_NS mdsd_half
#define MDSD_MAX_SLABS 64
#include "draft_kernel.h"

#include "launch_half.h"

namespace mdsd_half {

template <int METHOD, int DT, int NIT>
static void launch_nit(bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    if (masked)
        hipLaunchKernelGGL((draft_kernel<DT, true, METHOD, NIT, true>), grid, dim3(kWG), 0, st, P);
    else
        hipLaunchKernelGGL((draft_kernel<DT, true, METHOD, NIT, false>), grid, dim3(kWG), 0, st, P);
}

template <int METHOD, int NIT>
static void launch_of(int dtype, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    (dtype == MDSD_FP32 ? launch_nit<METHOD, 0, NIT> : launch_nit<METHOD, 1, NIT>)(masked, grid, st, P);
}

void launch_draft(int method, int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    if (nit == 16)
        launch_of<kRRSw, 16>(dtype, masked, grid, st, P);
    else
        (method == kSpecHub ? launch_of<kSpecHub, 8> : method == kRRS ? launch_of<kRRS, 8> : launch_of<kRRSw, 8>)(dtype, masked,
                                                                                                                grid, st, P);
}

}  // namespace mdsd_half
