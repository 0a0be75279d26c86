// Draft kernels for logit rows in registers, 1024 threads per node (see launch_wide.h).
#define MDSD_WG 1024
#define MDSD_NS mdsd_wide
#define MDSD_MAX_SLABS 512
#include "draft_kernel.h"

#include "launch_wide.h"

namespace mdsd_wide {

void launch_draft(int method, dim3 grid, hipStream_t st, const Params& P)
{
    const dim3 block(kWG);
    if (method == kRRS)
        hipLaunchKernelGGL((draft_kernel<0, true, kRRS, 8, false>), grid, block, 0, st, P);
    else if (P.masked)
        hipLaunchKernelGGL((draft_kernel<1, true, kSpecHub, 4, true>), grid, block, 0, st, P);
    else
        hipLaunchKernelGGL((draft_kernel<1, true, kSpecHub, 4, false>), grid, block, 0, st, P);
}

}  // namespace mdsd_wide
