// Draft kernels for short rows, every method.
#include "group_kernels.h"

namespace mdsd {

template <int DT, bool LG, int METHOD>
static void launch_group_draft_t(int lanes, hipStream_t st, const Params& P)
{
    const int64_t nodes = (int64_t)P.B * (P.first_child ? P.N : P.n_internal > 0 ? P.n_internal : 1);
    const int groups = kGroupThreads / lanes;
    const dim3 grid((unsigned)((nodes + groups - 1) / groups)), block(kGroupThreads);
    switch (lanes) {
    case 4: hipLaunchKernelGGL((group_draft_kernel<DT, LG, METHOD, 4>), grid, block, 0, st, P); break;
    case 8: hipLaunchKernelGGL((group_draft_kernel<DT, LG, METHOD, 8>), grid, block, 0, st, P); break;
    case 16: hipLaunchKernelGGL((group_draft_kernel<DT, LG, METHOD, 16>), grid, block, 0, st, P); break;
    case 32: hipLaunchKernelGGL((group_draft_kernel<DT, LG, METHOD, 32>), grid, block, 0, st, P); break;
    default: hipLaunchKernelGGL((group_draft_kernel<DT, LG, METHOD, 64>), grid, block, 0, st, P); break;
    }
}

template <int METHOD>
static void launch_group_draft_m(int lanes, int dtype, bool logits, hipStream_t st, const Params& P)
{
    if (dtype == MDSD_FP32) {
        if (logits)
            launch_group_draft_t<0, true, METHOD>(lanes, st, P);
        else
            launch_group_draft_t<0, false, METHOD>(lanes, st, P);
    } else {
        if (logits)
            launch_group_draft_t<1, true, METHOD>(lanes, st, P);
        else
            launch_group_draft_t<1, false, METHOD>(lanes, st, P);
    }
}

void launch_group_draft(int method, int lanes, int dtype, bool logits, hipStream_t st, const Params& P)
{
    if (method == kSpecHub)
        launch_group_draft_m<kSpecHub>(lanes, dtype, logits, st, P);
    else if (method == kRRS)
        launch_group_draft_m<kRRS>(lanes, dtype, logits, st, P);
    else
        launch_group_draft_m<kRRSw>(lanes, dtype, logits, st, P);
}

}  // namespace mdsd
