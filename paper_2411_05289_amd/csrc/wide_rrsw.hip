// RRSw verify for logit rows in registers, 1024 threads per node (see launch_wide.h).
#define MDSD_WG 1024
#define MDSD_NS mdsd_wide
#define MDSD_MAX_SLABS 512
#include "rrs_resident_kernels.h"

#include "launch_wide.h"

namespace mdsd_wide {

template <int DT, int NIT>
static void launch_nit(dim3 grid, hipStream_t st, const Params& P)
{
    const dim3 block(kWG);
    // rows of up to 4096 chunks come here as unaligned bf16 or, by the head that they do not have, as aligned fp32
    constexpr bool kComesMasked = DT == 1 || NIT > 4;
    if (!P.stats_in)
        hipLaunchKernelGGL((rrs_verify_resident<DT, NIT, true, true, false>), grid, block, 0, st, P);
    else if (kComesMasked && P.masked)
        hipLaunchKernelGGL((rrs_verify_resident<DT, NIT, kComesMasked, true, true>), grid, block, 0, st, P);
    else
        hipLaunchKernelGGL((rrs_verify_resident<DT, NIT, false, true, true>), grid, block, 0, st, P);
}

void launch_rrsw(int dtype, int nit, dim3 grid, hipStream_t st, const Params& P)
{
    if (dtype == MDSD_FP32)
        nit == 4    ? launch_nit<0, 4>(grid, st, P)
        : nit == 8  ? launch_nit<0, 8>(grid, st, P)
        : nit == 16 ? launch_nit<0, 16>(grid, st, P)
                    : launch_nit<0, 20>(grid, st, P);
    else
        nit == 4    ? launch_nit<1, 4>(grid, st, P)
        : nit == 8  ? launch_nit<1, 8>(grid, st, P)
        : nit == 16 ? launch_nit<1, 16>(grid, st, P)
                    : launch_nit<1, 20>(grid, st, P);
}

}  // namespace mdsd_wide
