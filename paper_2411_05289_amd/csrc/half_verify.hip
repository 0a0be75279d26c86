// The verify kernels for rows in registers, 256 threads per node (see launch_half.h).
#define MDSD_WG 256
#define MDSD_NS mdsd_half
#define MDSD_MAX_SLABS 64
#include "spechub_resident_kernels.h"
#include "rrs_resident_kernels.h"

#include "launch_half.h"

namespace mdsd_half {

static_assert(kMaxChunks == 16 * kWG && kMaxSlabs * 64 >= kMaxChunks, "sixteen chunks per lane");

void launch_spechub(int dtype, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    const dim3 block(kWG);
    if (dtype == MDSD_FP32) {
        if (masked)
            hipLaunchKernelGGL((spechub_verify_resident<0, 16, true, true>), grid, block, 0, st, P);
        else
            hipLaunchKernelGGL((spechub_verify_resident<0, 16, false, true>), grid, block, 0, st, P);
    } else {
        if (masked)
            hipLaunchKernelGGL((spechub_verify_resident<1, 16, true, true>), grid, block, 0, st, P);
        else
            hipLaunchKernelGGL((spechub_verify_resident<1, 16, false, true>), grid, block, 0, st, P);
    }
}

template <int DT, bool WO>
static void launch_rrs_of(bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    if (masked)
        hipLaunchKernelGGL((rrs_verify_resident<DT, 16, true, WO, true>), grid, dim3(kWG), 0, st, P);
    else
        hipLaunchKernelGGL((rrs_verify_resident<DT, 16, false, WO, true>), grid, dim3(kWG), 0, st, P);
}

void launch_rrs(bool without_replacement, int dtype, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    if (dtype == MDSD_FP32)
        without_replacement ? launch_rrs_of<0, true>(masked, grid, st, P) : launch_rrs_of<0, false>(masked, grid, st, P);
    else
        without_replacement ? launch_rrs_of<1, true>(masked, grid, st, P) : launch_rrs_of<1, false>(masked, grid, st, P);
}

}  // namespace mdsd_half
