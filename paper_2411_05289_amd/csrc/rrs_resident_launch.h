// Launch code of the RRS / RRSw kernels for rows in registers, one method per translation unit.
#pragma once
#include "rrs_resident_kernels.h"

namespace mdsd {

template <int DT, int NIT, bool WO>
static void launch_rrs_resident_n(bool masked, bool path, dim3 grid, dim3 block, hipStream_t st, const Params& P)
{
    if (path) {
#define MDSD_LAUNCH_PATH(M, S) hipLaunchKernelGGL((rrs_path_resident<DT, NIT, M, WO, S>), grid, block, 0, st, P)
        if (P.stats_in) {
            if (masked) MDSD_LAUNCH_PATH(true, true); else MDSD_LAUNCH_PATH(false, true);
        } else {
            if (masked) MDSD_LAUNCH_PATH(true, false); else MDSD_LAUNCH_PATH(false, false);
        }
#undef MDSD_LAUNCH_PATH
        return;
    }
#define MDSD_LAUNCH_RRS(M, S) hipLaunchKernelGGL((rrs_verify_resident<DT, NIT, M, WO, S>), grid, block, 0, st, P)
    if (P.stats_in) {
        if (masked) MDSD_LAUNCH_RRS(true, true); else MDSD_LAUNCH_RRS(false, true);
    } else {
        if (masked) MDSD_LAUNCH_RRS(true, false); else MDSD_LAUNCH_RRS(false, false);
    }
#undef MDSD_LAUNCH_RRS
}

template <int DT, bool WO>
static void launch_rrs_resident_t(int nit, bool masked, bool path, dim3 grid, dim3 block, hipStream_t st, const Params& P)
{
    if (nit == 4)
        launch_rrs_resident_n<DT, 4, WO>(masked, path, grid, block, st, P);
    else if (nit == 8)
        launch_rrs_resident_n<DT, 8, WO>(masked, path, grid, block, st, P);
    else
        launch_rrs_resident_n<DT, 16, WO>(masked, path, grid, block, st, P);
}

template <bool WO>
static void launch_rrs_resident_m(int dtype, int nit, bool masked, bool path, dim3 grid, dim3 block, hipStream_t st,
                                  const Params& P)
{
    if (dtype == MDSD_FP32)
        launch_rrs_resident_t<0, WO>(nit, masked, path, grid, block, st, P);
    else
        launch_rrs_resident_t<1, WO>(nit, masked, path, grid, block, st, P);
}

}  // namespace mdsd
