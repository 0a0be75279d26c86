// Launcher of the RRSw kernels for rows in registers, main build (512 threads per node).
#include "rrs_resident_launch.h"

namespace mdsd {

void launch_rrsw_resident(int dtype, int nit, bool masked, bool path, dim3 grid, dim3 block, hipStream_t st, const Params& P)
{
    launch_rrs_resident_m<true>(dtype, nit, masked, path, grid, block, st, P);
}

}  // namespace mdsd
