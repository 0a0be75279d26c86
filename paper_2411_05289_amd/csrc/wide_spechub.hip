// SpecHub verify for logit rows in registers, 1024 threads per node (see launch_wide.h).
#define MDSD_WG 1024
#define MDSD_NS mdsd_wide
#define MDSD_MAX_SLABS 512
#include "spechub_resident_kernels.h"

#include "launch_wide.h"

namespace mdsd_wide {

template <int DT, int NIT, bool MASKED, bool STATS>
static void launch_one(bool path, dim3 grid, hipStream_t st, const Params& P)
{
    if (path)
        hipLaunchKernelGGL((spechub_path_resident<DT, NIT, MASKED, STATS>), grid, dim3(kWG), 0, st, P);
    else
        hipLaunchKernelGGL((spechub_verify_resident<DT, NIT, MASKED, STATS>), grid, dim3(kWG), 0, st, P);
}

template <int DT, int NIT>
static void launch_nit(bool path, dim3 grid, hipStream_t st, const Params& P)
{
    if (P.stats_in)
        P.masked ? launch_one<DT, NIT, true, true>(path, grid, st, P) : launch_one<DT, NIT, false, true>(path, grid, st, P);
    else if constexpr (NIT <= kMaxNitTwoRows)
        P.masked ? launch_one<DT, NIT, true, false>(path, grid, st, P) : launch_one<DT, NIT, false, false>(path, grid, st, P);
}

void launch_spechub(int dtype, int nit, bool path, dim3 grid, hipStream_t st, const Params& P)
{
    static_assert(kMaxSlabs * 64 >= 16 * kWG, "sixteen chunks per lane");
    if (dtype == MDSD_FP32)
        nit == 4   ? launch_nit<0, 4>(path, grid, st, P)
        : nit == 8 ? launch_nit<0, 8>(path, grid, st, P)
                   : launch_nit<0, 16>(path, grid, st, P);
    else
        nit == 4   ? launch_nit<1, 4>(path, grid, st, P)
        : nit == 8 ? launch_nit<1, 8>(path, grid, st, P)
                   : launch_nit<1, 16>(path, grid, st, P);
}

}  // namespace mdsd_wide
