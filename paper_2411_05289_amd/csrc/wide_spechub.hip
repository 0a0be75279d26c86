// SpecHub verify for logit rows in registers, 1024 threads per node (see launch_wide.h).
#define MDSD_WG 1024
#define MDSD_NS mdsd_wide
#define MDSD_MAX_SLABS 512
#include "spechub_resident_kernels.h"

#include "launch_wide.h"

namespace mdsd_wide {

template <int DT, int NIT, bool MASKED, bool STATS>
static void launch_one(dim3 grid, hipStream_t st, const Params& P)
{
    hipLaunchKernelGGL((spechub_verify_resident<DT, NIT, MASKED, STATS>), grid, dim3(kWG), 0, st, P);
}
template <int DT, int NIT, bool MASKED, bool STATS>
static void launch_path_one(dim3 grid, hipStream_t st, const Params& P)
{
    hipLaunchKernelGGL((spechub_path_resident<DT, NIT, MASKED, STATS>), grid, dim3(kWG), 0, st, P);
}

template <int DT>
static void launch_t(int nit, bool path, dim3 grid, hipStream_t st, const Params& P)
{
    static_assert(kMaxSlabs * 64 >= 16 * kWG, "sixteen chunks per lane");
    if (path) {
        if (nit == 8)
            launch_path_one<DT, 8, true, false>(grid, st, P);
        else
            P.masked ? launch_path_one<DT, 16, true, true>(grid, st, P) : launch_path_one<DT, 16, false, true>(grid, st, P);
    } else if (nit == 16) {
        P.masked ? launch_one<DT, 16, true, true>(grid, st, P) : launch_one<DT, 16, false, true>(grid, st, P);
    } else if (P.stats_in) {
        P.masked ? launch_one<DT, 8, true, true>(grid, st, P) : launch_one<DT, 8, false, true>(grid, st, P);
    } else {
        P.masked ? launch_one<DT, 8, true, false>(grid, st, P) : launch_one<DT, 8, false, false>(grid, st, P);
    }
}

void launch_spechub(int dtype, int nit, bool path, dim3 grid, hipStream_t st, const Params& P)
{
    (dtype == MDSD_FP32 ? launch_t<0> : launch_t<1>)(nit, path, grid, st, P);
}

}  // namespace mdsd_wide
