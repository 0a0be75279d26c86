// The step kernels for rows of up to 512 chunks: two wavefronts per node (see launch_small.h).
#define MDSD_WG 128
#define MDSD_NS mdsd_pair
#define MDSD_MAX_SLABS 8
#include "step_resident_kernels.h"

#include "launch_small.h"

namespace mdsd_pair {

template <int METHOD>
static void launch_of(int dtype, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    (dtype == MDSD_FP32 ? launch_step_nit<METHOD, 0, 4> : launch_step_nit<METHOD, 1, 4>)(masked, grid, st, P);
}

void launch_step(int method, int dtype, bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    static_assert(kMaxChunks == 4 * kWG && kMaxSlabs * 64 >= kMaxChunks, "four chunks per lane");
    (method == kSpecHub ? launch_of<kSpecHub> : method == kRRS ? launch_of<kRRS> : launch_of<kRRSw>)(dtype, masked, grid,
                                                                                                    st, P);
}

}  // namespace mdsd_pair
