// SpecHub verify for rows of up to 256 chunks in large batches: the generic kernel with one wavefront per
// node (launch_small.h).
#define MDSD_WG 64
#define MDSD_NS mdsd_wave
#define MDSD_MAX_SLABS 4
#include "verify_generic.h"

#include "launch_small.h"

namespace mdsd_wave {

static_assert(kMaxChunks == 4 * kWG && kMaxSlabs * 64 >= kMaxChunks, "four chunks per lane");

template <int DT, bool LG>
static void launch_one(bool path, dim3 grid, hipStream_t st, const mdsd::Params& P)
{
    if (path)
        hipLaunchKernelGGL((verify_path_kernel<DT, LG, kSpecHub, 4>), grid, dim3(kWG), 0, st, P);
    else
        hipLaunchKernelGGL((verify_kernel<DT, LG, kSpecHub, 4>), grid, dim3(kWG), 0, st, P);
}

void launch_spechub(int dtype, bool logits, bool path, dim3 grid, hipStream_t st, const mdsd::Params& P)
{
    if (dtype == MDSD_FP32)
        logits ? launch_one<0, true>(path, grid, st, P) : launch_one<0, false>(path, grid, st, P);
    else
        logits ? launch_one<1, true>(path, grid, st, P) : launch_one<1, false>(path, grid, st, P);
}

}  // namespace mdsd_wave
