// Verify kernels for short rows, one method.
#include "group_verify_launch.h"

namespace mdsd {

void launch_group_rrsw(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P)
{
    launch_group_verify<kRRSw>(lanes, dtype, logits, path, st, P);
}

}  // namespace mdsd
