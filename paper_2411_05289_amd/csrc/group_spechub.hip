// Verify kernels for short rows, one method.
#include "group_verify_launch.h"

namespace mdsd {

void launch_group_spechub(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P)
{
    launch_group_verify<kSpecHub>(lanes, dtype, logits, path, st, P);
}

}  // namespace mdsd
