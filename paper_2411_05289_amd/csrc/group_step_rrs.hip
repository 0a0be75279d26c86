// Step kernels of one method for short rows: a group of lanes drafts and verifies a node.
#include "group_verify_launch.h"

namespace mdsd {

void launch_group_step_rrs(int lanes, int dtype, hipStream_t st, const Params& P)
{
    with_lanes(lanes, [&](auto G) {
        if (dtype == MDSD_FP32)
            launch_group_nodes_g<0, true, kRRS, decltype(G)::value, true>(st, P);
        else
            launch_group_nodes_g<1, true, kRRS, decltype(G)::value, true>(st, P);
    });
}

}  // namespace mdsd
