// Step kernels of one method for short rows: a group of lanes drafts and verifies a node.
#include "group_verify_launch.h"

namespace mdsd {

void launch_group_step_spechub(int lanes, int dtype, hipStream_t st, const Params& P)
{
    with_lanes(lanes, [&](auto G) {
        if (dtype == MDSD_FP32)
            launch_group_nodes_g<0, true, kSpecHub, decltype(G)::value, true>(st, P);
        else
            launch_group_nodes_g<1, true, kSpecHub, decltype(G)::value, true>(st, P);
    });
}

}  // namespace mdsd
