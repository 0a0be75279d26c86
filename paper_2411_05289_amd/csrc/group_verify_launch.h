// Launch code of the verify kernels for short rows, one method per translation unit (group_*.hip).
#pragma once
#include "group_kernels.h"

namespace mdsd {

template <int DT, bool LG, int METHOD, int G>
static void launch_group_verify_g(bool path, hipStream_t st, const Params& P)
{
    if (path) {
        const int groups = kGroupThreads / G;
        hipLaunchKernelGGL((group_path_kernel<DT, LG, METHOD, G>), dim3((unsigned)((P.B + groups - 1) / groups)),
                           dim3(kGroupThreads), 0, st, P);
        return;
    }
    if (P.accept_depth && walks_in_workgroups(G, P.N, P.k, (int64_t)P.B * P.N)) {
        if constexpr (G < 64) {
            if (wave_per_node(G, P.N, P.k, (int64_t)P.B * P.N)) {
                const int trees = 64 / G;
                hipLaunchKernelGGL((group_tree_kernel<DT, LG, METHOD, G>), dim3((unsigned)((P.B + trees - 1) / trees)),
                                   dim3(64 * P.N), 0, st, P);
                return;
            }
        }
        const int threads = G * P.N <= kGroupThreads ? kGroupThreads : kGroupMaxThreads;
        const int trees = threads / G / P.N;
        hipLaunchKernelGGL((group_verify_kernel<DT, LG, METHOD, G, true>), dim3((unsigned)((P.B + trees - 1) / trees)),
                           dim3(threads), 0, st, P);
        return;
    }
    const int groups = kGroupThreads / G;
    int64_t nodes = (int64_t)P.B * P.N;
    if (P.first_child && table_by_waves(G, DT == 1, nodes)) {  // whole wavefronts: the last ones may be short of trees
        constexpr int trees = 64 / G;
        nodes = ((int64_t)P.B + trees - 1) / trees * trees * P.N;
    }
    hipLaunchKernelGGL((group_verify_kernel<DT, LG, METHOD, G, false>), dim3((unsigned)((nodes + groups - 1) / groups)),
                       dim3(kGroupThreads), 0, st, P);
}

template <int DT, bool LG, int METHOD>
static void launch_group_verify_t(int lanes, bool path, hipStream_t st, const Params& P)
{
    switch (lanes) {
    case 4: launch_group_verify_g<DT, LG, METHOD, 4>(path, st, P); break;
    case 8: launch_group_verify_g<DT, LG, METHOD, 8>(path, st, P); break;
    case 16: launch_group_verify_g<DT, LG, METHOD, 16>(path, st, P); break;
    case 32: launch_group_verify_g<DT, LG, METHOD, 32>(path, st, P); break;
    default: launch_group_verify_g<DT, LG, METHOD, 64>(path, st, P); break;
    }
}

template <int METHOD>
static void launch_group_verify(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P)
{
    if (dtype == MDSD_FP32) {
        if (logits)
            launch_group_verify_t<0, true, METHOD>(lanes, path, st, P);
        else
            launch_group_verify_t<0, false, METHOD>(lanes, path, st, P);
    } else {
        if (logits)
            launch_group_verify_t<1, true, METHOD>(lanes, path, st, P);
        else
            launch_group_verify_t<1, false, METHOD>(lanes, path, st, P);
    }
}

}  // namespace mdsd
