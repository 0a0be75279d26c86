// Launch code of the verify kernels for short rows, one method per translation unit (group_*.hip).
#pragma once
#include "group_kernels.h"

namespace mdsd {

template <int DT, bool LG, int METHOD, int G>
static void launch_group_path_g(hipStream_t st, const Params& P)
{
    const int groups = kGroupThreads / G;
    hipLaunchKernelGGL((group_path_kernel<DT, LG, METHOD, G>), dim3((unsigned)((P.B + groups - 1) / groups)),
                       dim3(kGroupThreads), 0, st, P);
}

template <int DT, bool LG, int METHOD, int G, bool STEP = false>
static void launch_group_nodes_g(hipStream_t st, const Params& P)
{
    if (P.accept_depth && walks_in_workgroups(G, P.N, P.k, (int64_t)P.B * P.N)) {
        if constexpr (G < 64) {
            if (wave_per_node(G, P.N, P.k, (int64_t)P.B * P.N)) {
                const int trees = 64 / G;
                hipLaunchKernelGGL((group_tree_kernel<DT, LG, METHOD, G, STEP>), dim3((unsigned)((P.B + trees - 1) / trees)),
                                   dim3(64 * P.N), 0, st, P);
                return;
            }
        }
        const int threads = G * P.N <= kGroupThreads ? kGroupThreads : kGroupMaxThreads;
        const int trees = threads / G / P.N;
        hipLaunchKernelGGL((group_verify_kernel<DT, LG, METHOD, G, true, STEP>), dim3((unsigned)((P.B + trees - 1) / trees)),
                           dim3(threads), 0, st, P);
        return;
    }
    const int groups = kGroupThreads / G;
    int64_t nodes = (int64_t)P.B * P.N;
    if (P.first_child && table_by_waves(G, DT == 1, nodes)) {  // whole wavefronts: the last ones may be short of trees
        constexpr int trees = 64 / G;
        nodes = ((int64_t)P.B + trees - 1) / trees * trees * P.N;
    }
    hipLaunchKernelGGL((group_verify_kernel<DT, LG, METHOD, G, false, STEP>), dim3((unsigned)((nodes + groups - 1) / groups)),
                       dim3(kGroupThreads), 0, st, P);
}

// f(integral_constant<int, lanes>)
template <class F>
static void with_lanes(int lanes, F f)
{
    switch (lanes) {
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    default: f(std::integral_constant<int, 64>{}); break;
    }
}

template <int DT, bool LG, int METHOD>
static void launch_group_verify_t(int lanes, bool path, hipStream_t st, const Params& P)
{
    with_lanes(lanes, [&](auto G) {
        if (path)
            launch_group_path_g<DT, LG, METHOD, decltype(G)::value>(st, P);
        else
            launch_group_nodes_g<DT, LG, METHOD, decltype(G)::value>(st, P);
    });
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
