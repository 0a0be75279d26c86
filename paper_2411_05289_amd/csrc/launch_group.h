// Launchers of the kernels for short rows, a group of lanes per node (group_kernels.h).
#pragma once
#include <hip/hip_runtime.h>

#include "params.h"

namespace mdsd {

constexpr int kGroupThreads = 256;     // threads per workgroup
constexpr int kGroupMaxThreads = 512;  // where a tree's groups need more

// Lanes per node for rows of `chunks` 16-byte chunks, at most four per lane; 0: the rows are too long.
// Few lanes make the most of every instruction, many make a node's chain of instructions short.  Up to
// kGroupFewWaves wavefronts, which the chip holds at once, the short chain wins (bf16 rows of 60 elements,
// 2000 nodes: step 16.5 us with 4 lanes per node, 11.9 with 32; 60000 nodes: 20.9 and 53.3).  nodes: those
// that get a group.  walk_nodes: nodes per tree where the launch is to walk the trees, else 1: the lanes
// are then not more than lets a workgroup hold a tree, if there is such a choice (the same rows, 2000
// nodes in trees of 15: 32 lanes 11.9 us, 64 lanes with the walk by arrival count 14.9).
constexpr int64_t kGroupFewWaves = 2048;
// Whether the workgroups of a launch hold whole trees, which they then walk: a tree's groups must fit a
// workgroup.  Up to kGroupTreesMaxNodes nodes: a wavefront then holds nodes of both kinds and waits for
// its workgroup, which costs more than a launch once the chip is full (15-node trees of 250 bf16 elements,
// 8000 nodes: 10.1 us against 7.7 and the walk's 2.5; 60000 nodes: 39 against 24 and 3).
constexpr int64_t kGroupTreesMaxNodes = 16384;
inline bool group_walks_inside(int lanes, int N, int64_t nodes)
{
    return nodes <= kGroupTreesMaxNodes && (int64_t)lanes * N <= kGroupMaxThreads;
}
inline int group_lanes(int64_t chunks, int64_t nodes, int walk_nodes, bool path)
{
    if (chunks > 4 * 64) return 0;
    int least = 4;
    while (4 * least < chunks) least *= 2;
    int g = least;
    while (g < 64 && (path || g < chunks) && 2 * g * nodes <= 64 * kGroupFewWaves) g *= 2;
    if (!group_walks_inside(g, walk_nodes, nodes) && group_walks_inside(least, walk_nodes, nodes))
        while (!group_walks_inside(g, walk_nodes, nodes)) g /= 2;
    return g;
}

// Verify.  The walk is part of the launch (P.accept_depth set) where group_walks_inside() says so, or
// with P.tree_count; otherwise it is the caller's.  path: one group per tree, the walk always inside.
void launch_group_spechub(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P);
void launch_group_rrs(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P);
void launch_group_rrsw(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P);

void launch_group_draft(int method, int lanes, int dtype, bool logits, hipStream_t st, const Params& P);

}  // namespace mdsd
