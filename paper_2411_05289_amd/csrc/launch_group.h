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
// 2000 nodes: step 16.5 us with 4 lanes per node, 11.9 with 32; 60000 nodes: 20.9 and 53.3); rows of more than 64
// chunks, whose wavefronts wait for memory longer, up to twice as many (1000 elements, 2100 nodes: SpecHub verify
// 7.4 us with 32 lanes, 6.2 with 64).  path: trees follow their nodes one by one, so that the chain is all there is,
// also for rows that leave most lanes without a part (60 elements, 64 lanes against 16: 16 trees 13.0 -> 10.5,
// 1000 14.4 -> 11.7, 4000, where 32 lanes are left, 14.9 -> 15.5).
constexpr int64_t kGroupFewWaves = 2048;
// Whether the workgroups of a launch hold whole trees, which they then walk: a tree's groups must fit a
// workgroup.  Up to kGroupTreesMaxNodes nodes: a wavefront then holds nodes of both kinds and waits for
// its workgroup, which costs more than a launch once the chip is full (15-node trees of 250 bf16 elements,
// 8000 nodes: 10.1 us against 7.7 and the walk's 2.5; 60000 nodes: 39 against 24 and 3); with one tree of 32 lanes
// per node in 512 threads sooner (rows of 500 fp32 elements, 15-node trees: 4500 nodes 9.1 inside, 9.8 outside;
// 9000 nodes 14.3 and 12.0).
constexpr int64_t kGroupTreesMaxNodes = 16384, kGroupTreesMaxNodes32Lanes = 6144;
inline bool group_walks_inside(int lanes, int N, int64_t nodes)
{
    const int64_t threads = (int64_t)lanes * N;
    if (threads > kGroupMaxThreads) return false;
    return nodes <= (lanes >= 32 && threads > kGroupThreads ? kGroupTreesMaxNodes32Lanes : kGroupTreesMaxNodes);
}
// Where the call walks its trees: wavefront n of a workgroup takes node n of 64 / lanes trees, and the one that comes last
// walks them.  A wavefront's nodes are of one kind, nothing is divided to find them, none waits for the others, and a tree's
// rows, which share cache lines where they are short, are read by the same CU (toy workload: 148 -> 111 MB, 29 us with the
// walk's launch -> 26).  Its price is that a workgroup starts only where all its wavefronts find a place.  Against
// workgroups that hold whole trees of mixed wavefronts (group_walks_inside()) it wins with k = 2 at every size (7-node
// trees, 14000 nodes: 400 bf16 elements 12.3 -> 9.6 us, 900 24.2 -> 20.3; 3-node trees, 6000 nodes of 16 fp32 6.2 -> 4.8); k = 4,
// whose nodes with children outlast their leaves, up to 3072 wavefronts (rows of 60 bf16 6000 nodes 13.9 -> 12.2; of 400,
// 3500 wavefronts, 18.6 -> 20.5).  Against nodes in any order and the walk's launch up to 3072 wavefronts too (7-node trees of
// 50 fp32, 40000 nodes 10.0 -> 7.6; 100000 13.8 -> 14.9; of 400 bf16, 20000 nodes 14.7 -> 16.2), and 3-node trees of rows in
// four lanes always (50 fp32, 100000 nodes 14.5 -> 12.3; eight lanes, 200 bf16 25.2 -> 26.4).
constexpr int64_t kWavePerNodeMaxWaves = 3072;
inline bool wave_per_node(int lanes, int N, int k, int64_t nodes)
{
    if (lanes == 64 || N < 2 || N > kGroupMaxThreads / 64) return false;
    if (lanes * nodes <= 64 * kWavePerNodeMaxWaves || (lanes == 4 && N <= 3)) return true;
    return k == 2 && group_walks_inside(lanes, N, nodes);
}
// Trees given by a table whose walk is not in the workgroup.  Rows in four lanes are shorter than two cache lines: node by
// node over the batch, the neighbours that share a line are read far apart (rows of 50 fp32 elements, SpecHub step, 31-node
// trees, 20000 nodes 16.7 us, 150000 40.3; tree by tree 15.6 and 34.9), and tree by tree a wavefront mixes kinds of
// nodes.  So a wavefront takes one node number of its 16 trees and the next one the next number: 15.4 and 34.0 (9-node
// trees, 20000 and 150000 nodes: node by node 15.2 and 35.7, tree by tree 15.3 and 34.9, now 14.6 and 31.8).  bf16 rows, whose chunks
// are twice the work, up to 64 K nodes (60 elements, 9-node trees, 20000 nodes 17.1 -> 16.7, 50000 24.7 -> 23.1, 150000 39.0
// -> 40.2; 100 elements 43.1 -> 45.1).  More lanes: node by node (240 bf16 elements, 50000 nodes 31.8 against 33.2; tree by
// tree 39.1).
constexpr int64_t kTableByWavesMaxNodesBf16 = 65536;
__host__ __device__ constexpr bool table_by_waves(int lanes, bool bf16, int64_t nodes)
{
    return lanes == 4 && (!bf16 || nodes <= kTableByWavesMaxNodesBf16);
}
// Whether the call's workgroups hold whole trees and walk them, by either of the two.
inline bool walks_in_workgroups(int lanes, int N, int k, int64_t nodes)
{
    return wave_per_node(lanes, N, k, nodes) || group_walks_inside(lanes, N, nodes);
}
// walk_nodes: nodes per tree where the launch is to walk the trees, else 1: half the lanes are taken where that
// lets a workgroup hold a tree (rows of 60 bf16 elements, 2000 nodes in trees of 15: 32 lanes 11.9 us, 64 lanes with
// the walk by arrival count 14.9), but not for rows of more than 96 chunks (1000 elements, 1050 nodes: 9.5 us with
// 32 lanes, 8.4 with 64 and the walk's launch; fp32 300, 75 chunks: 7.2 and 7.5) and never a quarter (250 elements,
// 31-node trees: 10.0 with 16 lanes, 8.9 with 64 and the launch).
inline int group_lanes(int64_t chunks, int64_t nodes, int walk_nodes, bool path)
{
    if (chunks > 4 * 64) return 0;
    int least = 4;
    while (4 * least < chunks) least *= 2;
    int g = least;
    const int64_t waves = chunks > 64 ? 2 * kGroupFewWaves : kGroupFewWaves;
    while (g < 64 && (path || g < chunks) && 2 * g * nodes <= 64 * waves) g *= 2;
    if (chunks <= 96 && g > least && !group_walks_inside(g, walk_nodes, nodes) &&
        group_walks_inside(g / 2, walk_nodes, nodes))
        g /= 2;
    return g;
}

// Verify.  The walk is part of the launch (P.accept_depth set) where walks_in_workgroups() says so, or
// with P.tree_count; otherwise it is the caller's.  path: one group per tree, the walk always inside.
void launch_group_spechub(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P);
void launch_group_rrs(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P);
void launch_group_rrsw(int lanes, int dtype, bool logits, bool path, hipStream_t st, const Params& P);

// Logit rows, drafted and verified in one launch; the walk as for the verify calls.
void launch_group_step_spechub(int lanes, int dtype, hipStream_t st, const Params& P);
void launch_group_step_rrs(int lanes, int dtype, hipStream_t st, const Params& P);
void launch_group_step_rrsw(int lanes, int dtype, hipStream_t st, const Params& P);

void launch_group_draft(int method, int lanes, int dtype, bool logits, hipStream_t st, const Params& P);

}  // namespace mdsd
