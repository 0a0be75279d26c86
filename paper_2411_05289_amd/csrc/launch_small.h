// Launchers of the builds of the generic kernels for rows that are short, but too long for a group of
// lanes (group_kernels.h): a node is handled by 128 or 256 threads instead of 512, four 16-byte chunks of
// the row per lane, so that no wavefront of a node is without a part of the row (pair_*.hip, quad_*.hip).
// Same arguments as the launchers of the main build.  verify: the caller's grid has one workgroup per node
// (path: per tree).  wave_verify.hip: one wavefront per node, SpecHub verify in large batches only.
#pragma once
#include <hip/hip_runtime.h>

#include "params.h"

#define MDSD_DECLARE_SMALL_BUILD(ns, threads)                                                                      \
    namespace ns {                                                                                                 \
    /* the longest row of this build, in 16-byte chunks (head of an unaligned row included) */                     \
    constexpr int kMaxChunks = 4 * (threads);                                                                      \
    void launch_verify(int method, int dtype, bool logits, bool path, dim3 grid, hipStream_t st,                   \
                       const mdsd::Params& P);                                                                     \
    void launch_draft(int method, int dtype, bool logits, hipStream_t st, const mdsd::Params& P);                  \
    }

MDSD_DECLARE_SMALL_BUILD(mdsd_pair, 128)  // two: up to 4088 bf16 / 2044 fp32 elements
MDSD_DECLARE_SMALL_BUILD(mdsd_quad, 256)  // four: up to 8184 / 4092

#undef MDSD_DECLARE_SMALL_BUILD

namespace mdsd_pair {
// logit rows, drafted and verified in one launch (four wavefronts per node: mdsd_half::launch_step)
void launch_step(int method, int dtype, bool masked, dim3 grid, hipStream_t st, const mdsd::Params& P);
}  // namespace mdsd_pair

namespace mdsd_wave {
constexpr int kMaxChunks = 4 * 64;
void launch_spechub(int dtype, bool logits, bool path, dim3 grid, hipStream_t st, const mdsd::Params& P);
}  // namespace mdsd_wave
