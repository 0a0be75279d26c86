// Launchers of the kernels for logit rows in registers built for 1024 threads per node: batches that leave
// CUs without a node, where a node's own chain of passes is what a call waits for.  Twice the wavefronts
// ask for the row at once and share every pass; and long rows of the RRS methods, of which a CU's registers
// and LDS (nine chunks per lane of the draft row) hold what 512-thread workgroups would stream again in
// every rejected round.  The caller chooses by size (mdsd.hip, where the two sides are measured).
// nit, chunks per lane: RRS methods 4, 8, 16 or 20 (20: some of the row spilled, and still ahead: bf16 rows of
// 152064, k = 4, 672 nodes 145 -> 93 us).  SpecHub verify 8 (without the draft call's records, both rows) or,
// with records, 8 or 16; path-only 8 for masked rows without records, 16 with records.  Draft: SpecHub on bf16 rows
// of up to four chunks per lane, RRS on aligned fp32 rows of up to eight.
#pragma once
#include <hip/hip_runtime.h>

#include "params.h"

namespace mdsd_wide {

constexpr int kThreads = 1024;

void launch_spechub(int dtype, int nit, bool path, dim3 grid, hipStream_t st, const mdsd::Params& P);
void launch_rrs(int dtype, int nit, dim3 grid, hipStream_t st, const mdsd::Params& P);
void launch_rrsw(int dtype, int nit, dim3 grid, hipStream_t st, const mdsd::Params& P);
// drafted and verified in one launch
void launch_step_spechub(int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const mdsd::Params& P);
void launch_step_rrs(int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const mdsd::Params& P);
void launch_step_rrsw(int dtype, int nit, bool masked, dim3 grid, hipStream_t st, const mdsd::Params& P);
void launch_draft(int method, dim3 grid, hipStream_t st, const mdsd::Params& P);

}  // namespace mdsd_wide
