// Draft and verification of a node in one go, for logit rows whose target sits in registers: the kernels of the calls
// that are handed both rows of every node at once.
//
// A node's verification needs nothing but its own rows and its own draft, so a batch's draft launch and its verify launch
// have no reason to be two: in one, the target row travels while the node draws its tokens, the leaves' loads fill the
// gaps that the draws of the nodes with children leave, the record and the tokens do not come back from memory, and of
// the draft row that a rejection needs again the first chunks per lane stay in LDS (kept or read again: 64 trees of 32000
// SpecHub 49.0 -> 48.7 us, RRS on 16000 fp32 43.1 -> 41.9).  Without replacement the draft mass outside the drafted tokens
// comes from the slab sums of the draft instead of the first rejected round's pass, whose second form it had been (that
// pass had 13 spilled registers: 61.3 -> 55.4 us).
// Bound like the kernels it joins, by instruction issue and memory in about equal parts.  us a step in two launches ->
// in one, 31-node trees, bf16: SpecHub 32000, 16 trees 25.4 -> 21.2, 64 52.1 -> 46.9, 256 159 -> 151; 12000, 16 17.7 -> 13.1, 64
// 32.2 -> 24.3; RRS 32000, 64 54.5 -> 51.9, RRSw 57.4 -> 55.4, unaligned 32001 74.8 -> 59.0; fp32 32000, one 15-node tree 19.0 ->
// 16.6.
// 128 and 1024 threads: 64 trees of bf16 3000 23.2 -> 17.0, RRSw 26.2 -> 19.0; 8 trees of 128256 SpecHub 49.9 -> 46.6, RRS 61.8 -> 52.8.
// Registers: at four waves per SIMD the bf16 kernels of sixteen chunks on aligned rows spill 15 of them (64 bytes a lane; SpecHub
// with 256 and 1024 threads, RRS with any), those of twenty chunks 13 to 71 (RRS on aligned rows 212 bytes); without them, by an
// exact maximum, the 256-thread kernel was slower (46.9 -> 48.8).
// Both rows asked for at the start (two nodes per CU) was slower (64 trees 55.0), and so were leaves among the nodes with
// children (one to every four of them 51.3, to every one 58.2).
#pragma once
#include "rrs_resident_kernels.h"
#include "spechub_resident_kernels.h"

namespace MDSD_NS {

// Chunks per lane of the draft row while it is drafted from, 0 = streamed: the draft kernels' choice, with whose slab sums,
// records and tokens a step's agree bit for bit (a draw among 100 thousand tokens is within rounding of its neighbour once in
// a thousand).  Not RRS on aligned fp32 rows at 1024 threads, which a draft call holds in registers in small batches only.
template <int METHOD, int DT, int NIT, bool MASKED>
constexpr int kStepDraftNit =
    NIT * kWG <= 4096 || (kWG == 1024 && NIT == 8 && METHOD == kRRS && DT == 0 && !MASKED) ? NIT : 0;

// The draft row's first chunks stay in LDS from the draft on (where they were in registers for it).
template <int METHOD, int DT, int NIT, bool MASKED>
constexpr int kStepKept = kStepDraftNit<METHOD, DT, NIT, MASKED> ? kDraftChunksKept<NIT> : 0;

template <int METHOD, int DT, int NIT, bool MASKED>
__device__ __forceinline__ NodeOut step_node_resident(const Params& P, const NodeId& id, Shared& sh,
                                                      uint4 (*q_kept)[kWG], int& phase)
{
    constexpr int kKept = kStepKept<METHOD, DT, NIT, MASKED>;
    constexpr int NU = METHOD == kSpecHub ? 2 : 0;
    const int k = NU ? NU : P.k;
    const float* ur = P.u + id.row * (k + 1);
    const RowView rp = make_row<DT>(P.target, P.ld_t, id.row, P.V);
    RowSrc<DT, NIT, MASKED> sp;
    NodeOut o{MDSD_NONE, -1, 0, 0.f};
    if (id.n == 0 && (int)threadIdx.x == 0) P.tokens_out[(int64_t)id.b * P.N] = -1;
    if (id.c0 < 0) {
        sp.issue(rp, ExpW::fill());
        write_leaf_draft(P, id, P.draft_flags);
        leaf_resident<DT, NIT, MASKED, METHOD != kSpecHub || !MASKED, false>(P, rp, sp, ur[k], nullptr, sh, phase, o);
    } else {
        const RowView rq = make_row<DT>(P.draft, P.ld_d, id.row, P.V);
        const NodeDraft d = draft_node<DT, true, METHOD, kStepDraftNit<METHOD, DT, NIT, MASKED>, MASKED, METHOD == kRRSw>(
            P, id, rq, P.u_draft + id.row * k, P.draft_flags, sh, phase, [&](const auto& row) {
                if constexpr (kKept > 0) {
                    const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
                    for (int it = 0; it < kKept; ++it) q_kept[it][threadIdx.x] = row.chunk_of(it, lane, wave);
                }
                asm volatile("" ::: "memory");  // not before the draft row's registers are free
                sp.issue(rp, ExpW::fill());
            });
        const mdsd_row_stats record = d.record(sh);
        if constexpr (METHOD == kSpecHub) {
            NodeIn in;
            int flags = 0;
            in.u0 = ur[0];
            in.u1 = ur[1];
            in.u2 = ur[2];
            in.x1 = uniform(token_of_draws<kSpecHub>(sh, 2, record.hub, 0, flags));
            in.x2 = uniform(token_of_draws<kSpecHub>(sh, 2, record.hub, 1, flags));
            in.tokens_ok = in.x1 >= 0 && in.x1 < P.V && in.x2 >= 0 && in.x2 < P.V;
            in.hub = record.hub >= 0 && record.hub < P.V ? record.hub : -1;
            in.q_max = record.max_stored;
            in.q_rest = record.rest_mass;
            fetch_node_lookups<DT, true>(id, P.V, rp, rq, in);
            RowSrc<DT, NIT, MASKED> unused;
            spechub_resident<DT, NIT, MASKED, true, false, kKept>(P, in, rp, rq, sp, unused, false, nullptr, sh, phase, o,
                                                                     q_kept);
        } else {
            rrs_resident<DT, NIT, MASKED, METHOD == kRRSw, true, true, (kKept > 0)>(P, id, rp, rq, sp, false, nullptr, sh,
                                                                                    q_kept, phase, o, d.token, record);
        }
    }
    write_node_outputs(P, id, o.outcome, o.token, o.rmass, o.flags);
    return o;
}

template <int DT, int NIT, bool MASKED>
__global__ __launch_bounds__(kWG, (kVerifyWavesPerSimd<NIT, true>)) void spechub_step_resident(const Params P)
{
    constexpr int kKept = kStepKept<kSpecHub, DT, NIT, MASKED>;
    __shared__ Shared sh;
    __shared__ uint4 q_kept[kKept ? kKept : 1][kWG];
    int phase = 0;
    step_node_resident<kSpecHub, DT, NIT, MASKED>(P, node_of_block(P), sh, q_kept, phase);
}

template <int DT, int NIT, bool MASKED, bool WO>
__global__ __launch_bounds__(kWG, (kWG > 512 || kWG == 256 || NIT > 8 ? 4 : kStatsWavesPerSimd)) void rrs_step_resident(const Params P)
{
    __shared__ Shared sh;
    __shared__ uint4 q_kept[kDraftChunksKept<NIT>][kWG];
    int phase = 0;
    step_node_resident<(WO ? kRRSw : kRRS), DT, NIT, MASKED>(P, node_of_block(P), sh, q_kept, phase);
}

template <int METHOD, int DT, int NIT, bool MASKED>
static void launch_step_one(dim3 grid, hipStream_t st, const Params& P)
{
    if constexpr (METHOD == kSpecHub)
        hipLaunchKernelGGL((spechub_step_resident<DT, NIT, MASKED>), grid, dim3(kWG), 0, st, P);
    else
        hipLaunchKernelGGL((rrs_step_resident<DT, NIT, MASKED, METHOD == kRRSw>), grid, dim3(kWG), 0, st, P);
}

template <int METHOD, int DT, int NIT>
static void launch_step_nit(bool masked, dim3 grid, hipStream_t st, const Params& P)
{
    if (masked)
        launch_step_one<METHOD, DT, NIT, true>(grid, st, P);
    else
        launch_step_one<METHOD, DT, NIT, false>(grid, st, P);
}

}  // namespace MDSD_NS
