// The draft kernel: the k draft tokens of every internal node (SpecHub: the pair from Q;
// RRS: k independent draws; RRSw: k draws without replacement), and the record of the draft row
// that the verify call can take over.  Instantiated per method in draft_*.hip.
#pragma once
#include "draw_tokens.h"
#include "launch.h"

namespace MDSD_NS {

// ---------------------------------------------------------------- one node's draft
// Entries of a leaf, which drafts nothing, by the node's first thread.
__device__ __forceinline__ void write_leaf_draft(const Params& P, const NodeId& id, int32_t* flags)
{
    if ((int)threadIdx.x != 0) return;
    if (P.hub_out) P.hub_out[id.row] = -1;
    if (flags) flags[id.row] = 0;
    if (P.stats_out) P.stats_out[id.row] = mdsd_row_stats{0.f, 0.f, -1, 0};
}

// What a node's draft leaves with its threads: the record of the draft row in all of them (its rest_mass in sh.bcast_f),
// draft token i in thread i < k.  (sh.node_x still holds the draws that token_of_draws() reads.)
struct NodeDraft {
    float max_stored;
    int hub, token;

    __device__ __forceinline__ mdsd_row_stats record(const Shared& sh) const
    {
        return mdsd_row_stats{uniform(max_stored), uniform(sh.bcast_f), uniform(hub), 0};
    }
};

// The k draft tokens of a node with children, with their record, written to memory and returned.  u: the node's k
// uniforms; flags: where draft flags go, or nullptr.  row_done(row) is called once the row's slab sums are on their way
// to LDS; the registers that hold the row are free behind it.  LEFT: see draw_tokens().
template <int DT, bool LOGITS, int METHOD, int NIT, bool MASKED, bool LEFT = false, class RowDone>
__device__ __forceinline__ NodeDraft draft_node(const Params& P, const NodeId& id, const RowView& rq, const float* u,
                                                int32_t* flags_out, Shared& sh, int& phase, RowDone row_done)
{
    using CV = ToWeight<LOGITS>;
    const int64_t row = id.row;
    const int k = P.k;
    RowSrc<DT, NIT, MASKED ? kEndsPacked : kNoEnds> sq;
    sq.init(rq, CV::fill());
    int32_t* xt = P.tokens_out + (int64_t)id.b * P.N + id.c0;

    CV cq{0.f, 0.f};
    int a_virt = rq.head;
    float mm[1] = {0.f};
    bool swept = false;
    if constexpr (LOGITS && NIT == 0) {
        // a streamed logit row: maximum, weights and slab sums in one sweep
        float Z, mq_lane;
        int mq_chunk = 0;
        cq.s = P.scale_d;
        swept = sweep_streamed_row<DT, true, 2, METHOD == kSpecHub>(sq, cq.s, sh, phase, mm[0], Z, &mq_lane,
                                                METHOD == kSpecHub ? &mq_chunk : nullptr);
        if (swept) {
            cq.ms = mm[0] * cq.s;
            if constexpr (METHOD == kSpecHub) a_virt = block_argmax_at<DT>(rq, mq_lane, mm[0], mq_chunk, sh, phase);
        }
    }
    if constexpr (!LOGITS && NIT == 0) {
        // a streamed row of probabilities: largest element and slab sums in one sweep; a chunk is a dozen instructions of
        // work, so the loads in flight bound it and eight chunks are asked for ahead
        constexpr int E = Elem<DT>::kPerChunk;
        float lane_m = -__builtin_inff();
        int lane_m_chunk = 0;
        sq.template for_each_sums<8>(sh.slab_w, [&](int, int chunk, const float(&a)[E]) {
            if constexpr (METHOD == kSpecHub) {
                float cm = a[0];
#pragma unroll
                for (int e = 1; e < E; ++e) cm = fmaxf(cm, a[e]);
                lane_m_chunk = cm > lane_m ? chunk : lane_m_chunk;
                lane_m = fmaxf(lane_m, cm);
            }
            return chunk_sum<E>(a);
        });
        if constexpr (METHOD == kSpecHub) {
            mm[0] = lane_m;
            block_max<kWaves, 1>(mm, sh.red, phase);
            a_virt = block_argmax_at<DT>(rq, lane_m, mm[0], lane_m_chunk, sh, phase);
        }
        swept = true;
    }
    if (!swept) {
        if (LOGITS || METHOD == kSpecHub) {
            const float mq_lane = lane_max_of_row(sq);
            mm[0] = mq_lane;
            block_max<kWaves, 1>(mm, sh.red, phase);
            if constexpr (METHOD == kSpecHub) a_virt = block_argmax(sq, mq_lane, mm[0], sh, phase);
            if constexpr (LOGITS) {
                cq.s = P.scale_d;
                cq.ms = mm[0] * cq.s;
            }
        }
        pass_weights_to_slabs<CV>(sq, cq, nullptr, 0, sh.slab_w);
    }

    row_done(sq);

    const Drawn d = draw_tokens<METHOD, DT, LEFT>(rq, cq, sh, u, k, a_virt);
    if (d.here) sh.node_x[threadIdx.x & 63] = d.token;
    node_barrier();
    const int hub = METHOD == kSpecHub ? a_virt - rq.head : -1;
    int flags = 0;
    NodeDraft out{mm[0], hub, -1};
    if ((int)threadIdx.x < k) {
        out.token = token_of_draws<METHOD>(sh, k, hub, (int)threadIdx.x, flags);
        xt[threadIdx.x] = out.token;
    }
    if ((int)threadIdx.x == 0) {
        if (P.stats_out) P.stats_out[row] = mdsd_row_stats{mm[0], sh.bcast_f, hub, 0};
        if (P.hub_out) P.hub_out[row] = hub;
        if (flags_out) flags_out[row] = flags;
    }
    return out;
}

// ---------------------------------------------------------------- draft kernel
template <int DT, bool LOGITS, int METHOD, int NIT, bool MASKED = true>
__global__ __launch_bounds__(kWG) void draft_kernel(const Params P)
{
    __shared__ Shared sh;
    int phase = 0;
    // one group of kWG threads per node; a leaf only records that it has no hub
    const NodeId id = node_of_block(P);
    if (id.n == 0 && (int)threadIdx.x == 0) P.tokens_out[(int64_t)id.b * P.N] = -1;
    if (id.c0 < 0) {
        write_leaf_draft(P, id, P.flags);
        return;
    }
    const RowView rq = make_row<DT>(P.draft, P.ld_d, id.row, P.V);
    draft_node<DT, LOGITS, METHOD, NIT, MASKED>(P, id, rq, P.u + id.row * P.k, P.flags, sh, phase, [](const auto&) {});
}

template <int DT, bool LG, int METHOD>
static void launch_draft_n(int nit, bool masked, dim3 grid, dim3 block, hipStream_t st, const Params& P)
{
    // rows that need no masking of their first and last chunk: a variant without the checks,
    // for the two common register sizes
    if (!masked && nit == 4) {
        hipLaunchKernelGGL((draft_kernel<DT, LG, METHOD, 4, false>), grid, block, 0, st, P);
        return;
    }
    if (!masked && nit == 8) {
        hipLaunchKernelGGL((draft_kernel<DT, LG, METHOD, 8, false>), grid, block, 0, st, P);
        return;
    }
    if constexpr (!LG && METHOD != kSpecHub) {  // the others of this size are streamed
        if (nit == 16) {
            hipLaunchKernelGGL((draft_kernel<DT, LG, METHOD, 16>), grid, block, 0, st, P);
            return;
        }
    }
    switch (nit) {
    case 4: hipLaunchKernelGGL((draft_kernel<DT, LG, METHOD, 4>), grid, block, 0, st, P); break;
    case 8: hipLaunchKernelGGL((draft_kernel<DT, LG, METHOD, 8>), grid, block, 0, st, P); break;
    default: hipLaunchKernelGGL((draft_kernel<DT, LG, METHOD, 0>), grid, block, 0, st, P); break;
    }
}

template <int METHOD>
static void launch_draft_method(int dtype, bool logits, int nit, bool masked, dim3 grid, dim3 block, hipStream_t st,
                                const Params& P)
{
    if (dtype == MDSD_FP32) {
        if (logits)
            launch_draft_n<0, true, METHOD>(nit, masked, grid, block, st, P);
        else
            launch_draft_n<0, false, METHOD>(nit, masked, grid, block, st, P);
    } else {
        if (logits)
            launch_draft_n<1, true, METHOD>(nit, masked, grid, block, st, P);
        else
            launch_draft_n<1, false, METHOD>(nit, masked, grid, block, st, P);
    }
}

}  // namespace MDSD_NS
