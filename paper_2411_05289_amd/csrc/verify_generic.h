// The generic verify kernel: every method, probabilities or logits, rows in registers or
// streamed, one workgroup per node or (path-only) per tree.  Instantiated per method in
// verify_generic_*.hip.
#pragma once
#include "draft_kernel.h"

namespace MDSD_NS {

// The softmax scales arrive in scalar registers.  The streamed passes of the SpecHub form of this
// kernel measured 4 % slower with the scale as a scalar operand of their multiply-adds than with
// the scale in a vector register (config 4), so it is moved there once; the RRS forms have no
// register to spare for it (one more would cost them a wave per SIMD) and keep the scalar.
__device__ __forceinline__ float in_vgpr(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// ---------------------------------------------------------------- verify kernel
// Ends of rows in registers by element where that measured faster than packed (packed -> by element, 4030 nodes):
// SpecHub on fp32 probabilities, 256 threads per node (3501 elements 14.7 -> 13.8 us; path-only the other way; 512 threads,
// 15-node trees without records: 8000 elements, 240 nodes 7.6 -> 8.0, 4200 elements 480 nodes 7.0 -> 7.3, 2250 14.3 ->
// 13.2), the RRS methods on fp32 rows (2501 probabilities, RRS 17.6 -> 16.3; 2501 logits, RRSw 26.9 -> 25.2;
// path-only 24.3 -> 23.5) and RRS on bf16 probabilities (9001 40.6 -> 39.6), RRSw path-only on bf16 rows (124 nodes, 5001
// probabilities 19.0 -> 17.2).  Packed ends keep the others: RRSw bf16 9001 73.6 -> 49.0.
template <int DT, bool LOGITS, int METHOD, int NIT, bool PATH>
constexpr bool kEndsPerElement =
    kWG > 64 && (PATH                 ? METHOD != kSpecHub && (DT == 0 || METHOD == kRRSw)
                 : METHOD == kSpecHub ? kWG == 256 && DT == 0 && !LOGITS
                 : DT == 0            ? METHOD == kRRSw || !LOGITS
                                      : METHOD == kRRS && !LOGITS && kWG == 512);

// Streamed rows of probabilities are bound by the loads in flight: a chunk is a dozen instructions of work, and SpecHub's
// passes ask for as many chunks ahead as the registers of three nodes per CU take, of one row and of a pair of rows
// (logits, whose chunks are a hundred instructions, gain nothing from more than one or two).  The RRS methods' rounds
// lose by it (two rows four ahead, 480 nodes with records of 32000 fp32 elements 23.4 -> 24.2 us, RRSw 27.3 -> 29.3;
// bf16 20001, 4000 nodes 47.6 -> 54.1; so do their leaves), and so they ask ahead in the sweep for the draft mass only.
constexpr int kProbsAhead = 8, kProbsPairAhead = 4;

// STEP: the node is drafted first, and its record and its tokens do not come back from memory.
template <int DT, bool LOGITS, int METHOD, int NIT, bool PATH, bool STEP = false>
__device__ __forceinline__ NodeOut verify_node(const Params& P, const NodeId& id, Shared& sh, int& phase)
{
    constexpr int E = Elem<DT>::kPerChunk;
    using CV = ToWeight<LOGITS>;
    using Src = RowSrc<DT, NIT, kEndsPerElement<DT, LOGITS, METHOD, NIT, PATH> ? kEndsByElement : kEndsPacked>;
    const int k = P.k;
    const float* ur = P.u + id.row * (k + 1);
    const bool need_full = (P.resid_mass != nullptr) || (P.resid_prob != nullptr);
    float* rprob = P.resid_prob ? P.resid_prob + id.row * (int64_t)P.V : nullptr;

    constexpr bool kProbsStreamed = !LOGITS && NIT == 0;
    const RowView rp = make_row<DT>(P.target, P.ld_t, id.row, P.V);
    Src sp;
    int outcome = MDSD_NONE, token = -1, flags = 0;
    float rmass = 0.f;

    sp.init(rp, CV::fill());

    if constexpr (STEP) {
        if (id.n == 0 && (int)threadIdx.x == 0) P.tokens_out[id.row] = -1;
    }
    if (id.c0 < 0) {
        // ---- leaf: the k = 0 case of Alg. 1, token ~ p
        if constexpr (STEP) write_leaf_draft(P, id, P.draft_flags);
        CV cp{0.f, 0.f};
        bool swept = false;
        if constexpr (LOGITS && NIT == 0) {
            float M, Z;
            cp.s = (METHOD == kSpecHub ? in_vgpr(P.scale_t) : P.scale_t);
            swept = sweep_streamed_row<DT, true>(sp, cp.s, sh, phase, M, Z);
            cp.ms = M * cp.s;
        }
        if (!swept) {
            if constexpr (LOGITS) {
                float mm[1] = {lane_max(sp)};
                block_max<kWaves, 1>(mm, sh.red, phase);
                cp.s = (METHOD == kSpecHub ? in_vgpr(P.scale_t) : P.scale_t);
                cp.ms = mm[0] * cp.s;
            }
            if constexpr (kProbsStreamed && METHOD == kSpecHub)
                sp.template for_each_sums<kProbsAhead>(sh.slab_w, [](int, int, const float(&a)[E]) { return chunk_sum<E>(a); });
            else
                pass_weights_to_slabs<CV>(sp, cp, nullptr, 0, sh.slab_w);
            node_barrier();
        }
        float W = 0.f;
        int v = -1;
        if (PATH || kWaves == 1 || rprob || wave_id() == 0) v = draw_from_row<DT, CV>(rp, cp, nullptr, 0, sh.slab_w, ur[k], W);
        token = v < 0 ? -1 : v - rp.head;
        if (v < 0) flags |= MDSD_FLAG_ZERO_RESIDUAL;
        rmass = LOGITS ? 1.f : W;
        if (rprob)
            write_resid_prob<DT>(rprob, rp, W, [&](int s, float(&w)[E]) {
                chunk_weights<DT, CV>(rp, cp, nullptr, 0, s, w);
            });
    } else {
        const RowView rq = make_row<DT>(P.draft, P.ld_d, id.row, P.V);
        Src sq;
        // the draft row is asked for when a pass first needs it: with the draft call's record of
        // the row at hand, a node that accepts in its first test never reads it
        bool q_asked = false;
        auto need_q = [&]() {
            if (!q_asked) sq.init(rq, CV::fill());
            q_asked = true;
        };
        // one wavefront per node: the rows are a few hundred bytes and every trip to memory is a
        // quarter of the node's life, so the draft row is asked for together with the target row
        if constexpr (kWaves == 1) need_q();
        mdsd_row_stats record{0.f, 0.f, -1, 0};
        if constexpr (STEP) {
            record = draft_node<DT, LOGITS, METHOD, NIT, true, METHOD == kRRSw>(P, id, rq, P.u_draft + id.row * k, P.draft_flags,
                                                                               sh, phase, [](const auto&) {}).record(sh);
        }
        const int32_t* xt = P.tokens + (int64_t)id.b * P.N + id.c0;
        CV cp{0.f, 0.f}, cq{0.f, 0.f};

        if constexpr (METHOD == kSpecHub) {
            // The pair is read ahead of the rows (960 nodes of 9000 bf16 probabilities, read where it is tested: step 16.3 -> 16.5
            // us; 6200 of 6000 bf16 logits 40.9 -> 41.2), but not by single wavefronts (60000 nodes of 736 fp32 logits 84.6 us, read
            // here 85.9; of 832 bf16, 43000 nodes, 57.2 and 57.9).
            constexpr bool kPairLate = kWaves == 1 && !kProbsStreamed;
            int x1 = -1, x2 = -1;
            if constexpr (STEP) {
                int none = 0;
                x1 = uniform(token_of_draws<kSpecHub>(sh, 2, record.hub, 0, none));
                x2 = uniform(token_of_draws<kSpecHub>(sh, 2, record.hub, 1, none));
            } else if constexpr (!kPairLate) {
                x1 = xt[0];
                x2 = xt[1];
            }
            // streamed probabilities: those at the pair are asked for too, at indices brought into the rows
            float p_x1 = 0.f, q_x1 = 0.f, p_x2 = 0.f, q_x2 = 0.f;
            if constexpr (kProbsStreamed) {
                const int c1 = min(max(x1, 0), P.V - 1), c2 = min(max(x2, 0), P.V - 1);
                p_x1 = load_elem<DT>(rp, c1);
                q_x1 = load_elem<DT>(rq, c1);
                p_x2 = load_elem<DT>(rp, c2);
                q_x2 = load_elem<DT>(rq, c2);
            }
            // ---- hub (argmax of the stored draft row), softmax maxima, normalisers: Zp (logits
            // only) and the draft mass outside the hub, Zq' = sum_{y != a} eq.  With the draft
            // call's record of the row at hand, the draft row is not read for any of them.
            const bool have_stats = STEP || P.stats_in != nullptr;
            mdsd_row_stats st{0.f, 0.f, 0, 0};
            if (have_stats) {
                if constexpr (STEP)
                    st = record;
                else
                    st = P.stats_in[id.row];
                if (st.hub < 0 || st.hub >= P.V) st.hub = -1;
            }
            float mm[2], z[2] = {0.f, 0.f};
            int a_virt;
            bool swept = false;
            if (have_stats) {
                mm[0] = 0.f;
                if constexpr (LOGITS && NIT == 0) {
                    // maximum and Zp of the streamed target row in one sweep
                    swept = sweep_streamed_row<DT, false>(sp, in_vgpr(P.scale_t), sh, phase, mm[0], z[0]);
                }
                if (!swept) {
                    float m1[1] = {LOGITS ? lane_max(sp) : 0.f};
                    if constexpr (LOGITS) block_max<kWaves, 1>(m1, sh.red, phase);
                    mm[0] = m1[0];
                }
                mm[1] = st.max_stored;
                a_virt = rq.head + (st.hub < 0 ? 0 : st.hub);
            } else if constexpr (kProbsStreamed) {
                // one sweep over the draft row; the target row is not needed for the first tests
                need_q();
                float mq_lane = -__builtin_inff();
                int mq_chunk = 0;
                sq.template for_each_sums<kProbsAhead>(sh.slab_w, [&](int, int chunk, const float(&a)[E]) {
                    float cm = a[0];
#pragma unroll
                    for (int e = 1; e < E; ++e) cm = fmaxf(cm, a[e]);
                    mq_chunk = cm > mq_lane ? chunk : mq_chunk;
                    mq_lane = fmaxf(mq_lane, cm);
                    return chunk_sum<E>(a);
                });
                float m1[1] = {mq_lane};
                block_max<kWaves, 1>(m1, sh.red, phase);  // barrier: slab sums visible
                mm[0] = 0.f;
                mm[1] = m1[0];
                a_virt = block_argmax_at<DT>(rq, mq_lane, mm[1], mq_chunk, sh, phase);
            } else {
                need_q();
                const float mq_lane = lane_max(sq);
                mm[0] = LOGITS ? lane_max(sp) : 0.f;
                mm[1] = mq_lane;
                block_max<kWaves, 2>(mm, sh.red, phase);
                a_virt = block_argmax(sq, mq_lane, mm[1], sh, phase);
            }
            const int a = a_virt - rq.head;
            if constexpr (LOGITS) {
                cp.s = in_vgpr(P.scale_t);
                cp.ms = mm[0] * cp.s;
                cq.s = in_vgpr(P.scale_d);
                cq.ms = mm[1] * cq.s;
            }
            const int a_slab = a_virt / (64 * E);
            if (have_stats) {
                if (LOGITS && !swept) {
                    float z1[1] = {0.f};
                    sp.for_each([&](int, int, const float(&pa_)[E]) {
                        float wp[E];
#pragma unroll
                        for (int e = 0; e < E; ++e) wp[e] = cp(pa_[e]);
                        z1[0] += chunk_sum<E>(wp);
                    });
                    block_sum<kWaves, 1>(z1, sh.red, phase);
                    z[0] = z1[0];
                }
                z[1] = st.rest_mass;
            } else if constexpr (kProbsStreamed) {
                // the mass outside the hub: its slab's sum formed again without it
                float w[E];
                chunk_weights<DT, CV>(rq, cq, &a_virt, 1, a_slab, w);
                const float without = wave_sum(chunk_sum<E>(w));
                z[1] = slab_total(rq.nslab, [&](int i) { return i == a_slab ? without : sh.slab_w[i]; });
                node_barrier();  // every wave has read the slab sums
            } else {
                for_each2<2>(sp, sq, [&](int s, int chunk, const float(&pa_)[E], const float(&qa_)[E]) {
                    float wp[E], wq[E];
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        wp[e] = cp(pa_[e]);
                        wq[e] = cq(qa_[e]);
                    }
                    if (s == a_slab) zero_excluded<E>(wq, chunk, &a_virt, 1);
                    z[0] += chunk_sum<E>(wp);
                    z[1] += chunk_sum<E>(wq);
                });
                block_sum<kWaves, 2>(z, sh.red, phase);
            }
            const float ea_q = cq(load_elem<DT>(rq, a));
            const float ea_p = cp(load_elem<DT>(rp, a));
            const float Zq_rest = z[1];
            HubScal h;
            h.iZp = LOGITS ? 1.f / z[0] : 1.f;
            h.iZq = LOGITS ? 1.f / (Zq_rest + ea_q) : 1.f;
            h.c = ea_q / Zq_rest;  // q(a) / (1 - q(a)); unused when Zq_rest == 0
            const float pa = ea_p * h.iZp;
            const float qa = ea_q * h.iZq;

            if constexpr (kPairLate && !STEP) {
                x1 = xt[0];
                x2 = xt[1];
            }
            const bool tokens_ok = x1 >= 0 && x1 < P.V && x2 >= 0 && x2 < P.V;
            bool decided = false, degenerate = false;
            int hub_slot = -1;  // slot of the hub token in the pair
            if (have_stats && st.hub < 0) {  // no usable record for this node
                flags |= MDSD_FLAG_BAD_PAIR;
                outcome = MDSD_BAD_PAIR;
                decided = true;
            } else if (!tokens_ok) {
                flags |= MDSD_FLAG_BAD_TOKEN;
                outcome = MDSD_BAD_TOKEN;
                decided = true;
            } else if (!(Zq_rest > 0.f)) {
                degenerate = true;
                flags |= MDSD_FLAG_DEGENERATE_HUB;
                if (x1 != a || x2 != a) {
                    flags |= MDSD_FLAG_BAD_PAIR;
                    outcome = MDSD_BAD_PAIR;
                    decided = true;
                } else if (ur[0] * qa < pa) {
                    outcome = 0;
                    token = a;
                    decided = true;
                }
            } else if (x2 == a && x1 != a) {
                hub_slot = 1;
                const float px = cp(kProbsStreamed ? p_x1 : load_elem<DT>(rp, x1)) * h.iZp;
                const float qx = cq(kProbsStreamed ? q_x1 : load_elem<DT>(rq, x1)) * h.iZq;
                if (ur[0] * qx < px) {  // pair (x, a): min(p(x)/Q(x,a), 1)
                    outcome = 0;
                    token = x1;
                    decided = true;
                }
            } else if (x1 == a && x2 != a) {
                hub_slot = 0;
                const float px = cp(kProbsStreamed ? p_x2 : load_elem<DT>(rp, x2)) * h.iZp;
                const float qx = cq(kProbsStreamed ? q_x2 : load_elem<DT>(rq, x2)) * h.iZq;
                if (ur[0] * (h.c * qx) < fmaxf(px - qx, 0.f)) {  // pair (a, x): min(p'(x)/Q(a,x), 1)
                    outcome = 1;
                    token = x2;
                    decided = true;
                } else if (ur[1] * qa < pa) {
                    // S_ax <= sum_{y != a} Q(a,y) = q(a): the hub's test holds whatever the sum is
                    outcome = 0;
                    token = a;
                    decided = true;
                }
            } else {
                flags |= MDSD_FLAG_BAD_PAIR;
                outcome = MDSD_BAD_PAIR;
                decided = true;
            }

            if (!decided || need_full) {
                if (degenerate) {
                    // residual of the single-draft case: p with the hub removed
                    pass_weights_to_slabs<CV>(sp, cp, &a_virt, 1, sh.slab_w);
                    node_barrier();
                    float W;
                    const int v = draw_from_row<DT, CV>(rp, cp, &a_virt, 1, sh.slab_w, ur[2], W);
                    rmass = W * h.iZp;
                    if (!decided) {
                        token = v < 0 ? -1 : v - rp.head;
                        if (v < 0) flags |= MDSD_FLAG_ZERO_RESIDUAL;
                    }
                    if (rprob)
                        write_resid_prob<DT>(rprob, rp, W, [&](int s, float(&w)[E]) {
                            chunk_weights<DT, CV>(rp, cp, &a_virt, 1, s, w);
                        });
                } else {
                    // ---- residual sums: S_xa = sum Q'(.,a), S_ax = sum Q'(a,.), slab sums of p''
                    float sacc[2] = {0.f, 0.f};
                    need_q();
                    for_each2<(LOGITS ? 2 : kProbsPairAhead)>(sp, sq, [&](int s, int chunk, const float(&pa_)[E], const float(&qa_)[E]) {
                        float ep[E], eq[E], t_xa[E], t_ax[E], w[E];
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            ep[e] = cp(pa_[e]);
                            eq[e] = cq(qa_[e]);
                        }
                        if (s == a_slab) {
                            zero_excluded<E>(ep, chunk, &a_virt, 1);
                            zero_excluded<E>(eq, chunk, &a_virt, 1);
                        }
#pragma unroll
                        for (int e = 0; e < E; ++e) spechub_terms(ep[e], eq[e], h, t_xa[e], t_ax[e], w[e]);
                        sacc[0] += chunk_sum<E>(t_xa);
                        sacc[1] += chunk_sum<E>(t_ax);
                        store_slab_sum(sh.slab_w, s, chunk_sum<E>(w));
                    });
                    block_sum<kWaves, 2>(sacc, sh.red, phase);  // barrier: slab sums visible
                    const float S_xa = sacc[0], S_ax = sacc[1];
                    if (!decided) {
                        if (hub_slot == 1) {  // pair (x, a): hub draws on what pairs (a,.) left
                            const float pa1 = fmaxf(pa - S_ax, 0.f);
                            if (ur[1] * S_xa < pa1) {
                                outcome = 1;
                                token = a;
                                decided = true;
                            }
                        } else {  // pair (a, x)
                            if (ur[1] * S_ax < pa) {
                                outcome = 0;
                                token = a;
                                decided = true;
                            }
                        }
                    }
                    auto sv = [&](int i) { return sh.slab_w[i]; };
                    auto cw = [&](int s, float(&w)[E]) {
                        spechub_chunk_w<DT, CV>(rp, rq, cp, cq, h, a_virt, s, w);
                    };
                    const float W = slab_total(rp.nslab, sv);
                    rmass = W;
                    bool wrote_prob = false;
                    if (!decided) {
                        int v = -1;
                        if (W > 0.f && (PATH || kWaves == 1 || wave_id() == 0)) v = icdf_slabs<E>(rp.nslab, ur[2], W, sv, cw);
                        if (!(W > 0.f)) {
                            // no residual mass: fall back to p itself
                            flags |= MDSD_FLAG_ZERO_RESIDUAL;
                            node_barrier();
                            pass_weights_to_slabs<CV>(sp, cp, nullptr, 0, sh.slab_w);
                            node_barrier();
                            float Wp;
                            v = draw_from_row<DT, CV>(rp, cp, nullptr, 0, sh.slab_w, ur[2], Wp);
                            if (rprob) {
                                write_resid_prob<DT>(rprob, rp, Wp, [&](int s, float(&w)[E]) {
                                    chunk_weights<DT, CV>(rp, cp, nullptr, 0, s, w);
                                });
                                wrote_prob = true;
                            }
                        }
                        if (v < 0) flags |= MDSD_FLAG_ZERO_RESIDUAL;
                        token = v < 0 ? -1 : v - rp.head;
                    }
                    if (rprob && !wrote_prob) write_resid_prob<DT>(rprob, rp, W, cw);
                }
            }
        } else {
            // ---- RRS / RRSw (Alg. 1).  State: residual U = max(p - c q, 0) with mass Wc.
            constexpr bool WO = (METHOD == kRRSw);
            int xs[MDSD_MAX_K];
            bool bad = false;
            for (int i = 0; i < k; ++i) {
                if constexpr (STEP) {
                    const int x = uniform(sh.node_x[i]);  // as token_of_draws() has it
                    xs[i] = x < 0 ? (i > 0 ? xs[i - 1] : 0) : x;
                } else {
                    xs[i] = xt[i];
                }
                if (xs[i] < 0 || xs[i] >= P.V) bad = true;
            }
            if (bad) {
                flags |= MDSD_FLAG_BAD_TOKEN;
                outcome = MDSD_BAD_TOKEN;
            } else {
                // The draft call's record (largest stored element, total mass) stands in for the
                // statistics of the draft row.  Without replacement the mass outside the drafted
                // tokens is needed too, from the second round on: the first rejected round's pass
                // over the draft row sums it.
                const bool have_stats = STEP || P.stats_in != nullptr;
                mdsd_row_stats st = record;
                if (!STEP && have_stats) st = P.stats_in[id.row];
                float z[2] = {0.f, 0.f};
                bool swept = false;
                if constexpr (LOGITS) {
                    float mm[2];
                    if (have_stats) {
                        mm[0] = 0.f;
                        if constexpr (NIT == 0)
                            swept = sweep_streamed_row<DT, false>(sp, P.scale_t, sh, phase, mm[0], z[0]);
                        if (!swept) {
                            float m1[1] = {lane_max(sp)};
                            block_max<kWaves, 1>(m1, sh.red, phase);
                            mm[0] = m1[0];
                        }
                        mm[1] = st.max_stored;
                    } else {
                        need_q();
                        mm[0] = lane_max(sp);
                        mm[1] = lane_max(sq);
                        block_max<kWaves, 2>(mm, sh.red, phase);
                    }
                    cp.s = P.scale_t;
                    cp.ms = mm[0] * cp.s;
                    cq.s = P.scale_d;
                    cq.ms = mm[1] * cq.s;
                }
                // exclusion list (virtual indices) and duplicate marks
                int xv[MDSD_MAX_K];
                bool dup[MDSD_MAX_K];
                for (int i = 0; i < k; ++i) {
                    xv[i] = xs[i] + rp.head;
                    dup[i] = false;
                    for (int j = 0; j < i; ++j) dup[i] = dup[i] || (xs[j] == xs[i]);
                }
                // normalisers; without replacement the draft sum leaves out every draft token,
                // so that the mass remaining after i removals is a sum of positive terms
                if (have_stats) {
                    if (LOGITS && !swept) {
                        float z1[1] = {0.f};
                        sp.for_each([&](int, int, const float(&pa_)[E]) {
                            float wp[E];
#pragma unroll
                            for (int e = 0; e < E; ++e) wp[e] = cp(pa_[e]);
                            z1[0] += chunk_sum<E>(wp);
                        });
                        block_sum<kWaves, 1>(z1, sh.red, phase);
                        z[0] = z1[0];
                    }
                    z[1] = st.rest_mass;
                } else if constexpr (kProbsStreamed) {
                    // the draft row alone (4000 nodes of 32000 fp32 elements: rrs_verify 180 -> 141 us; 480 nodes 33 -> 29)
                    need_q();
                    float z1[1] = {0.f};
                    sq.template for_each<kProbsAhead>([&](int s, int chunk, const float(&qa_)[E]) {
                        float wq[E];
#pragma unroll
                        for (int e = 0; e < E; ++e) wq[e] = qa_[e];
                        if constexpr (WO) {
                            if (slab_has_excluded<E>(s, xv, k)) zero_excluded<E>(wq, chunk, xv, k);
                        }
                        z1[0] += chunk_sum<E>(wq);
                    });
                    block_sum<kWaves, 1>(z1, sh.red, phase);
                    z[1] = z1[0];
                } else {
                    need_q();
                    for_each2(sp, sq, [&](int s, int chunk, const float(&pa_)[E], const float(&qa_)[E]) {
                        float wp[E], wq[E];
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            wp[e] = cp(pa_[e]);
                            wq[e] = cq(qa_[e]);
                        }
                        if constexpr (WO) {
                            if (slab_has_excluded<E>(s, xv, k)) zero_excluded<E>(wq, chunk, xv, k);
                        }
                        z[0] += chunk_sum<E>(wp);
                        z[1] += chunk_sum<E>(wq);
                    });
                    block_sum<kWaves, 2>(z, sh.red, phase);
                }
                float eqx[MDSD_MAX_K];
                for (int i = 0; i < k; ++i) eqx[i] = cq(load_elem<DT>(rq, xs[i]));
                // draft mass (unnormalised) left before round i: what no draft took (a sum of
                // positive terms; with a record, known after the first rejected round) plus the
                // drafts still to come, a repeated token counting once
                const bool rem_pending = WO && !STEP && have_stats;
                float rem_k = rem_pending ? 0.f : z[1];
                if constexpr (WO && STEP) rem_k = uniform(sh.bcast_left);
                auto mass_left = [&](int i) {
                    float m = rem_k;
                    for (int j = k - 1; j >= i; --j) m += (WO && !dup[j]) ? eqx[j] : 0.f;
                    return m;
                };
                const float Zq = have_stats ? z[1] : mass_left(0);
                const float iZp = LOGITS ? 1.f / z[0] : 1.f;
                const float iZq = LOGITS ? 1.f / Zq : 1.f;

                float c = 0.f, Wc = 1.f;
                float slab_c = -1.f;  // c of the slab sums in LDS (-1: none)
                int slab_nx = -1;
                bool decided = false;
                int n_rej = 0;  // tokens xs[0..n_rej) have been rejected
                for (int i = 0; i < k; ++i) {
                    const float px = cp(load_elem<DT>(rp, xs[i])) * iZp;
                    const float qx = eqx[i] * iZq;
                    // draft probability of x_i in this round and the factor rho that rescales q;
                    // without replacement a repeated token has no mass left (Alg. 1, red lines)
                    float Qi = qx, rho = 1.f;
                    if (WO && i > 0) {
                        const float left = mass_left(i);
                        Qi = dup[i] ? 0.f : eqx[i] / left;
                        rho = 1.f / (left * iZq);
                    }
                    bool seen = false;
                    for (int j = 0; j < i; ++j) seen = seen || (xs[j] == xs[i]);
                    const float Ux = seen ? 0.f : fmaxf(fmaf(-c, qx, px), 0.f);
                    if (ur[i] * Qi * Wc < Ux) {  // Alg. 1 returns at the first acceptance
                        outcome = i;
                        token = xs[i];
                        decided = true;
                        break;
                    }
                    // reject: U <- max(p - (c + Wc rho) q, 0)
                    const float c_new = fmaf(Wc, rho, c);
                    n_rej = i + 1;
                    if (i > 0) node_barrier();  // earlier readers of slab_w are done
                    const float c_iZq = c_new * iZq;
                    const bool want_rem = rem_pending && i == 0;
                    float lane_rem[1] = {0.f};
                    need_q();
                    for_each2(sp, sq, [&](int s, int chunk, const float(&pa_)[E], const float(&qa_)[E]) {
                        float w[E], wq[E];
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            wq[e] = cq(qa_[e]);
                            w[e] = rrs_term(cp(pa_[e]), wq[e], iZp, c_iZq);
                        }
                        if (slab_has_excluded<E>(s, xv, n_rej)) zero_excluded<E>(w, chunk, xv, n_rej);
                        store_slab_sum(sh.slab_w, s, chunk_sum<E>(w));
                        if (want_rem) {
                            if (slab_has_excluded<E>(s, xv, k)) zero_excluded<E>(wq, chunk, xv, k);
                            lane_rem[0] += chunk_sum<E>(wq);
                        }
                    });
                    if (want_rem) {
                        block_sum<kWaves, 1>(lane_rem, sh.red, phase);
                        rem_k = lane_rem[0];
                    }
                    node_barrier();
                    const float W_new = slab_total(rp.nslab, [&](int j) { return sh.slab_w[j]; });
                    if (W_new > 0.f) {
                        c = c_new;
                        Wc = W_new;
                        slab_c = c_new;
                        slab_nx = n_rej;
                    } else {
                        flags |= MDSD_FLAG_ZERO_RESIDUAL;
                        slab_c = -1.f;
                    }
                    if constexpr (WO) {
                        if (!(mass_left(i + 1) > 0.f)) {
                            flags |= MDSD_FLAG_Q_EXHAUSTED;
                            break;
                        }
                    }
                }
                if (decided && n_rej == 0 && !rprob) {
                    rmass = 1.f;  // nothing rejected, nothing taken
                } else if (!decided || need_full) {
                    const float c_iZq = c * iZq;
                    auto cw = [&](int s, float(&w)[E]) {
                        rrs_chunk_w<DT, CV>(rp, rq, cp, cq, iZp, c_iZq, xv, n_rej, s, w);
                    };
                    if (slab_c != c || slab_nx != n_rej) {
                        // the slab sums in LDS are not those of the current residual (accepted in
                        // the first round, or a round without mass): rebuild them
                        node_barrier();
                        need_q();
                        for_each2(sp, sq, [&](int s, int chunk, const float(&pa_)[E], const float(&qa_)[E]) {
                            float w[E];
#pragma unroll
                            for (int e = 0; e < E; ++e) w[e] = rrs_term(cp(pa_[e]), cq(qa_[e]), iZp, c_iZq);
                            if (slab_has_excluded<E>(s, xv, n_rej)) zero_excluded<E>(w, chunk, xv, n_rej);
                            store_slab_sum(sh.slab_w, s, chunk_sum<E>(w));
                        });
                        node_barrier();
                    }
                    auto sv = [&](int j) { return sh.slab_w[j]; };
                    const float W = slab_total(rp.nslab, sv);
                    // the mass the rejections took p down to: nothing rejected, nothing taken
                    // (rows of probabilities are used as given and need not sum to 1)
                    rmass = n_rej == 0 ? 1.f : W;
                    if (!decided) {
                        int v = -1;
                        if (PATH || wave_id() == 0) v = icdf_slabs<E>(rp.nslab, ur[k], W, sv, cw);
                        token = v < 0 ? -1 : v - rp.head;
                        if (v < 0) flags |= MDSD_FLAG_ZERO_RESIDUAL;
                    }
                    if (rprob) write_resid_prob<DT>(rprob, rp, W, cw);
                }
            }
        }
    }

    write_node_outputs(P, id, outcome, token, rmass, flags);
    return NodeOut{outcome, token, flags, rmass};
}

template <int DT, bool LOGITS, int METHOD, int NIT>
__global__ __launch_bounds__(kWG) void verify_kernel(const Params P)
{
    __shared__ Shared sh;
    int phase = 0;
    const NodeId id = node_of_block(P);
    verify_node<DT, LOGITS, METHOD, NIT, false>(P, id, sh, phase);
}

// Steps on rows too long for registers, three nodes per CU like the verify kernel (two launches -> one: config 4, SpecHub
// 627 -> 603 us; 32 15-node trees of 128256 65.6 -> 63.2; 128 21-node trees of 152064, k = 4, RRS 313 -> 315, RRSw 335 -> 322).
template <int DT, int METHOD>
__global__ __launch_bounds__(kWG, 6) void step_streamed_kernel(const Params P)
{
    __shared__ Shared sh;
    int phase = 0;
    verify_node<DT, true, METHOD, 0, false, true>(P, node_of_block(P), sh, phase);
}

template <int DT, bool LOGITS, int METHOD, int NIT>
__global__ __launch_bounds__(kWG) void verify_path_kernel(const Params P)
{
    __shared__ Shared sh;
    int phase = 0;
    walk_and_verify(P, [&](const NodeId& id) { return verify_node<DT, LOGITS, METHOD, NIT, true>(P, id, sh, phase); });
}

template <int DT, bool LG, int METHOD>
static void launch_verify_n(int nit, bool path, dim3 grid, dim3 block, hipStream_t st, const Params& P)
{
    if (path) {
        // a tree's nodes follow one another: the row is streamed whatever its size would allow,
        // except for the common 8-chunk case of SpecHub on probabilities
        if constexpr (METHOD == kSpecHub && !LG) {
            if (nit == 8) {
                hipLaunchKernelGGL((verify_path_kernel<DT, LG, METHOD, 8>), grid, block, 0, st, P);
                return;
            }
        }
        hipLaunchKernelGGL((verify_path_kernel<DT, LG, METHOD, 0>), grid, block, 0, st, P);
        return;
    }
    // logit rows that fit in registers have kernels of their own; rows of probabilities in registers: four chunks
    // per lane at most, and only where they are not the better streamed
    if constexpr (!LG) {
        // SpecHub, 512 threads per node: streamed.  An internal node reads its draft row once, in one sweep, and both
        // rows again only where the first tests leave it undecided, and three nodes share a CU instead of the one or two
        // whose rows its registers hold (registers -> streamed, 15-node trees, verify alone without records and with: fp32
        // rows of 32000, 15 nodes 13.3 -> 11.3 us, 8.2 -> 7.9, 480 24.1 -> 19.9, 16.9 -> 13.1, 2250 95 -> 67, 67 -> 52; of 9000, 15
        // 7.1 -> 7.0, 5.0 -> 5.1, 480 10.1 -> 9.7, 7.6 -> 7.2; bf16 rows of 18000, 15 8.3 -> 7.9, 5.7 -> 5.7, 480 11.4 -> 10.5, 8.4 -> 7.9).
        // Rows of four chunks per lane, of which a CU holds two nodes in registers, only in part:
        // fp32, the longer ones where nodes share a CU (8001 elements, 240 nodes 7.6 -> 7.6, 5.3 -> 5.4, 480 9.7 -> 9.3, 7.3 ->
        // 6.9, 2250 21.6 -> 21.2, 16.0 -> 14.8; 6001, 240 6.8 -> 7.1, 5.0 -> 5.2, 480 8.7 -> 8.3, 6.3 -> 6.0, 2250 16.9 -> 17.3,
        // 13.1 -> 12.9; 4200, 480 7.0 -> 7.4, 5.2 -> 5.6, 2250 14.3 -> 15.8, 11.0 -> 12.2);
        // bf16, twice the work per chunk, where a third node per CU saves a round, from 513 to 768 nodes (9000 elements, 480
        // nodes 8.2 -> 8.3, 5.8 -> 6.1, 600 9.7 -> 9.3, 6.7 -> 6.8, 750 10.2 -> 9.5, 7.4 -> 7.1, 900 10.4 -> 10.0, 7.7 -> 8.2, 1200
        // 11.8 -> 13.1, 8.4 -> 9.7), and the longer ones from 257 (14001 elements, 240 nodes 8.2 -> 8.0, 5.7 -> 5.8, 480 10.3 ->
        // 9.6, 7.6 -> 7.0; 12000 7.6 -> 7.8, 5.4 -> 5.7, 9.5 -> 9.2, 6.8 -> 6.7).
        if (nit == 4) {
            bool streams = false;
            if constexpr (METHOD == kSpecHub && kWG == 512) {
                const int64_t nodes = (int64_t)P.B * P.N;
                const bool longer = P.row_chunks > 1400;
                streams = DT == 0 ? longer && nodes > 256 : nodes > (longer ? 256 : 512) && nodes <= 768;
            }
            if (!streams) {
                hipLaunchKernelGGL((verify_kernel<DT, LG, METHOD, 4>), grid, block, 0, st, P);
                return;
            }
        }
    }
    hipLaunchKernelGGL((verify_kernel<DT, LG, METHOD, 0>), grid, block, 0, st, P);
}

template <int METHOD>
static void launch_verify_generic(int dtype, bool logits, int nit, bool path, dim3 grid, dim3 block, hipStream_t st,
                                  const Params& P)
{
    if (dtype == MDSD_FP32) {
        if (logits)
            launch_verify_n<0, true, METHOD>(nit, path, grid, block, st, P);
        else
            launch_verify_n<0, false, METHOD>(nit, path, grid, block, st, P);
    } else {
        if (logits)
            launch_verify_n<1, true, METHOD>(nit, path, grid, block, st, P);
        else
            launch_verify_n<1, false, METHOD>(nit, path, grid, block, st, P);
    }
}

}  // namespace MDSD_NS
