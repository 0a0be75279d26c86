// RRS and RRS without replacement (Alg. 1) for logit rows that fit in registers.
// Device code and kernels; the launchers are in the translation units that include this file
// (rrs_resident.hip: the main build; half_verify.hip: 256 threads per node).
#pragma once
#include "draft_kernel.h"

namespace MDSD_NS {

// ---------------------------------------------------------------- RRS / RRSw, rows in registers
// Alg. 1 for one internal node, with the draft call's record of the draft row (largest stored element,
// total mass) where there is one: the target row sits in registers, the draft row is streamed once
// per rejected round, and a node whose first draft is accepted never reads it.  The state after
// i rejections is the residual U = max(p - c q, 0) with mass W (c_1 = 0, W_0 = 1,
// c_{i+1} = c_i + W_i rho_{i+1}): round i + 1 accepts x with probability U(x) / (W q_{i+1}(x)).
// WO (without replacement): q_{i+1} is q without the tokens rejected so far, rescaled by
// rho_{i+1} = (mass of q) / (mass left); the mass outside all k drafted tokens is summed (positive
// terms only) in the first pass over the draft row, the masses left are that plus the later drafts'.
// STATS = false: no record; the draft row's largest element and its mass come from one more pass over it,
// while the target row is on its way.
// The first pass over the draft row (without records the one for its mass) leaves its first kDraftChunksKept chunks per lane in LDS, so
// that the passes of later rounds read only the rest of it from memory.
// Bound by instruction issue and the reads of the draft row in about equal parts (see the residual pass).
// Marked tokens as bits and row ends filled in the packed chunks: bf16 rows of 32001 elements, 31-node
// trees, B = 64: rrs_verify 49.7 -> 39.8 us, rrsw_verify 52.0 -> 47.9, B = 128 rrsw_verify 94 -> 71; of 50257
// elements, B = 16: 29.1 -> 25.0 and 32.5 -> 27.5 (those rows were streamed before).  Without records, B = 64
// trees of 15: 45.7 -> 33.8 us.
// (40 KB per node at 512 threads, three nodes per CU; 28 KB at 256 threads, four nodes per CU; 144 KB at
// 1024 threads, one node per CU)
template <int NIT>
constexpr int kDraftChunksKept = kWG == 1024  ? (NIT < 9 ? NIT : 9)
                                 : kWG == 256 ? (NIT < 7 ? NIT : 7)
                                              : (NIT < 5 ? NIT : 5);

// STEP: the node was drafted here a moment ago: draft token i is thread i's `drafted`, `record` its record, and without replacement
// sh.bcast_left the draft mass outside the drafted tokens.  KEPT_AT_ENTRY: q_kept holds the draft row's first chunks.
template <int DT, int NIT, bool MASKED, bool WO, bool STATS, bool STEP = false, bool KEPT_AT_ENTRY = false>
__device__ __forceinline__ void rrs_resident(const Params& P, const NodeId& id, const RowView& rp,
                                             const RowView& rq, const RowSrc<DT, NIT, MASKED>& sp,
                                             bool need_full, float* rprob, Shared& sh,
                                             uint4 (*q_kept)[kWG], int& phase, NodeOut& o,
                                             int drafted = -1, mdsd_row_stats record = {})
{
    static_assert(STATS || !STEP, "a step has its record");
    constexpr int E = Elem<DT>::kPerChunk;
    constexpr int HE = E / 2;
    using Src = RowSrc<DT, NIT, MASKED>;
    const int k = P.k;
    const float* ur = P.u + id.row * (k + 1);
    const int32_t* xt = P.tokens + (int64_t)id.b * P.N + id.c0;
    mdsd_row_stats st;
    if constexpr (STEP)
        st = record;
    else if constexpr (STATS)
        st = P.stats_in[id.row];
    // tokens, the stored logits at them and the uniforms go through LDS (lane i of the first wave
    // fetches draft i), so that no lane holds arrays of them; visible after the first barrier.
    // The tokens and uniforms come over the scalar path (their addresses are the same in every
    // lane), so that waiting for a token does not wait for the row behind it; the look-ups at the
    // tokens are then queued right behind the row, at indices brought into it, and arrive with it.
    int x = -1;
    if constexpr (STEP) x = drafted;
    float u_mine = 0.f;
    for (int i = 0; i < k; ++i) {
        int xi = -1;
        if constexpr (!STEP) xi = xt[i];
        const float ui = ur[i];
        if ((int)threadIdx.x == i) {
            if constexpr (!STEP) x = xi;
            u_mine = ui;
        }
    }
    const float u_k = ur[k];
    {
        const bool ok = x >= 0 && x < P.V;
        const int xc = ok ? x : 0;
        if ((int)threadIdx.x < k) {
            const float lp = load_elem<DT>(rp, xc), lq = load_elem<DT>(rq, xc);
            sh.node_x[threadIdx.x] = ok ? x : -1;
            sh.node_lp[threadIdx.x] = ok ? lp : 0.f;
            sh.node_lq[threadIdx.x] = ok ? lq : 0.f;
            sh.node_u[threadIdx.x] = u_mine;
        }
    }
    if (threadIdx.x == 0) sh.node_u[k] = u_k;

    ExpW cp, cq;
    cp.s = P.scale_t;
    cq.s = P.scale_d;
    float z1[1];
    if constexpr (!STATS) {
        // Both rows' masses against their largest elements: with references that may lie 20 below them (a sweep
        // against the first elements, the cheap estimate of the target's maximum) the residual masses of
        // peaked rows (T = 0.3) were off by 2.0e-7 instead of 0.8e-7.  The draft row is read once, while the
        // target row is on its way: every lane sums against the largest element it has met and rescales its
        // sum when that grows (two passes took 2 us more of 30, V = 32000, 960 nodes).  A huge negative
        // number is no reference (see wave_shifted_norm()).
        RowSrc<DT, 0> row;
        row.init(rq, ExpW::fill());
        const float ninf = -__builtin_inff();
        float mm[2] = {ninf, ninf}, z[2] = {0.f, 0.f}, lane_ms = ninf;
        const int lane = threadIdx.x & 63, wave = wave_id();
        uint4 c0 = fetch_chunk(rq, wave * 64 + lane), c1 = fetch_chunk(rq, (wave + kWaves) * 64 + lane);
        for (int it = 0, s = wave; s < rq.nslab; ++it, s += kWaves) {
            const uint4 next = fetch_chunk(rq, (s + 2 * kWaves) * 64 + lane);
            row.end_of_row(c0, s, lane);
            if (it < kDraftChunksKept<NIT>) q_kept[it][threadIdx.x] = c0;
            float a[E];
            unpack<DT>(c0, a);
#pragma unroll
            for (int e = 0; e < E; ++e) mm[1] = fmaxf(mm[1], a[e]);
            const float ms = mm[1] * cq.s;
            const bool refers = fabsf(ms) < 0x1p31f;
            ExpW cw;
            cw.s = cq.s;
            cw.ms = refers ? ms : 0.f;
            float w[E];
#pragma unroll
            for (int e = 0; e < E; ++e) w[e] = cw(a[e]);
            z[1] = fmaf(z[1], __builtin_amdgcn_exp2f(lane_ms - cw.ms), chunk_sum<E>(w));
            lane_ms = refers ? ms : ninf;
            c0 = c1;
            c1 = next;
        }
        mm[0] = lane_max(sp);
        block_max<kWaves, 2>(mm, sh.red, phase);
        cp.ms = uniform(mm[0] * cp.s);
        cq.ms = uniform(mm[1] * cq.s);
        z[1] *= __builtin_amdgcn_exp2f(lane_ms - cq.ms);
        sp.for_each([&](int, int, const float(&a)[E]) {
            float w[E];
#pragma unroll
            for (int e = 0; e < E; ++e) w[e] = cp(a[e]);
            z[0] += chunk_sum<E>(w);
        });
        block_sum<kWaves, 2>(z, sh.red, phase);
        z1[0] = z[0];
        st.rest_mass = z[1];
    } else {
        // ---- target row: shift (cheap estimate first, where there is one) and Zp
        cq.ms = uniform(st.max_stored * cq.s);
        auto normaliser = [&](float lane_m) {
            const RowNorm n = wave_shifted_norm<false>(sp, cp.s, lane_m, sh, phase);
            cp.ms = uniform(n.ms);
            z1[0] = n.Z;
        };
        if constexpr (Src::kHasShiftEstimate) {
            normaliser(sp.lane_shift_estimate());
            if (__builtin_expect(!(z1[0] > 0.f && z1[0] < __builtin_inff()), 0)) normaliser(lane_max(sp));
        } else {
            normaliser(lane_max(sp));
        }
    }
    const float iZp = uniform(1.f / z1[0]);
    const float iZq = uniform(1.f / st.rest_mass);
    bool bad = false;
    for (int i = 0; i < k; ++i) bad = bad || sh.node_x[i] < 0;
    if (bad) {
        o.flags |= MDSD_FLAG_BAD_TOKEN;
        o.outcome = MDSD_BAD_TOKEN;
        return;
    }
    constexpr bool KEPT_BY_NOW = KEPT_AT_ENTRY || !STATS;
    float c = 0.f, Wc = 1.f;
    bool decided = false, slabs_current = false;
    int n_rej = 0;
    float rem_k = 0.f;  // WO: unnormalised draft mass outside all k drafted tokens (after the first pass)
    constexpr bool SUMS_LEFT = WO && !STEP;
    if constexpr (WO && STEP) rem_k = uniform(sh.bcast_left);
    // The marked tokens that this lane's chunks hold, one bit per element: a chunk whose byte is 0 in
    // every lane -- nearly all are -- costs a pass one test.  (The tokens' places compared chunk by chunk
    // instead filled the passes with scalars: 390 to 2800 spills of them.)
    constexpr int kWords = (NIT * E + 31) / 32;
    uint32_t marks[kWords] = {};
    auto mark = [&](int token) {
        const int v = token + rp.head, chunk = v / E, s = chunk / 64;
        const int bit = (s / kWaves) * E + v % E;
        const bool here = s % kWaves == wave_id() && (chunk & 63) == (int)(threadIdx.x & 63);
#pragma unroll
        for (int i = 0; i < kWords; ++i) marks[i] |= here && bit / 32 == i ? 1u << (bit & 31) : 0u;
    };
    // One pass over both rows: slab sums (and total) of max(p - c_new q, 0), rejected tokens counting 0.
    // KEPT: part of the draft row comes from LDS.  REM (without replacement, the first rejected round):
    // the draft mass outside the drafted tokens is summed as well; the marks are then those of all drafted
    // tokens, of which the first is the rejected one.  Otherwise they are those of the rejected tokens.
    auto residual_pass = [&](float c_new, auto KEPT, auto REM_) {
        constexpr bool REM = decltype(REM_)::value;
        const float c_iZq = c_new * iZq;
        float lane_rem = 0.f;
        SlabSums<NIT> sums;
        // Opaque copies: the weights of the target row do not change from round to round, and
        // the compiler would otherwise compute all of them once, ahead of the rounds, and hold
        // one register per element.
        int lane_o = threadIdx.x & 63, wave_o = wave_id();
        ExpW cpo = cp;
        asm volatile("" : "+v"(lane_o), "+s"(wave_o), "+s"(cpo.ms));
        for_each_streamed_cached<1, kDraftChunksKept<NIT>, decltype(KEPT)::value>(
            lane_o, wave_o, sp, rq, ExpW::fill(), q_kept, [&](int it, int, int chunk, const uint4& dp, const uint4& dq) {
            const uint32_t bits = marks[it * E / 32] >> (it * E % 32);
            const bool some = __ballot((bits & ((1u << E) - 1u)) != 0) != 0;
            float part[2];
            auto half = [&](auto H) {
                constexpr int hv = decltype(H)::value;
                float ep[HE], eq[HE], w[HE];
                unpack_half<DT, hv>(dp, ep);
                unpack_half<DT, hv>(dq, eq);
#pragma unroll
                for (int e = 0; e < HE; ++e) {
                    eq[e] = cq(eq[e]);
                    w[e] = rrs_term01(cpo(ep[e]), eq[e], iZp, c_iZq);
                }
                if (__builtin_expect(some, 0)) {
                    asm volatile("" ::: "memory");
                    const int v_first = REM ? uniform(sh.node_x[0]) + rp.head : 0;
#pragma unroll
                    for (int e = 0; e < HE; ++e) {
                        const bool marked = (bits >> (hv * HE + e)) & 1u;
                        w[e] = (REM ? chunk * E + hv * HE + e == v_first : marked) ? 0.f : w[e];
                        if constexpr (REM) eq[e] = marked ? 0.f : eq[e];
                    }
                }
                part[hv] = HE == 4 ? (w[0] + w[1]) + (w[HE - 2] + w[HE - 1]) : w[0] + w[1];
                if constexpr (REM) lane_rem += HE == 4 ? (eq[0] + eq[1]) + (eq[HE - 2] + eq[HE - 1]) : eq[0] + eq[1];
            };
            half(std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            half(std::integral_constant<int, 1>{});
            sums.put(it, part[0] + part[1]);
        });
        sums.store(sh.slab_w, rp.nslab);
        if constexpr (REM) {
            float rr[1] = {lane_rem};
            block_sum<kWaves, 1>(rr, sh.red, phase);
            rem_k = rr[0];
        }
        __syncthreads();
        return slab_total(rp.nslab, [&](int j) { return sh.slab_w[j]; });
    };
    // WO: unnormalised draft mass left before round i (i >= 1): what no draft took, plus the
    // drafts still to come (a repeated token counts once)
    auto mass_left = [&](int i) {
        float m = rem_k;
        for (int j = k - 1; j >= i; --j) {
            bool dup = false;
            for (int l = 0; l < j; ++l) dup = dup || (sh.node_x[l] == sh.node_x[j]);
            if (!dup) m += cq(sh.node_lq[j]);
        }
        return m;
    };

    for (int i = 0; i < k; ++i) {
        const int xi = uniform(sh.node_x[i]);
        const float px = cp(sh.node_lp[i]) * iZp, qx = cq(sh.node_lq[i]) * iZq, ui = sh.node_u[i];
        bool seen = false;
        for (int j = 0; j < i; ++j) seen = seen || (sh.node_x[j] == xi);
        const float Ux = seen ? 0.f : fmaxf(fmaf(-c, qx, px), 0.f);
        // draft probability of x_i in this round and the factor that rescales q; without
        // replacement a repeated token has no mass left
        float Qi = qx, rho = 1.f;
        if (WO && i > 0) {
            const float left = mass_left(i);
            Qi = seen ? 0.f : cq(sh.node_lq[i]) / left;
            rho = 1.f / (left * iZq);
        }
        if (ui * Qi * Wc < Ux) {  // Alg. 1 returns at the first acceptance
            o.outcome = i;
            o.token = xi;
            decided = true;
            break;
        }
        const float c_new = fmaf(Wc, rho, c);
        n_rej = i + 1;
        if (i > 0) __syncthreads();  // earlier readers of the slab sums are done
        float W_new;
        if (i == 0) {
            if constexpr (SUMS_LEFT)
                for (int j = 1; j < k; ++j) mark(sh.node_x[j]);
            mark(xi);
            W_new = residual_pass(c_new, std::bool_constant<KEPT_BY_NOW>{}, std::bool_constant<SUMS_LEFT>{});
            if constexpr (SUMS_LEFT) {
#pragma unroll
                for (int j = 0; j < kWords; ++j) marks[j] = 0;
                mark(xi);
            }
        } else {
            mark(xi);
            W_new = residual_pass(c_new, std::true_type{}, std::false_type{});
        }
        if (W_new > 0.f) {
            c = c_new;
            Wc = W_new;
            slabs_current = true;
        } else {
            o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
            slabs_current = false;
        }
        if constexpr (WO) {
            if (!(mass_left(i + 1) > 0.f)) {
                o.flags |= MDSD_FLAG_Q_EXHAUSTED;
                break;
            }
        }
    }
    // A first draft accepted: the mass is 1 as it stands, and only the distribution itself needs the pass over both rows
    // (31-node trees asked for masses, three nodes in five: 64 trees of 32000 without records 56.9 -> 51.9 us).
    if (decided && (!need_full || (n_rej == 0 && !rprob))) {
        o.rmass = 1.f;
        return;
    }
    if (!slabs_current) {
        __syncthreads();
        residual_pass(c, std::bool_constant<KEPT_BY_NOW>{}, std::false_type{});  // rare: the pass once more, with the c of before
    }
    const float c_iZq = c * iZq;
    auto cw = [&](int s, float(&w)[E]) {
        rrs_chunk_w<DT, ExpW, true>(rp, rq, cp, cq, iZp, c_iZq, nullptr, 0, s, w);
        const int chunk = s * 64 + (threadIdx.x & 63);
        for (int j = 0; j < n_rej; ++j) {
            const int off = sh.node_x[j] + rp.head - chunk * E;
#pragma unroll
            for (int e = 0; e < E; ++e) w[e] = (e == off) ? 0.f : w[e];
        }
    };
    auto sv = [&](int j) { return sh.slab_w[j]; };
    const float W = slab_total(rp.nslab, sv);
    o.rmass = n_rej == 0 ? 1.f : W;
    if (!decided) {
        // (the kernel's first thread writes the outputs: the first wave's draw is the one that counts)
        int v = -1;
        if (wave_id() == 0) v = icdf_slabs<E>(rp.nslab, sh.node_u[k], W, sv, cw);
        o.token = v < 0 ? -1 : v - rp.head;
        if (v < 0) o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
    }
    if (rprob) write_resid_prob<DT>(rprob, rp, W, cw);
}

template <int DT, int NIT, bool MASKED, bool WO, bool STATS>
__device__ __forceinline__ NodeOut rrs_node_resident(const Params& P, const NodeId& id, Shared& sh,
                                                     uint4 (*q_kept)[kWG], int& phase)
{
    const bool need_full = (P.resid_mass != nullptr) || (P.resid_prob != nullptr);
    float* rprob = P.resid_prob ? P.resid_prob + id.row * (int64_t)P.V : nullptr;
    const RowView rp = make_row<DT>(P.target, P.ld_t, id.row, P.V);
    RowSrc<DT, NIT, MASKED> sp;
    sp.issue(rp, ExpW::fill());
    NodeOut o{MDSD_NONE, -1, 0, 0.f};
    if (id.c0 < 0) {
        leaf_resident<DT, NIT, MASKED, STATS, false>(P, rp, sp, P.u[id.row * (P.k + 1) + P.k], rprob, sh, phase, o);
    } else {
        const RowView rq = make_row<DT>(P.draft, P.ld_d, id.row, P.V);
        rrs_resident<DT, NIT, MASKED, WO, STATS>(P, id, rp, rq, sp, need_full, rprob, sh, q_kept, phase, o);
    }
    write_node_outputs(P, id, o.outcome, o.token, o.rmass, o.flags);
    return o;
}

template <int DT, int NIT, bool MASKED, bool WO, bool STATS>
__global__ __launch_bounds__(kWG, (kWG != 512 || NIT > 8 ? 4 : kStatsWavesPerSimd)) void rrs_verify_resident(const Params P)
{
    __shared__ Shared sh;
    __shared__ uint4 q_kept[kDraftChunksKept<NIT>][kWG];
    int phase = 0;
    rrs_node_resident<DT, NIT, MASKED, WO, STATS>(P, node_of_block(P), sh, q_kept, phase);
}

// Path-only: one workgroup per tree.  A node's decisions are the same in every wave; its token, and the draw that may give
// it, are the first wave's, which writes them.  Where the row was streamed from memory in every round before, draft and path
// call, us, 31-node trees: bf16 32000, 16 trees RRS 46.6 -> 34.2, RRSw 57.5 -> 39.1, 64 68.5 -> 49.4, 77.3 -> 53.0, 1000 287 -> 260,
// 312 -> 267; 50304, 64 83 -> 63, 100 -> 71; 64 21-node trees of 32000, k = 4, 65.5 -> 43.2, 85.6 -> 55.4.
// Two workgroups per CU are asked for, at which the bf16 instances of eight chunks per lane on aligned rows and those of sixteen
// spill 13 to 17 vector registers (up to 68 bytes a lane), fp32 ones of sixteen up to 10, and the walk's scalars go to vector
// lanes (90 to 190 of them).  What one workgroup per CU would give has not been measured.
template <int DT, int NIT, bool MASKED, bool WO, bool STATS>
__global__ __launch_bounds__(kWG, 4) void rrs_path_resident(const Params P)
{
    __shared__ Shared sh;
    __shared__ uint4 q_kept[kDraftChunksKept<NIT>][kWG];
    int phase = 0;
    walk_and_verify(P, [&](const NodeId& id) {
        return rrs_node_resident<DT, NIT, MASKED, WO, STATS>(P, id, sh, q_kept, phase);
    });
}

}  // namespace MDSD_NS
