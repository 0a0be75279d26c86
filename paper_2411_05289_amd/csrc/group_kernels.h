// Draft and verify kernels for short rows: a node is handled by a group of G lanes (G = 4 to 64, four
// 16-byte chunks of each row per lane), 64 / G nodes share a wavefront, and a node's rows live in
// registers from the first load to the last draw.
//
// What bounds such nodes is the number of wavefronts and the instructions each of them issues, not
// bandwidth: a wavefront lives for two or three trips to memory whatever it works on, and a reduction,
// a draw or an acceptance test costs the same issue slots for one node as for sixteen.  So the group is
// the smallest that holds the row, every cross-lane step is a DPP move inside the group (permlane swaps
// from 32 lanes on), the weights are formed once and kept, and nothing goes through LDS but the
// outcomes that the tree walk reads.  Toy workload (V = 50 fp32, 307200 nodes, G = 4) against one
// wavefront per node: draft 113 -> 12 us, verify 150 -> 25 us, the step 265 -> 41 us.
//
// Groups of one wavefront may take different branches: a cross-lane step only ever uses values of its
// own group's lanes, which are always active together.
#pragma once
#include "launch.h"

#include "launch_group.h"

namespace mdsd {

constexpr int kGroupChunks = 4;  // chunks of a row per lane
constexpr int kGroupWavesPerSimd = 4;

// ---------------------------------------------------------------- steps inside a group of G lanes
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
constexpr int kRowMirror = 0x140;  // lane i reads lane 15 - i of its row of 16

// f over the G lanes of the group, the same bits in every lane (f commutative)
template <int G, class T, class F>
__device__ __forceinline__ T group_reduce(T v, F f)
{
    auto step = [&](auto CTRL) {
        v = f(v, __builtin_bit_cast(T, dpp_mov<decltype(CTRL)::value>(__builtin_bit_cast(int, v))));
    };
    if constexpr (G >= 2) step(std::integral_constant<int, kQuadXor1>{});
    if constexpr (G >= 4) step(std::integral_constant<int, kQuadXor2>{});
    if constexpr (G >= 8) step(std::integral_constant<int, kRowHalfMirror>{});  // the quads hold one value each
    if constexpr (G >= 16) step(std::integral_constant<int, kRowMirror>{});     // and so do the halves
    // the two results of a swap hold the values of the even and of the odd rows (halves) in every lane
    if constexpr (G >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v),
                                                        __builtin_bit_cast(uint32_t, v), false, false);
        v = f(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
    }
    if constexpr (G >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v),
                                                        __builtin_bit_cast(uint32_t, v), false, false);
        v = f(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
    }
    return v;
}
template <int G>
__device__ __forceinline__ float group_sum(float v)
{
    return group_reduce<G>(v, [](float a, float b) { return a + b; });
}
template <int G>
__device__ __forceinline__ float group_max(float v)
{
    return group_reduce<G>(v, [](float a, float b) { return fmaxf(a, b); });
}
template <int G>
__device__ __forceinline__ int group_min(int v)
{
    return group_reduce<G>(v, [](int a, int b) { return min(a, b); });
}
template <int G>
__device__ __forceinline__ int group_max(int v)
{
    return group_reduce<G>(v, [](int a, int b) { return max(a, b); });
}

// sum of the lanes below this one in its group
template <int G>
__device__ __forceinline__ float group_sum_below(float v, int l)
{
    // rows of 16 lanes hold whole groups or are part of one; a lane of a smaller group drops what a
    // shift brought from its neighbour
    auto shifted = [&](auto CTRL, int d) {
        const float t = dpp<decltype(CTRL)::value>(0.f, v);
        v += (G >= 16 || l >= d) ? t : 0.f;
    };
    shifted(std::integral_constant<int, kRowShr1>{}, 1);
    if constexpr (G > 2) shifted(std::integral_constant<int, kRowShr2>{}, 2);
    if constexpr (G > 4) shifted(std::integral_constant<int, kRowShr4>{}, 4);
    if constexpr (G > 8) shifted(std::integral_constant<int, kRowShr8>{}, 8);
    if constexpr (G > 16) v += dpp<kRowBcast15, 0xa>(0.f, v);
    if constexpr (G > 32) v += dpp<kRowBcast31, 0xc>(0.f, v);
    const float below = G <= 16 ? dpp<kRowShr1>(0.f, v) : dpp<kWaveShr1>(0.f, v);
    return l == 0 ? 0.f : below;
}

// ---------------------------------------------------------------- a row in a group's registers
// Part i of a row is its chunks i G .. i G + G - 1, one per lane, so that a load instruction of a group
// covers 16 G consecutive bytes.  A row of `row_chunks` chunks has ceil(row_chunks / G) parts, the same
// for every row of a launch: parts that no row has are skipped by a scalar branch.
template <int N, class F>
__device__ __forceinline__ void for_parts(int parts, F&& f)
{
    static_for<N>([&](auto I) {
        if (decltype(I)::value == 0 || decltype(I)::value < parts) f(I);
    });
}

// A row's elements, those that are not the row's holding the fill of CV (logits: -inf, weight 0).
// KEEP = true: unpacked, and from form_weights() on as weights.  KEEP = false: as they were stored, the
// weights formed again by every pass: half the registers for bf16 rows.
template <int DT, int G, class CV, bool KEEP>
struct GroupRow {
    static constexpr int E = Elem<DT>::kPerChunk;
    static constexpr int C = kGroupChunks;
    static constexpr bool kKeep = KEEP;
    uint4 d[C];
    float w[KEEP ? C : 1][E];
    CV cv;

    __device__ __forceinline__ void ask(const RowView& r, int l, int parts)
    {
        for_parts<C>(parts, [&](auto I) { d[I] = fetch_chunk(r, I * G + l); });
    }
    // which elements of this lane's chunk of part i are the row's: f(e, true or false) for all e, called
    // for parts only that may have others.  P.masked: some row of the call may start or end inside a
    // chunk (the same for the whole launch); only the first part can hold elements in front of a row,
    // only parts that reach past V elements behind it.
    template <int I, class F>
    static __device__ __forceinline__ void own_elements(const RowView& r, int l, const Params& P, F f)
    {
        const int chunk = I * G + l;
        if (P.masked) {
            const int x0 = chunk * E - r.head;
            if constexpr (I == 0) {
#pragma unroll
                for (int e = 0; e < E; ++e) f(e, (uint32_t)(x0 + e) < (uint32_t)P.V);
            } else if ((I + 1) * G * E > P.V) {
#pragma unroll
                for (int e = 0; e < E; ++e) f(e, x0 < P.V - e);
            }
        } else if ((I + 1) * G > P.row_chunks) {
#pragma unroll
            for (int e = 0; e < E; ++e) f(e, chunk < P.row_chunks);
        }
    }
    __device__ __forceinline__ void take(const RowView& r, int l, const Params& P, int parts)
    {
        for_parts<C>(parts, [&](auto I) {
            if constexpr (KEEP) {
                unpack<DT>(d[I], w[I]);
                own_elements<decltype(I)::value>(r, l, P, [&](int e, bool own) { w[I][e] = own ? w[I][e] : CV::fill(); });
            } else {
                own_elements<decltype(I)::value>(r, l, P, [&](int e, bool own) { set(I, e, !own); });
            }
        });
    }
    // KEEP = false: put `value` into element e of part i where `there`
    __device__ __forceinline__ void set(int i, int e, bool there, float value = CV::fill())
    {
        const uint32_t fb = as_i(value);
        uint32_t* word = DT == 0 ? &(&d[i].x)[e] : &(&d[i].x)[e / 2];
        if constexpr (DT == 0) {
            *word = there ? fb : *word;
        } else {
            const uint32_t half = e % 2 ? 0xffff0000u : 0x0000ffffu, m = there ? half : 0u;
            *word = (*word & ~m) | ((e % 2 ? fb : fb >> 16) & m);
        }
    }
    // this lane's stored elements (KEEP after form_weights(): weights) of part I
    template <int I>
    __device__ __forceinline__ void elements(float (&x)[E]) const
    {
        if constexpr (KEEP) {
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = w[I][e];
        } else {
            unpack<DT>(d[I], x);
        }
    }
    // this lane's maximum of every part, and the row's (fmed3 with +inf is a maximum that drops NaNs
    // without first quieting its operands)
    __device__ __forceinline__ float max_of_row(float (&m)[C], int parts) const
    {
        float all = -__builtin_inff();
        for_parts<C>(parts, [&](auto I) {
            float x[E];
            elements<decltype(I)::value>(x);
            m[I] = -__builtin_inff();
#pragma unroll
            for (int e = 0; e < E; ++e) m[I] = __builtin_amdgcn_fmed3f(m[I], x[e], __builtin_inff());
            all = fmaxf(all, m[I]);
        });
        return group_max<G>(all);
    }
    __device__ __forceinline__ float max_of_row(int parts) const
    {
        float m[C];
        return max_of_row(m, parts);
    }
    // lowest virtual index that holds M, the largest of the lanes' part maxima m, else `none`
    __device__ __forceinline__ int first_index_of(float M, const float (&m)[C], int l, int none, int parts) const
    {
        int part = -1;
        for_parts<C>(parts, [&](auto I) { part = part < 0 && m[I] == M ? (int)I : part; });
        int at = INT_MAX;
        if (part >= 0) {
            float x[E];
            pick_elements(part, x, parts);
#pragma unroll
            for (int e = E - 1; e >= 0; --e) at = x[e] == M ? (part * G + l) * E + e : at;
        }
        at = group_min<G>(at);
        return at == INT_MAX ? none : at;
    }
    // from here on weights() gives the weights
    __device__ __forceinline__ void form_weights(CV c, int parts)
    {
        cv = c;
        if constexpr (KEEP)
            for_parts<C>(parts, [&](auto I) {
#pragma unroll
                for (int e = 0; e < E; ++e) w[I][e] = cv(w[I][e]);
            });
    }
    template <int I>
    __device__ __forceinline__ void weights(float (&x)[E]) const
    {
        elements<I>(x);
        if constexpr (!KEEP)
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = cv(x[e]);
    }
    // weights 4 H .. 4 H + 3 of part I
    template <int I, int H>
    __device__ __forceinline__ void four_weights(float (&x)[4]) const
    {
        if constexpr (KEEP) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = w[I][4 * H + e];
        } else if constexpr (DT == 0) {
            weights<I>(x);
        } else {
            const uint32_t w0 = H == 0 ? d[I].x : d[I].z, w1 = H == 0 ? d[I].y : d[I].w;
            x[0] = cv(__builtin_bit_cast(float, w0 << 16));
            x[1] = cv(__builtin_bit_cast(float, w0 & 0xffff0000u));
            x[2] = cv(__builtin_bit_cast(float, w1 << 16));
            x[3] = cv(__builtin_bit_cast(float, w1 & 0xffff0000u));
        }
    }
    // the same of part `part` (known at run time)
    __device__ __forceinline__ void pick_elements(int part, float (&x)[E], int parts) const
    {
        if constexpr (KEEP) {
            elements<0>(x);
            for_parts<C>(parts, [&](auto I) {
                if constexpr (decltype(I)::value > 0) {
#pragma unroll
                    for (int e = 0; e < E; ++e) x[e] = part == I ? w[I][e] : x[e];
                }
            });
        } else {
            uint4 c = d[0];
            for_parts<C>(parts, [&](auto I) {
                if constexpr (decltype(I)::value > 0) {
                    const bool here = part == I;
                    c.x = here ? d[I].x : c.x;
                    c.y = here ? d[I].y : c.y;
                    c.z = here ? d[I].z : c.z;
                    c.w = here ? d[I].w : c.w;
                }
            });
            unpack<DT>(c, x);
        }
    }
    __device__ __forceinline__ void pick(int part, float (&x)[E], int parts) const
    {
        pick_elements(part, x, parts);
        if constexpr (!KEEP)
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = cv(x[e]);
    }
    // where virtual index v lies among this lane's elements (part * E + element); -1 in other lanes
    static __device__ __forceinline__ int place_of(int v, int l)
    {
        const int chunk = v / E;
        return (chunk & (G - 1)) == l ? chunk / G * E + v % E : -1;
    }
    // the element at this lane's `place` has no weight from here on (after form_weights())
    __device__ __forceinline__ void drop(int place, int parts)
    {
        for_parts<C>(parts, [&](auto I) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (KEEP)
                    w[I][e] = place == I * E + e ? 0.f : w[I][e];
                else
                    set(I, e, place == I * E + e);
            }
        });
    }
    // undo drop(): the element's weight and its stored value
    __device__ __forceinline__ void put_back(int place, float weight, float stored, int parts)
    {
        for_parts<C>(parts, [&](auto I) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (KEEP)
                    w[I][e] = place == I * E + e ? weight : w[I][e];
                else
                    set(I, e, place == I * E + e, stored);
            }
        });
    }
    // the group's sum of every part
    __device__ __forceinline__ void part_sums(float (&t)[C], int parts) const
    {
#pragma unroll
        for (int i = 0; i < C; ++i) t[i] = 0.f;
        for_parts<C>(parts, [&](auto I) {
            float x[E];
            weights<decltype(I)::value>(x);
            t[I] = group_sum<G>(chunk_sum<E>(x));
        });
    }
};

__device__ __forceinline__ float parts_total(const float (&t)[kGroupChunks])
{
    static_assert(kGroupChunks == 4, "a balanced tree over the parts");
    return (t[0] + t[1]) + (t[2] + t[3]);
}
// Sum of a row's weights.  Part by part across the lanes, then over the parts: for rows of up to 64
// elements the balanced tree over the chunks in their order, whose rounding the residual of a peaked
// row sees a hundredfold; chunks summed inside the lanes first would save two steps and err more.
template <class Row>
__device__ __forceinline__ float row_total(const Row& r, int parts)
{
    float t[kGroupChunks];
    r.part_sums(t, parts);
    return parts_total(t);
}

// Inverse CDF: the virtual index of the first element whose running sum exceeds u * W, where t holds
// the part sums and W their total; part_of(part, x) gives this lane's weights of a part.  Elements
// without weight are never returned; if rounding leaves no crossing the last element with weight is
// taken; -1 without mass.  The same in every lane of the group.
template <int E, int G, class PartOf>
__device__ __forceinline__ int group_draw(const float (&t)[kGroupChunks], float W, float u, int l, PartOf part_of)
{
    if (!(W > 0.f)) return -1;
    float bound = u * W, before = 0.f, run = 0.f;
    int part = -1, last = 0;
#pragma unroll
    for (int i = 0; i < kGroupChunks; ++i) {
        const float next = run + t[i];
        if (part < 0 && next > bound) {
            part = i;
            before = run;
        }
        if (t[i] > 0.f) last = i;
        run = next;
    }
    if (part < 0) {
        part = last;
        bound = __builtin_inff();
    }
    float x[E];
    part_of(part, x);
    run = before + group_sum_below<G>(chunk_sum<E>(x), l);
    const int v0 = (part * G + l) * E;
    int hit = INT_MAX;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        run += x[e];
        if (hit == INT_MAX && x[e] > 0.f && run > bound) hit = v0 + e;
    }
    hit = group_min<G>(hit);
    if (hit == INT_MAX) {  // no crossing: the last element with weight
        hit = -1;
#pragma unroll
        for (int e = 0; e < E; ++e) hit = x[e] > 0.f ? v0 + e : hit;
        hit = group_max<G>(hit);
    }
    return hit;
}

// write norm(weights) of the row: weights_of(I, w) gives this lane's weights of part I
template <int E, int G, class WeightsOf>
__device__ __forceinline__ void group_write_prob(float* out, const RowView& r, int l, int parts, float W,
                                                 WeightsOf weights_of)
{
    const float iW = W > 0.f ? 1.f / W : 0.f;
    for_parts<kGroupChunks>(parts, [&](auto I) {
        const int x0 = (I * G + l) * E - r.head;
        float w[E];
        weights_of(I, w);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((uint32_t)(x0 + e) < (uint32_t)(r.nvirt - r.head)) out[x0 + e] = w[e] * iW;
    });
}

// With the draft call's record of the draft row at hand a node that its first tests decide never needs
// that row.  SpecHub nodes of 16 lanes and more ask for it only then: half of its traffic is saved (60000
// nodes of 1000 bf16 elements 81 -> 68 us).  Smaller groups ask for it together with the target row: a
// wavefront holds so many nodes that one of them nearly always needs it, and all would wait for another
// trip to memory.  The RRS methods always do so: every rejection needs the row at once, and a row that may
// or may not be there yet costs them a third of their wavefronts in registers (98 -> 130 us).
template <int G, int METHOD>
constexpr bool kLateDraft = G >= 16 && METHOD == kSpecHub;

// Rows kept as weights: fp32 rows (the stored values take the same registers) and the RRS methods, which
// use a row's weights once per round.  bf16 SpecHub nodes use them once or twice: formed again they cost
// less than the registers.
template <int DT, int METHOD>
constexpr bool kKeepWeights = DT == 0 || METHOD != kSpecHub;

// ---------------------------------------------------------------- one node's draft
// What a group's draft leaves in its lanes: the record, and SpecHub's pair.
struct GroupDrafted {
    mdsd_row_stats record;
    int x1, x2;
};

// The entries of a leaf, which drafts nothing, by the lane that calls it.
__device__ __forceinline__ void group_leaf_draft(const Params& P, int64_t row, int32_t* flags)
{
    if (P.hub_out) P.hub_out[row] = -1;
    if (flags) flags[row] = 0;
    if (P.stats_out) P.stats_out[row] = mdsd_row_stats{0.f, 0.f, -1, 0};
}

// The draft of one node with children.  q: its draft row, asked for; behind the call it holds the row's weights.  ur: the
// node's uniforms, the first of which is u0.  put(i, x): draft token i, the same in every lane of the group.
template <int DT, bool LOGITS, int METHOD, int G, class Row, class Put>
__device__ __forceinline__ GroupDrafted group_draft_node(const Params& P, const RowView& rq, Row& q, int l, int parts,
                                                         const float* ur, float u0, int64_t row, int32_t* flags_out, Put put)
{
    constexpr int E = Elem<DT>::kPerChunk;
    constexpr int C = kGroupChunks;
    using CV = ToWeight<LOGITS>;
    const int k = P.k;
    GroupDrafted out{mdsd_row_stats{0.f, 0.f, -1, 0}, -1, -1};
    q.take(rq, l, P, parts);
    CV cq{0.f, 0.f};
    float m = 0.f;
    int hub = rq.head;
    int flags = 0;
    if (LOGITS || METHOD == kSpecHub) {
        float lane_m[C];
        m = q.max_of_row(lane_m, parts);
        if constexpr (METHOD == kSpecHub) hub = q.first_index_of(m, lane_m, l, rq.head, parts);
    }
    if constexpr (LOGITS) {
        cq.s = P.scale_d;
        cq.ms = m * cq.s;
    }
    q.form_weights(cq, parts);
    float t[C];
    q.part_sums(t, parts);
    // removed places are taken out where a part is looked at; only the sum of their part changes
    uint32_t removed = 0;
    auto part_of = [&](int part, float(&x)[E]) {
        q.pick(part, x, parts);
        const uint32_t bits = removed >> (part * E);
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = as_f(as_i(x[e]) & __builtin_amdgcn_sbfe(~bits, e, 1));
    };
    auto remove = [&](int v) {
        const int place = Row::place_of(v, l), part = v / (E * G);
        removed |= place < 0 ? 0u : 1u << place;
        float x[E];
        part_of(part, x);
        const float s = group_sum<G>(chunk_sum<E>(x));
#pragma unroll
        for (int i = 0; i < C; ++i) t[i] = part == i ? s : t[i];
    };
    if constexpr (METHOD == kSpecHub) {
        const float u1 = ur[1];
        const int v = group_draw<E, G>(t, parts_total(t), u0, l,
                                       [&](int part, float(&x)[E]) { q.pick(part, x, parts); });
        const int first = v;
        int second = hub;
        if (v == hub || P.stats_out) {
            remove(hub);
            const float rest = parts_total(t);
            out.record = mdsd_row_stats{m, rest, hub - rq.head, 0};
            if (P.stats_out && l == 0) P.stats_out[row] = out.record;
            if (v == hub) {
                second = group_draw<E, G>(t, rest, u1, l, part_of);
                if (second < 0) {
                    second = hub;
                    flags |= MDSD_FLAG_DEGENERATE_HUB;
                }
            }
        }
        out.x1 = first < 0 ? -1 : first - rq.head;
        out.x2 = second - rq.head;
        put(0, out.x1);
        put(1, out.x2);
    } else {
        int prev = rq.head;
        float W = parts_total(t), u = u0;
        out.record = mdsd_row_stats{m, W, -1, 0};
        if (P.stats_out && l == 0) P.stats_out[row] = out.record;
        for (int i = 0; i < k; ++i) {
            const float next_u = i + 1 < k ? ur[i + 1] : 0.f;
            int v = group_draw<E, G>(t, W, u, l, part_of);
            if (v < 0) {
                v = prev;
                flags |= MDSD_FLAG_Q_EXHAUSTED;
            } else if (METHOD == kRRSw && i + 1 < k) {
                remove(v);
                W = parts_total(t);
            }
            prev = v;
            u = next_u;
            put(i, v - rq.head);
        }
    }
    if (l == 0) {
        if (P.hub_out) P.hub_out[row] = METHOD == kSpecHub ? hub - rq.head : -1;
        if (flags_out) flags_out[row] = flags;
    }
    return out;
}

// ---------------------------------------------------------------- one node's verification
// The decisions, bounds and flags are those of verify_node() (verify_generic.h); what differs is where
// the weights live and how sums travel.  l: this lane's number in its group.
// STEP: the node is drafted first, and its draft row's weights, its record and its tokens stay where they are (the RRS
// methods' tokens in step_tokens, the group's own part of the LDS); the target row is asked for before the draft.  One launch
// instead of two, and each row read and unpacked once (us a step): toy workload 40.1 -> 34.1; 100 15-node trees of 1000 bf16 elements
// SpecHub 14.7 -> 10.4, RRSw 19.0 -> 15.5, 4000 RRS 70.2 -> 58.9; 1000 of 60 12.9 -> 10.5.
template <int DT, bool LOGITS, int METHOD, int G, bool STEP = false>
__device__ __forceinline__ NodeOut group_verify_node(const Params& P, const NodeId& id, int l, int* step_tokens = nullptr)
{
    constexpr int E = Elem<DT>::kPerChunk;
    constexpr int C = kGroupChunks;
    using CV = ToWeight<LOGITS>;
    using Row = GroupRow<DT, G, CV, kKeepWeights<DT, METHOD>>;
    const int k = P.k;
    const float* ur = P.u + id.row * (k + 1);
    const bool need_full = (P.resid_mass != nullptr) || (P.resid_prob != nullptr);
    float* rprob = P.resid_prob ? P.resid_prob + id.row * (int64_t)P.V : nullptr;
    NodeOut o{MDSD_NONE, -1, 0, 0.f};
    const int parts = (P.row_chunks + G - 1) / G;

    const RowView rp = make_row<DT>(P.target, P.ld_t, id.row, P.V);
    Row p;
    p.ask(rp, l, parts);

    if constexpr (STEP) {
        if (id.n == 0 && l == 0) P.tokens_out[id.row] = -1;
    }
    if (id.c0 < 0) {
        // ---- leaf: the k = 0 case of Alg. 1, token ~ p
        const float u = ur[k];
        if constexpr (STEP) {
            if (l == 0) group_leaf_draft(P, id.row, P.draft_flags);
        }
        p.take(rp, l, P, parts);
        CV cp{0.f, 0.f};
        if constexpr (LOGITS) {
            cp.s = P.scale_t;
            cp.ms = p.max_of_row(parts) * cp.s;
        }
        p.form_weights(cp, parts);
        float t[C];
        p.part_sums(t, parts);
        const float W = parts_total(t);
        const int v = group_draw<E, G>(t, W, u, l, [&](int part, float(&x)[E]) { p.pick(part, x, parts); });
        o.token = v < 0 ? -1 : v - rp.head;
        if (v < 0) o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
        o.rmass = LOGITS ? 1.f : W;
        if (rprob) group_write_prob<E, G>(rprob, rp, l, parts, W, [&](auto I, float(&w)[E]) { p.template weights<decltype(I)::value>(w); });
        return o;
    }

    const RowView rq = make_row<DT>(P.draft, P.ld_d, id.row, P.V);
    const bool have_stats = STEP || P.stats_in != nullptr;
    Row q;
    if (STEP || !kLateDraft<G, METHOD> || !have_stats) q.ask(rq, l, parts);
    const int32_t* xt = P.tokens + (int64_t)id.b * P.N + id.c0;
    mdsd_row_stats st{0.f, 0.f, 0, 0};
    GroupDrafted drafted;
    if constexpr (STEP) {
        const float* ud = P.u_draft + id.row * k;
        int32_t* out = P.tokens_out + (int64_t)id.b * P.N + id.c0;
        drafted = group_draft_node<DT, LOGITS, METHOD, G>(P, rq, q, l, parts, ud, ud[0], id.row, P.draft_flags, [&](int i, int x) {
            if (l != 0) return;
            out[i] = x;
            if constexpr (METHOD != kSpecHub) step_tokens[i] = x;
        });
        st = drafted.record;
        if constexpr (METHOD != kSpecHub) {
            // lanes of this wavefront only, whose LDS instructions run in order; the compiler has to keep them so
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            xt = step_tokens;
        }
    } else if (have_stats) {
        st = P.stats_in[id.row];
    }
    CV cp{0.f, 0.f}, cq{0.f, 0.f};
    if constexpr (LOGITS) {
        cp.s = P.scale_t;
        cq.s = P.scale_d;
    }
    auto look_up = [&](const RowView& r, int x) { return load_elem<DT>(r, min(max(x, 0), P.V - 1)); };

    if constexpr (METHOD == kSpecHub) {
        const int x1 = STEP ? drafted.x1 : xt[0], x2 = STEP ? drafted.x2 : xt[1];
        const float u0 = ur[0], u1 = ur[1], u2 = ur[2];
        // the stored values at the pair and the hub: asked for here, used behind the row's statistics
        const float lp1 = look_up(rp, x1), lq1 = look_up(rq, x1), lp2 = look_up(rp, x2), lq2 = look_up(rq, x2);
        if (have_stats && (st.hub < 0 || st.hub >= P.V)) st.hub = -1;
        float lpa = 0.f;
        if (have_stats) lpa = look_up(rp, st.hub);
        p.take(rp, l, P, parts);
        if constexpr (LOGITS) cp.ms = p.max_of_row(parts) * cp.s;
        p.form_weights(cp, parts);
        HubScal h;
        h.iZp = 1.f;
        if constexpr (LOGITS) h.iZp = 1.f / row_total(p, parts);
        float mq = st.max_stored, Zq_rest = st.rest_mass, ea_p;
        int a_virt = rq.head + max(st.hub, 0);
        int hub_place = -1;
        // the draft row's weights, the hub's set to 0
        auto take_q = [&]() {
            if constexpr (!STEP) q.take(rq, l, P, parts);
            if (!have_stats) {
                float m[C];
                mq = q.max_of_row(m, parts);
                a_virt = q.first_index_of(mq, m, l, rq.head, parts);  // a row of NaNs has no maximum: stay in bounds
            }
            if constexpr (LOGITS) cq.ms = mq * cq.s;
            if constexpr (!STEP) q.form_weights(cq, parts);
            hub_place = Row::place_of(a_virt, l);
            q.drop(hub_place, parts);
        };
        if (have_stats) {
            if constexpr (LOGITS) cq.ms = mq * cq.s;
            ea_p = cp(lpa);
        } else {
            take_q();
            Zq_rest = row_total(q, parts);
            lpa = load_elem<DT>(rp, a_virt - rq.head);
            ea_p = cp(lpa);
        }
        const int a = a_virt - rq.head;
        const float ea_q = cq(mq);
        h.iZq = LOGITS ? 1.f / (Zq_rest + ea_q) : 1.f;
        h.c = ea_q / Zq_rest;  // q(a) / (1 - q(a)); unused when Zq_rest == 0
        const float pa = ea_p * h.iZp, qa = ea_q * h.iZq;

        bool decided = false, degenerate = false;
        int hub_slot = -1;
        if (have_stats && st.hub < 0) {  // no usable record for this node
            o.flags |= MDSD_FLAG_BAD_PAIR;
            o.outcome = MDSD_BAD_PAIR;
            decided = true;
        } else if (x1 < 0 || x1 >= P.V || x2 < 0 || x2 >= P.V) {
            o.flags |= MDSD_FLAG_BAD_TOKEN;
            o.outcome = MDSD_BAD_TOKEN;
            decided = true;
        } else if (!(Zq_rest > 0.f)) {
            degenerate = true;
            o.flags |= MDSD_FLAG_DEGENERATE_HUB;
            if (x1 != a || x2 != a) {
                o.flags |= MDSD_FLAG_BAD_PAIR;
                o.outcome = MDSD_BAD_PAIR;
                decided = true;
            } else if (u0 * qa < pa) {
                o.outcome = 0;
                o.token = a;
                decided = true;
            }
        } else if (x2 == a && x1 != a) {
            hub_slot = 1;
            const float px = cp(lp1) * h.iZp, qx = cq(lq1) * h.iZq;
            if (u0 * qx < px) {  // pair (x, a): min(p(x)/Q(x,a), 1)
                o.outcome = 0;
                o.token = x1;
                decided = true;
            } else if (LOGITS && u1 * (Zq_rest * h.iZq) < pa - qa) {
                // the hub's test needs no sum: S_xa <= sum_{y != a} q(y) and S_ax <= q(a)
                o.outcome = 1;
                o.token = a;
                decided = true;
            }
        } else if (x1 == a && x2 != a) {
            hub_slot = 0;
            const float px = cp(lp2) * h.iZp, qx = cq(lq2) * h.iZq;
            if (u0 * (h.c * qx) < fmaxf(px - qx, 0.f)) {  // pair (a, x): min(p'(x)/Q(a,x), 1)
                o.outcome = 1;
                o.token = x2;
                decided = true;
            } else if (u1 * qa < pa) {
                // S_ax <= sum_{y != a} Q(a,y) = q(a): the hub's test holds whatever the sum is
                o.outcome = 0;
                o.token = a;
                decided = true;
            }
        } else {
            o.flags |= MDSD_FLAG_BAD_PAIR;
            o.outcome = MDSD_BAD_PAIR;
            decided = true;
        }
        if (decided && !need_full) return o;
        if (have_stats) {
            if constexpr (!STEP && kLateDraft<G, METHOD>) q.ask(rq, l, parts);
            take_q();
        }

        float t[C];
        if (degenerate) {
            // residual of the single-draft case: p with the hub removed
            p.drop(hub_place, parts);
            p.part_sums(t, parts);
            const float W = parts_total(t);
            const int v = group_draw<E, G>(t, W, u2, l, [&](int part, float(&x)[E]) { p.pick(part, x, parts); });
            o.rmass = W * h.iZp;
            if (!decided) {
                o.token = v < 0 ? -1 : v - rp.head;
                if (v < 0) o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
            }
            if (rprob) group_write_prob<E, G>(rprob, rp, l, parts, W, [&](auto I, float(&w)[E]) { p.template weights<decltype(I)::value>(w); });
            return o;
        }
        // ---- residual sums: S_xa = sum Q'(.,a), S_ax = sum Q'(a,.), part sums of p''.  The hub counts in
        // none of them: with its draft weight at 0 already it adds nothing to the first two, and what it
        // adds to the third (its own p) is taken out of its part by taking its target weight as 0
        p.drop(hub_place, parts);
        float s_xa = 0.f, s_ax = 0.f;
#pragma unroll
        for (int i = 0; i < C; ++i) t[i] = 0.f;
        for_parts<C>(parts, [&](auto I) {
            // four elements at a time, so that few values are live at once; the halves of chunk_sum's tree
            float sums[3][E / 4];
            static_for<E / 4>([&](auto H) {
                float pp[4], qq[4], t_xa[4], t_ax[4], w[4];
                p.template four_weights<decltype(I)::value, decltype(H)::value>(pp);
                q.template four_weights<decltype(I)::value, decltype(H)::value>(qq);
#pragma unroll
                for (int e = 0; e < 4; ++e) spechub_terms(pp[e], qq[e], h, t_xa[e], t_ax[e], w[e]);
                sums[0][H] = chunk_sum<4>(t_xa);
                sums[1][H] = chunk_sum<4>(t_ax);
                sums[2][H] = chunk_sum<4>(w);
                if constexpr (!Row::kKeep) __builtin_amdgcn_sched_barrier(0);
            });
            s_xa += E == 8 ? sums[0][0] + sums[0][E / 4 - 1] : sums[0][0];
            s_ax += E == 8 ? sums[1][0] + sums[1][E / 4 - 1] : sums[1][0];
            t[I] = group_sum<G>(E == 8 ? sums[2][0] + sums[2][E / 4 - 1] : sums[2][0]);
        });
        const float S_xa = group_sum<G>(s_xa), S_ax = group_sum<G>(s_ax);
        if (!decided) {
            if (hub_slot == 1) {  // pair (x, a): the hub draws on what the pairs (a,.) left of p(a)
                if (u1 * S_xa < fmaxf(pa - S_ax, 0.f)) {
                    o.outcome = 1;
                    o.token = a;
                    decided = true;
                }
            } else if (u1 * S_ax < pa) {  // pair (a, x)
                o.outcome = 0;
                o.token = a;
                decided = true;
            }
        }
        const float W = parts_total(t);
        o.rmass = W;
        bool from_p = false;
        if (!decided) {
            int v = group_draw<E, G>(t, W, u2, l, [&](int part, float(&x)[E]) {
                float pp[E], qq[E];
                p.pick(part, pp, parts);
                q.pick(part, qq, parts);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    float t0, t1;
                    spechub_terms(pp[e], qq[e], h, t0, t1, x[e]);
                }
            });
            if (v < 0) {
                // no residual mass: fall back to p itself, the hub's weight with it
                o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
                from_p = true;
                p.put_back(hub_place, ea_p, lpa, parts);
                p.part_sums(t, parts);
                v = group_draw<E, G>(t, parts_total(t), u2, l,
                                     [&](int part, float(&x)[E]) { p.pick(part, x, parts); });
            }
            o.token = v < 0 ? -1 : v - rp.head;
        }
        if (rprob) {
            if (from_p) {
                group_write_prob<E, G>(rprob, rp, l, parts, parts_total(t), [&](auto I, float(&w)[E]) { p.template weights<decltype(I)::value>(w); });
            } else {
                group_write_prob<E, G>(rprob, rp, l, parts, W, [&](auto I, float(&w)[E]) {
                    float pp[E], qq[E], t0, t1;
                    p.template weights<decltype(I)::value>(pp);
                    q.template weights<decltype(I)::value>(qq);
#pragma unroll
                    for (int e = 0; e < E; ++e) spechub_terms(pp[e], qq[e], h, t0, t1, w[e]);
                });
            }
        }
        return o;
    } else {
        // ---- RRS / RRSw (Alg. 1).  State: residual U = max(p - c q, 0) with mass Wc.  A rejected
        // token's target weight is set to 0, which takes it out of every later sum and draw.
        constexpr bool WO = (METHOD == kRRSw);
        int x = xt[0];
        float lp = look_up(rp, x), lq = look_up(rq, x), u = ur[0];
        bool bad = false;
        uint32_t drafted = 0;  // without replacement: bits of the drafted tokens' places in this lane
        for (int i = 0; i < k; ++i) {
            const int y = xt[i];
            bad = bad || y < 0 || y >= P.V;
            if constexpr (WO) {
                const int place = Row::place_of(rq.head + min(max(y, 0), P.V - 1), l);
                drafted |= place < 0 ? 0u : 1u << place;
            }
        }
        if (bad) {
            o.flags |= MDSD_FLAG_BAD_TOKEN;
            o.outcome = MDSD_BAD_TOKEN;
            return o;
        }
        p.take(rp, l, P, parts);
        if constexpr (LOGITS) cp.ms = p.max_of_row(parts) * cp.s;
        p.form_weights(cp, parts);
        float iZp = 1.f;
        if constexpr (LOGITS) iZp = 1.f / row_total(p, parts);
        if constexpr (!STEP) q.take(rq, l, P, parts);
        if constexpr (LOGITS) cq.ms = (have_stats ? st.max_stored : q.max_of_row(parts)) * cq.s;
        if constexpr (!STEP) q.form_weights(cq, parts);
        // the draft mass outside the drafted tokens (a sum of positive terms, never a difference)
        float rem_k = 0.f;
        if constexpr (WO) {
            float s[C] = {0.f, 0.f, 0.f, 0.f};
            for_parts<C>(parts, [&](auto I) {
                float w[E];
                q.template weights<decltype(I)::value>(w);
#pragma unroll
                for (int e = 0; e < E; ++e)  // all ones where the place's bit is clear
                    w[e] = as_f(as_i(w[e]) & __builtin_amdgcn_sbfe(~drafted, I * E + e, 1));
                s[I] = group_sum<G>(chunk_sum<E>(w));
            });
            rem_k = parts_total(s);
        }
        auto seen_before = [&](int y, int i) {
            bool seen = false;
            for (int j = 0; j < i; ++j) seen = seen || xt[j] == y;
            return seen;
        };
        // unnormalised draft mass left before round i: what no draft took plus the drafts still to
        // come, a repeated token counting once
        auto mass_left = [&](int i) {
            float m = rem_k;
            for (int j = k - 1; j >= i; --j) {
                const int y = xt[j];
                m += seen_before(y, j) ? 0.f : cq(load_elem<DT>(rq, y));
            }
            return m;
        };
        float Zq;
        if (have_stats)
            Zq = st.rest_mass;
        else if constexpr (WO)
            Zq = mass_left(0);
        else
            Zq = row_total(q, parts);
        const float iZq = LOGITS ? 1.f / Zq : 1.f;

        float c = 0.f, Wc = 1.f;
        float t[C];
        bool parts_current = false;
        bool decided = false;
        int n_rej = 0;
        auto residual_parts = [&](float c_new) {
            const float c_iZq = c_new * iZq;
#pragma unroll
            for (int i = 0; i < C; ++i) t[i] = 0.f;
            for_parts<C>(parts, [&](auto I) {
                float pp[E], qq[E], w[E];
                p.template weights<decltype(I)::value>(pp);
                q.template weights<decltype(I)::value>(qq);
#pragma unroll
                for (int e = 0; e < E; ++e) w[e] = rrs_term(pp[e], qq[e], iZp, c_iZq);
                t[I] = group_sum<G>(chunk_sum<E>(w));
            });
            return parts_total(t);
        };
        for (int i = 0; i < k; ++i) {
            const float px = cp(lp) * iZp, eqx = cq(lq), qx = eqx * iZq;
            const bool seen = seen_before(x, i);
            // draft probability of x_i in this round and the factor that rescales q; without
            // replacement a repeated token has no mass left
            float Qi = qx, rho = 1.f;
            if (WO && i > 0) {
                const float left = mass_left(i);
                Qi = seen ? 0.f : eqx / left;
                rho = 1.f / (left * iZq);
            }
            const float Ux = seen ? 0.f : fmaxf(fmaf(-c, qx, px), 0.f);
            if (u * Qi * Wc < Ux) {  // Alg. 1 returns at the first acceptance
                o.outcome = i;
                o.token = x;
                decided = true;
                break;
            }
            // reject: U <- max(p - (c + Wc rho) q, 0)
            const float c_new = fmaf(Wc, rho, c);
            n_rej = i + 1;
            p.drop(Row::place_of(rp.head + x, l), parts);
            if (i + 1 < k) {
                x = xt[i + 1];
                u = ur[i + 1];
                lp = load_elem<DT>(rp, x);
                lq = load_elem<DT>(rq, x);
            }
            const float W_new = residual_parts(c_new);
            if (W_new > 0.f) {
                c = c_new;
                Wc = W_new;
                parts_current = true;
            } else {
                o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
                parts_current = false;
            }
            if constexpr (WO) {
                if (!(mass_left(i + 1) > 0.f)) {
                    o.flags |= MDSD_FLAG_Q_EXHAUSTED;
                    break;
                }
            }
        }
        if (decided && (!need_full || (n_rej == 0 && !rprob))) {
            o.rmass = 1.f;
            return o;
        }
        if (!parts_current) residual_parts(c);
        const float W = parts_total(t);
        // the mass the rejections took p down to: nothing rejected, nothing taken
        // (rows of probabilities are used as given and need not sum to 1)
        o.rmass = n_rej == 0 ? 1.f : W;
        const float c_iZq = c * iZq;
        if (!decided) {
            const int v = group_draw<E, G>(t, W, ur[k], l, [&](int part, float(&y)[E]) {
                float pp[E], qq[E];
                p.pick(part, pp, parts);
                q.pick(part, qq, parts);
#pragma unroll
                for (int e = 0; e < E; ++e) y[e] = rrs_term(pp[e], qq[e], iZp, c_iZq);
            });
            o.token = v < 0 ? -1 : v - rp.head;
            if (v < 0) o.flags |= MDSD_FLAG_ZERO_RESIDUAL;
        }
        if (rprob)
            group_write_prob<E, G>(rprob, rp, l, parts, W, [&](auto I, float(&w)[E]) {
                float pp[E], qq[E];
                p.template weights<decltype(I)::value>(pp);
                q.template weights<decltype(I)::value>(qq);
#pragma unroll
                for (int e = 0; e < E; ++e) w[e] = rrs_term(pp[e], qq[e], iZp, c_iZq);
            });
        return o;
    }
}

__device__ __forceinline__ int group_first_child(const Params& P, int n)
{
    return walk_first_child(P.first_child, n, P.k, P.N);
}

// the walk of tree b (Sec. 2), node after node; the lane that `writes` writes its results
template <class OutcomeOf, class TokenOf>
__device__ __forceinline__ void lane_walk(const Params& P, int b, bool writes, OutcomeOf outcome_of, TokenOf token_of)
{
    int32_t* em = P.emitted + (int64_t)b * P.depth;
    int n = 0, d = 0;
    for (;;) {
        const int o = outcome_of(n), t = token_of(n);
        if (writes) em[d] = t;
        const int c0 = group_first_child(P, n);
        if (c0 < 0 || o < 0 || o >= P.k || d + 1 >= P.depth) break;
        n = c0 + o;
        ++d;
    }
    if (!writes) return;
    P.accept_depth[b] = d;
    for (int i = d + 1; i < P.depth; ++i) em[i] = -1;
}

__device__ __forceinline__ void write_group_outputs(const Params& P, const NodeId& id, const NodeOut& o)
{
    P.outcome[id.row] = o.outcome;
    P.token[id.row] = o.token;
    if (P.resid_mass) P.resid_mass[id.row] = o.rmass;
    if (P.flags) P.flags[id.row] = o.flags;
}

// The walk by arrival count (see write_node_outputs()), run by the whole group.
template <int G>
__device__ __forceinline__ void count_and_walk(const Params& P, const NodeId& id, const NodeOut& o, int l)
{
    int arrived = 0;
    if (l == 0) {
        __hip_atomic_store(P.outcome + id.row, o.outcome, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(P.token + id.row, o.token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // both stores have reached memory
        arrived = __hip_atomic_fetch_add(P.tree_count + id.b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int base = (int)(threadIdx.x & 63) - l;
    if (__shfl(arrived, base, 64) != P.N - 1) return;
    const int64_t row0 = (int64_t)id.b * P.N;
    if (P.N <= G) {
        // the whole tree in one trip to memory, then on registers
        const int n = min(l, P.N - 1);
        const int oc = load_node_word<true>(P.outcome + row0 + n), tk = load_node_word<true>(P.token + row0 + n);
        lane_walk(P, id.b, l == 0, [&](int m) { return __shfl(oc, base + m, 64); },
                  [&](int m) { return __shfl(tk, base + m, 64); });
    } else if (l == 0) {
        lane_walk(P, id.b, true, [&](int n) { return load_node_word<true>(P.outcome + row0 + n); },
                  [&](int n) { return load_node_word<true>(P.token + row0 + n); });
    }
    if (l == 0) __hip_atomic_store(P.tree_count + id.b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- verify kernels
// TREES = true: a workgroup holds whole trees, as many as its groups take (P.N <= groups of a
// workgroup; internal nodes in its first groups, so that most wavefronts hold nodes of one kind), and
// walks them from LDS: no arrival counters, no launch of its own for the walk.  TREES = false: nodes in
// one dimension, nodes with children first; the walk by arrival count, or left to the caller.
// STEP = true: the nodes are drafted first (see group_verify_node()).
template <int DT, bool LOGITS, int METHOD, int G, bool TREES, bool STEP = false>
__global__ __launch_bounds__(kGroupMaxThreads, kGroupWavesPerSimd) void group_verify_kernel(const Params P)
{
    __shared__ int drafts[STEP && METHOD != kSpecHub ? kGroupMaxThreads / G : 1][MDSD_MAX_K];
    const int l = threadIdx.x & (G - 1), slot = threadIdx.x / G, groups = blockDim.x / G;
    int* mine = drafts[STEP && METHOD != kSpecHub ? slot : 0];
    if constexpr (!TREES) {
        NodeId id;
        if (P.first_child && table_by_waves(G, DT == 1, (int64_t)P.B * P.N)) {
            const int wave = uniform((int)(blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64)), tile = wave / P.N;
            id.n = wave - tile * P.N;
            id.b = tile * (64 / G) + (int)(threadIdx.x & 63) / G;
            if (id.b >= P.B) return;
            id.c0 = group_first_child(P, id.n);
            id.row = (int64_t)id.b * P.N + id.n;
        } else {
            const int64_t item = (int64_t)blockIdx.x * groups + slot;
            if (item >= (int64_t)P.B * P.N) return;
            id = node_of_item(P, (int)item);
        }
        const NodeOut o = group_verify_node<DT, LOGITS, METHOD, G, STEP>(P, id, l, mine);
        if (P.tree_count == nullptr) {
            if (l == 0) write_group_outputs(P, id, o);
            return;
        }
        if (l == 0) {
            if (P.resid_mass) P.resid_mass[id.row] = o.rmass;
            if (P.flags) P.flags[id.row] = o.flags;
        }
        count_and_walk<G>(P, id, o, l);
    } else {
        __shared__ int oc[kGroupMaxThreads / G], tk[kGroupMaxThreads / G];
        const int trees = groups / P.N, b0 = blockIdx.x * trees;
        NodeId id;
        int tree;
        if (P.first_child == nullptr) {
            const int n_leaf = P.N - P.n_internal, inner = trees * P.n_internal;
            if (slot < inner) {
                tree = slot / P.n_internal;
                id.n = slot - tree * P.n_internal;
            } else {
                tree = (slot - inner) / n_leaf;
                id.n = P.n_internal + (slot - inner) - tree * n_leaf;
            }
        } else {
            tree = slot / P.N;
            id.n = slot - tree * P.N;
        }
        id.b = b0 + tree;
        if (tree < trees && id.b < P.B) {
            id.c0 = group_first_child(P, id.n);
            id.row = (int64_t)id.b * P.N + id.n;
            const NodeOut o = group_verify_node<DT, LOGITS, METHOD, G, STEP>(P, id, l, mine);
            if (l == 0) {
                write_group_outputs(P, id, o);
                oc[tree * P.N + id.n] = o.outcome;
                tk[tree * P.N + id.n] = o.token;
            }
        }
        __syncthreads();
        const int b = b0 + (int)threadIdx.x;
        if ((int)threadIdx.x >= trees || b >= P.B) return;
        const int32_t* tree_oc = oc + threadIdx.x * P.N;
        const int32_t* tree_tk = tk + threadIdx.x * P.N;
        lane_walk(P, b, true, [&](int n) { return tree_oc[n]; }, [&](int n) { return tree_tk[n]; });
    }
}

// Wavefront n of a workgroup takes node n of 64 / G trees; the one that comes last walks them (see wave_per_node()).
// Bound by instruction issue (toy workload: 77 % of the kernel's time, 492 instructions per wavefront of 16 nodes).
template <int DT, bool LOGITS, int METHOD, int G, bool STEP = false>
__global__ __launch_bounds__(kGroupMaxThreads, kGroupWavesPerSimd) void group_tree_kernel(const Params P)
{
    constexpr int T = 64 / G;
    __shared__ int drafts[STEP && METHOD != kSpecHub ? kGroupMaxThreads / G : 1][MDSD_MAX_K];
    int* mine = drafts[STEP && METHOD != kSpecHub ? threadIdx.x / G : 0];
    __shared__ int oc[kGroupMaxThreads / 64][T], tk[kGroupMaxThreads / 64][T], arrived;
    if (threadIdx.x == 0) arrived = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, l = lane & (G - 1), tree = lane / G;
    NodeId id;
    id.n = uniform((int)(threadIdx.x / 64));
    id.b = (int)blockIdx.x * T + tree;
    id.c0 = group_first_child(P, id.n);
    id.row = (int64_t)id.b * P.N + id.n;
    if (id.b < P.B) {
        const NodeOut o = group_verify_node<DT, LOGITS, METHOD, G, STEP>(P, id, l, mine);
        if (l == 0) {
            write_group_outputs(P, id, o);
            oc[id.n][tree] = o.outcome;
            tk[id.n][tree] = o.token;
        }
    }
    int before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(&arrived, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (uniform(before) != P.N - 1) return;
    const int b = (int)blockIdx.x * T + lane;
    if (lane >= T || b >= P.B) return;
    lane_walk(P, b, true, [&](int n) { return oc[n][lane]; }, [&](int n) { return tk[n][lane]; });
}

// path-only: a group per tree, node after accepted node
template <int DT, bool LOGITS, int METHOD, int G>
__global__ __launch_bounds__(kGroupThreads) void group_path_kernel(const Params P)
{
    const int l = threadIdx.x & (G - 1), groups = blockDim.x / G;
    const int b = blockIdx.x * groups + threadIdx.x / G;
    if (b >= P.B) return;
    const int64_t row0 = (int64_t)b * P.N;
    int32_t* em = P.emitted + (int64_t)b * P.depth;
    auto unvisited = [&](int i) {
        P.outcome[row0 + i] = MDSD_UNVISITED;
        P.token[row0 + i] = -1;
        if (P.flags) P.flags[row0 + i] = 0;
        if (P.resid_mass) P.resid_mass[row0 + i] = 0.f;
    };
    // trees of up to 64 nodes: the nodes off the path are written at the end.  Larger ones: all nodes
    // first, and lane 0 rewrites the visited ones once those stores have reached memory.
    const bool small_tree = P.N <= 64;
    uint64_t visited = 0;
    if (!small_tree) {
        for (int i = l; i < P.N; i += G) unvisited(i);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    int n = 0, d = 0;
    for (;;) {
        NodeId id;
        id.b = b;
        id.n = n;
        id.c0 = group_first_child(P, n);
        id.row = row0 + n;
        const NodeOut o = group_verify_node<DT, LOGITS, METHOD, G>(P, id, l);
        if (l == 0) {
            write_group_outputs(P, id, o);
            em[d] = o.token;
        }
        visited |= small_tree ? 1ull << n : 0;
        if (id.c0 < 0 || o.outcome < 0 || o.outcome >= P.k || d + 1 >= P.depth) break;
        n = id.c0 + o.outcome;
        ++d;
    }
    if (l == 0) P.accept_depth[b] = d;
    for (int i = d + 1 + l; i < P.depth; i += G) em[i] = -1;
    if (small_tree)
        for (int i = l; i < P.N; i += G)
            if (!((visited >> i) & 1)) unvisited(i);
}

// ---------------------------------------------------------------- draft kernel
// One group per node with children (complete trees: leaves get no group, their parent writes their
// entries; explicit topologies: one group per node).
template <int DT, bool LOGITS, int METHOD, int G>
__global__ __launch_bounds__(kGroupMaxThreads) void group_draft_kernel(const Params P)
{
    using Row = GroupRow<DT, G, ToWeight<LOGITS>, true>;
    const int l = threadIdx.x & (G - 1), groups = blockDim.x / G;
    const int64_t item = (int64_t)blockIdx.x * groups + threadIdx.x / G;
    const int k = P.k;
    // nodes per tree that have a group: a complete tree of one level still has its root
    const int per_tree = P.first_child ? P.N : max(P.n_internal, 1);
    if (item >= (int64_t)P.B * per_tree) return;
    const int b = (int)(item / per_tree), n = (int)(item - (int64_t)b * per_tree);
    const int c0 = group_first_child(P, n);
    const int64_t row = (int64_t)b * P.N + n;
    auto leaf_entries = [&](int64_t r) { group_leaf_draft(P, r, P.flags); };
    if (n == 0 && l == 0) P.tokens_out[row] = -1;
    if (c0 < 0) {
        if (l == 0) leaf_entries(row);
        return;
    }
    const RowView rq = make_row<DT>(P.draft, P.ld_d, row, P.V);
    Row q;
    const int parts = (P.row_chunks + G - 1) / G;
    q.ask(rq, l, parts);
    const float* ur = P.u + row * k;
    const float u0 = ur[0];
    int32_t* xt = P.tokens_out + (int64_t)b * P.N + c0;
    if (P.first_child == nullptr && c0 >= P.n_internal)
        for (int j = l; j < k; j += G) leaf_entries(row - n + c0 + j);
    else if (P.first_child == nullptr && c0 + k > P.n_internal)  // the last internal node's level ends among its children
        for (int j = l; j < k; j += G)
            if (c0 + j >= P.n_internal) leaf_entries(row - n + c0 + j);

    group_draft_node<DT, LOGITS, METHOD, G>(P, rq, q, l, parts, ur, u0, row, P.flags, [&](int i, int x) {
        if (l == 0) xt[i] = x;
    });
}

}  // namespace mdsd
