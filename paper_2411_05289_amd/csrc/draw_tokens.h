// Drawing a node's k tokens from the slab sums of its draft row, with the chunks that are searched read from
// memory: a wavefront per draw where the draws do not depend on each other, one for all where they do.
//
// Behind a row's slab sums a draft call is a chain of searches, and what it costs is the instructions of the waves that
// take part and the barriers between them: with every wave repeating every search and the owner of a drawn slab
// handing its result round, a CU's nodes all reached that chain at once and 3 to 4 us of the call went by in it.
// Now a draw is one wave's work, two draws run side by side, the waves without one are done, and the result crosses one
// barrier.  The price, a read of the searched slab (1 KiB, still in the caches), is the smaller.  us a call, 31-node
// trees, before -> after: bf16 rows of 32000, 64 trees SpecHub 18.4 -> 16.7, RRS 16.4 -> 14.7, RRSw 19.4 -> 15.8;
// of 8400, 400 trees 37.4 -> 32.7, 36.5 -> 27.2, 58.3 -> 34.0; one tree 5.9 -> 5.2, 4.9 -> 4.5, 6.2 -> 5.0; streamed
// rows of 128256, 64 trees 46.9 -> 43.6, 44.7 -> 41.2, 56.6 -> 43.1; fp32 probabilities of 32000, 480 nodes 13.0 -> 11.1.
#pragma once
#include "node_common.h"

namespace MDSD_NS {

// One inverse-CDF draw by one wavefront: W the slab sums' total.  weights_of(raw, s, w): this lane's weights
// of slab s, of which it holds the chunk `raw`.  Returns a virtual index, -1 without mass.
template <int DT, class SlabVal, class WeightsOf>
__device__ __forceinline__ int draw_one(const RowView& rq, SlabVal sv, float W, float u, WeightsOf weights_of)
{
    constexpr int E = Elem<DT>::kPerChunk;
    SlabHit h{0, 0.f, 0.f};
    const bool found = icdf_find_slab(rq.nslab, u, W, sv, h);
    const uint4 raw = fetch_chunk(rq, (found ? h.slab : 0) * 64 + (int)(threadIdx.x & 63));
    if (!found) return -1;
    float w[E];
    weights_of(raw, h.slab, w);
    return uniform(icdf_in_slab<E>(w, h));
}

// What a wavefront drew: lane i of the one that made draw i has `here` set and holds its token, -1 without mass.
struct Drawn {
    int token;
    bool here;
};

// The draws of a node, called by all of its wavefronts.  SpecHub makes two side by side: from the row, and from the row
// without the hub (the second token where the first draw gave the hub).  sh.slab_w: the slab sums of the row's
// weights cq, visible behind the barrier that this function begins with (RRSw takes drawn tokens out of them).  u: the
// node's k uniforms.  a_virt: SpecHub, the hub's virtual index.  Behind the caller's next barrier sh.bcast_f is the
// record's rest_mass (SpecHub: the mass outside the hub, otherwise the whole row's).
// A token that is removed changes its slab's sum only, which is formed again without it (never by subtraction).
// LEFT (RRSw): sh.bcast_left is then the mass outside all k drafted tokens.
template <int METHOD, int DT, bool LEFT = false, class CV>
__device__ __forceinline__ Drawn draw_tokens(const RowView& rq, CV cq, Shared& sh, const float* u, int k, int a_virt)
{
    constexpr int E = Elem<DT>::kPerChunk;
    static_assert(kWaves >= 2, "SpecHub's two draws take a wave each");
    const int lane = threadIdx.x & 63, wave = wave_id();
    auto sv = [&](int i) { return sh.slab_w[i]; };
    auto weights = [&](const uint4& raw, int s, float(&w)[E]) {
        float a[E];
        finish_chunk<DT>(rq, s * 64 + lane, raw, CV::fill(), a);
#pragma unroll
        for (int e = 0; e < E; ++e) w[e] = cq(a[e]);
    };
    uint4 hub_raw = make_uint4(0, 0, 0, 0);
    const int hub_slab = a_virt / (64 * E);
    if (METHOD == kSpecHub && wave == 1) hub_raw = fetch_chunk(rq, hub_slab * 64 + lane);
    node_barrier();
    Drawn out{-1, false};
    auto put = [&](int i, int v) {
        if (lane == i) out = Drawn{v < 0 ? -1 : v - rq.head, true};
    };
    if constexpr (METHOD == kSpecHub) {
        if (wave == 0) {
            put(0, draw_one<DT>(rq, sv, slab_total(rq.nslab, sv), u[0], weights));
        } else if (wave == 1) {
            // the mass outside the hub: its slab's sum without it
            float w[E];
            weights(hub_raw, hub_slab, w);
            zero_excluded<E>(w, hub_slab * 64 + lane, &a_virt, 1);
            const float without = wave_sum(chunk_sum<E>(w));
            auto sv_rest = [&](int i) { return i == hub_slab ? without : sh.slab_w[i]; };
            const float rest = slab_total(rq.nslab, sv_rest);
            if (lane == 0) sh.bcast_f = rest;
            put(1, draw_one<DT>(rq, sv_rest, rest, u[1], [&](const uint4& raw, int s, float(&ww)[E]) {
                weights(raw, s, ww);
                zero_excluded<E>(ww, s * 64 + lane, &a_virt, 1);
            }));
        }
    } else if constexpr (METHOD == kRRS) {
        if (wave < k) {
            const float W = slab_total(rq.nslab, sv);
            if (wave == 0 && lane == 0) sh.bcast_f = W;
            for (int i = wave; i < k; i += kWaves) put(i, draw_one<DT>(rq, sv, W, u[i], weights));
        }
    } else {
        if (wave != 0) return out;
        for (int i = 0; i < k; ++i) {
            const float W = slab_total(rq.nslab, sv);
            if (i == 0 && lane == 0) sh.bcast_f = W;
            int s_drawn = 0;
            float w[E];
            auto without = [&](int v) {
                const int off = v - (s_drawn * 64 + lane) * E;
#pragma unroll
                for (int e = 0; e < E; ++e) w[e] = e == off ? 0.f : w[e];
            };
            const int v = draw_one<DT>(rq, sv, W, u[i], [&](const uint4& raw, int s, float(&ww)[E]) {
                s_drawn = s;
                weights(raw, s, w);
                for (int j = 0; j < i; ++j) without(__builtin_amdgcn_readlane(out.token, j) + rq.head);
#pragma unroll
                for (int e = 0; e < E; ++e) ww[e] = w[e];
            });
            if (v >= 0 && (LEFT || i + 1 < k)) {  // nothing is drawn behind the last draw
                without(v);
                const float sum = wave_sum(chunk_sum<E>(w));
                // this wave's LDS instructions run in order; the compiler has to keep them so
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (lane == 0) sh.slab_w[s_drawn] = sum;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            put(i, v);
        }
        if constexpr (LEFT) {
            if (__builtin_amdgcn_readlane(out.token, 0) < 0) {  // no mass (or a NaN): token 0 is the draft, see token_of_draws()
                float w[E];
                weights(fetch_chunk(rq, lane), 0, w);
                const int token0 = rq.head;
                zero_excluded<E>(w, lane, &token0, 1);
                const float sum = wave_sum(chunk_sum<E>(w));
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (lane == 0) sh.slab_w[0] = sum;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            const float left = slab_total(rq.nslab, sv);
            if (lane == 0) sh.bcast_left = left;
        }
    }
    return out;
}

// Draft token number i that the draws in sh.node_x amount to, and the node's flags.  RRS, RRSw: a draw without mass
// repeats the token before it, the first gives token 0.
template <int METHOD>
__device__ __forceinline__ int token_of_draws(const Shared& sh, int k, int hub, int i, int& flags)
{
    if constexpr (METHOD == kSpecHub) {
        const int x = sh.node_x[0], y = sh.node_x[1];
        if (x != hub) return i == 0 ? x : hub;
        if (y < 0) flags |= MDSD_FLAG_DEGENERATE_HUB;
        return i == 0 || y < 0 ? hub : y;
    } else {
        int token = 0, mine = 0;
        for (int j = 0; j < k; ++j) {
            const int x = sh.node_x[j];
            if (x < 0) flags |= MDSD_FLAG_Q_EXHAUSTED;
            token = x < 0 ? token : x;
            mine = j == i ? token : mine;
        }
        return mine;
    }
}

}  // namespace MDSD_NS
