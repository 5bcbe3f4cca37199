// MoE routing tasks (paper Sec. 2.4): top-k routing and token grouping, the run-time resolution of a
// GroupGEMM row-tile slot, and the weighted combine of a token's expert outputs.
//
// Grouped rows.  The (token, slot) pairs of a step are sorted by (expert, token, slot); row p of the
// grouped tensors (expert activations, expert outputs) belongs to pair perm[p].  tok_indptr is the
// prefix sum of pairs per expert, exp_indptr the prefix sum of row tiles (tile_m rows each) per
// expert: expert e owns the row tiles [exp_indptr[e], exp_indptr[e+1]).  Everything is computed by
// counting and ranking, never by grabbing slots with atomics, so the permutation is the same in
// every run and under every schedule.
#pragma once
#include <type_traits>

#include "device_rt.hip.h"

namespace etc {

struct RowTile {
    int expert, row0, n;     // rows [row0, row0 + n) of the grouped tensors
    int shared;              // the expert has other row blocks
};
constexpr int kTileShared = 1 << 16;      // flag in tile_n

// Slot r of the static GroupGEMM grid -> its expert and rows; false for the surplus slots of this step, and for slots
// whose rows another slot of their expert has taken over (moel_scan).
__device__ __forceinline__ bool resolve_row_tile(const Params &P, int r, RowTile &rt)
{
    // One round trip: the entries of a slot beyond exp_indptr[E] are of an earlier step and not used.
    const int total_v = ld_i32(P.exp_indptr + P.E), expert_v = ld_i32(P.tile_expert + r), row0_v = ld_i32(P.tile_row0 + r),
              n_v = ld_i32(P.tile_n + r);
    const int total = __builtin_amdgcn_readfirstlane(total_v), n = __builtin_amdgcn_readfirstlane(n_v);
    rt.expert = __builtin_amdgcn_readfirstlane(expert_v);
    rt.row0 = __builtin_amdgcn_readfirstlane(row0_v);
    rt.n = n & (kTileShared - 1);
    rt.shared = n >= kTileShared;
    return r < total && rt.n > 0;
}

// ---- top-k of the router ---------------------------------------------------------------------------------
// Maximum / minimum over 16 consecutive lanes, the same value in all of them.
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v)
{
    v = max(v, (uint32_t)dpp_i32<0xB1>((int)v));
    v = max(v, (uint32_t)dpp_i32<0x4E>((int)v));
    v = max(v, (uint32_t)dpp_i32<0x141>((int)v));
    return max(v, (uint32_t)dpp_i32<0x140>((int)v));
}
__device__ __forceinline__ int row_min_i32(int v)
{
    v = min(v, dpp_i32<0xB1>(v));
    v = min(v, dpp_i32<0x4E>(v));
    v = min(v, dpp_i32<0x141>(v));
    return min(v, dpp_i32<0x140>(v));
}

// Top-k of 4 TG tokens by one wavefront, a token per row of 16 lanes, which share its experts out (lane l: l, l + 16, ..: NJ at
// most): token 4 u + row of the wavefront is row0 + u * step + row, valid below n_rows.  Lane k < K of the row gets the k-th expert
// and its logit; larger logit first, equal logits: lower expert first.  A round: the largest remaining ordered logit over
// registers and the row's lanes, then the lowest expert that holds it; four tokens to an instruction and no trip through scalar
// registers (a token per wavefront, 45 instructions and six scalar reads a round: 17 us for the 64 tokens of a block, 128 experts,
// now 6 with loads and stores).  seen(u, e, v): called with every logit.
template <int NJ, int TG, class SEEN>
__device__ __forceinline__ void rows_topk(const float *logits, int E, int K, int row0, int step, int n_rows, int (&id)[TG], float (&val)[TG],
                                          const SEEN &seen)
{
    const int l = lane_id() & 15, row = lane_id() >> 4;
    uint32_t key[TG][NJ];
    float v[TG][NJ];
#pragma unroll
    for (int u = 0; u < TG; ++u)           // no branch around a load: it would wait for the one before
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int b = row0 + u * step + row, e = l + 16 * j;
            v[u][j] = ld_f32(logits + (size_t)(b < n_rows ? b : n_rows - 1) * E + (e < E ? e : l));
        }
#pragma unroll
    for (int u = 0; u < TG; ++u) {
        const int b = row0 + u * step + row;
        id[u] = 0;
        val[u] = -INFINITY;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int e = l + 16 * j;
            const bool live = b < n_rows && e < E;
            if (live) seen(u, e, v[u][j]);
            const uint32_t bits = __float_as_uint(v[u][j]), ord = (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
            key[u][j] = live ? max(ord, 1u) : 0u;          // 0: taken, or no expert
        }
    }
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int u = 0; u < TG; ++u) {
            uint32_t mx = key[u][0];
#pragma unroll
            for (int j = 1; j < NJ; ++j) mx = max(mx, key[u][j]);
            mx = row_max_u32(mx);
            int e = 0x7FFFFFFF;
#pragma unroll
            for (int j = NJ - 1; j >= 0; --j) e = key[u][j] == mx ? l + 16 * j : e;
            e = row_min_i32(e);
            if (l == k) {
                id[u] = e;
                val[u] = __uint_as_float((mx & 0x80000000u) ? (mx & 0x7FFFFFFFu) : ~mx);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) key[u][j] = l + 16 * j == e ? 0u : key[u][j];
        }
    }
}
// Softmax over the first K lanes of each row of 16 (K <= 16).
__device__ __forceinline__ float row_softmax(float v, int K)
{
    const int l = lane_id() & 15;
    float mx = l < K ? v : -INFINITY;
    mx = fmaxf(mx, dpp_f32<0xB1>(mx));
    mx = fmaxf(mx, dpp_f32<0x4E>(mx));
    mx = fmaxf(mx, dpp_f32<0x141>(mx));
    mx = fmaxf(mx, dpp_f32<0x140>(mx));
    const float p = l < K ? __expf(v - mx) : 0.f;
    return p / lanes_sum<16>(p);
}

// Data-dependent event update and task triggering (Sec. 2.4), dynamic scheduler only.  The expert event
// tensor E_exp[e] is armed at run time with the number of tokens routed to e, plus one for tile 0, which
// publishes the per-expert tables: every tile knows that count from its own copy of the routing, so nobody
// has to write it first - a tile decrements, and the one that sees the count complete has fired the event
// (it puts the counter back to zero for the next layer).  The grouping tile of token t updates the events of
// topk[t, :]; when E_exp[e] fires, expert e releases its GroupGEMM-1 tiles, the row-tile slots
// [exp_indptr[e], exp_indptr[e+1]) of the static grid: their tasks are published to the ready queue, all
// fired experts of this tile under one reservation.  Slots beyond exp_indptr[E] are never released: tile 0
// takes them out of the counts that were fixed before the routing was known (the events between the two
// GroupGEMMs of those slots, the combine event, the number of tasks the step has to complete).
__device__ __forceinline__ void moe_update_and_trigger(const Params &P, int layer, int t, int group_ev,
                                                       const ETC_AS_LDS int32_t *ids_s, const ETC_AS_LDS int32_t *cnt,
                                                       const ETC_AS_LDS int32_t *expp)
{
    drain_vmem();            // this tile's share of the grouping (and tile 0's tables) is written
    __syncthreads();
    if (wave_id() != 0) return;
    const int lane = lane_id(), E = P.E, K = P.topk;
    const int G = P.moe_groups_gu, Gd = P.moe_groups_down;
    if (t == 0) {
        const int live = expp[E], dead = P.moe_rmax - live;
        const int ev_slot0 = gld_i32(P.moe_layer_events + 2 * layer), ev_y = gld_i32(P.moe_layer_events + 2 * layer + 1);
        for (int r = live + lane; r < P.moe_rmax; r += 64) st_i32(ev_counter(P, ev_slot0 + r), 0);
        ev_drop_producers(P, ev_y, live * Gd, P.moe_rmax * Gd);
        if (lane == 0 && dead > 0) {
            __hip_atomic_fetch_sub(as_global(P.ev_disp_cur + ((size_t)(ev_y & kEvIndex) << P.ev_shift)), dead * Gd, __ATOMIC_RELAXED, ETC_SCOPE);
            __hip_atomic_fetch_add(as_global(P.q_ctrl_cur + kQDone), dead * (G + Gd), __ATOMIC_RELAXED, ETC_SCOPE);
        }
        drain_vmem();        // the counts are in place before this tile's notifies can release anything
    }
    const int c0 = __builtin_amdgcn_readfirstlane(gld_i32(P.ev_consumers + group_ev));
    // Notify 0 of a lane: one pair of this token; notifies 1.. (tile 0 only): every routed expert, 64 per
    // round.  All decrements of the tile are in flight together, and what they release goes to the ready
    // queue under one reservation.
    constexpr int NV = 1 + kMaxExperts / 64;
    int ex[NV], first[NV], n_rel[NV];
    bool fired[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        ex[v] = -1;
        if (v == 0) {
            if (lane < K) ex[v] = ids_s[t * K + lane];
        } else if (t == 0) {
            const int cand = (v - 1) * 64 + lane;
            if (cand < E && cnt[cand] > 0) ex[v] = cand;
        }
    }
    int before[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v)
        before[v] = ex[v] >= 0 ? __hip_atomic_fetch_sub(as_global(P.exp_event + ex[v]), 1, __ATOMIC_RELAXED, ETC_SCOPE) : 0;
    int n_mine = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        fired[v] = ex[v] >= 0 && before[v] == -cnt[ex[v]];          // this was notify number cnt[e] + 1
        if (fired[v]) st_i32(P.exp_event + ex[v], 0);
        first[v] = fired[v] ? expp[ex[v]] * G : 0;
        n_rel[v] = fired[v] ? (expp[ex[v] + 1] - expp[ex[v]]) * G : 0;
        n_mine += n_rel[v];
    }
    drain_vmem();            // the fired counters are back at zero before the tasks they release are published:
                             // nothing released here can reach the next layer's router tiles ahead of the reset
    const int total = wave_sum_i(n_mine);
    if (total == 0) return;
    const int base = q_reserve_wave(P, total);
    if (base < 0) return;
    int off = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        uint64_t m = __ballot(fired[v]);
        while (m) {                                        // one fired expert after the other, 64 slots at a time
            const int src = __builtin_ctzll(m);
            m &= m - 1;
            const int s0 = __shfl(first[v], src, 64), n = __shfl(n_rel[v], src, 64);
            for (int i = lane; i < n; i += 64)
                __hip_atomic_store(as_global(P.q_slots + base + off + i),
                                   q_slot_word(P, gld_i32(P.consumer_ids + c0 + s0 + i) & 0xFFFFFF), __ATOMIC_RELAXED, ETC_SCOPE);
            off += n;
        }
    }
}

// Router tile of token t.  Every tile needs the ids of ALL tokens to rank its own pairs, so each
// recomputes the (cheap) top-k of every token from the shared logits instead of waiting one more event
// hop for them; it publishes only what belongs to token t.  Tile 0 also publishes the per-expert tables.
// Order of the selection: larger logit first, equal logits -> lower expert index first.
// Routing weights: softmax over the selected logits.
// group_ev: the event the tile notifies; under the dynamic scheduler its consumer list (the GroupGEMM-1
// tasks of the layer, row-tile slot major) is what the expert events trigger from.
__device__ __noinline__ void moe_route_and_group(const Params &P, int layer, int t, int group_ev, float *sm)
{
    layer = __builtin_amdgcn_readfirstlane(layer);
    t = __builtin_amdgcn_readfirstlane(t);
    group_ev = notify_event(__builtin_amdgcn_readfirstlane(group_ev));
    const int wave = wave_id(), lane = lane_id();
    const int E = P.E, K = P.topk, B = P.B, N = B * K, M = P.tile_m;
    ETC_AS_LDS int32_t *ids_s = reinterpret_cast<ETC_AS_LDS int32_t *>(as_lds(sm));   // [B*K] expert of every pair
    ETC_AS_LDS int32_t *cnt = ids_s + kMaxBatch * kMaxTopK;                            // [E]
    ETC_AS_LDS int32_t *tokp = cnt + kMaxExperts;                                      // [E+1]
    ETC_AS_LDS int32_t *expp = tokp + kMaxExperts + 1;                                 // [E+1]
    const int forced_bits = P.forced_mask != nullptr ? (int)*as_global(P.forced_mask + layer) : 0;
    const bool forced = (forced_bits & 1) != 0, forced_w = forced && (forced_bits & 2) != 0 && P.forced_w != nullptr;
    const bool dbg = (P.debug_flags & 4u) != 0 && P.dbg_logits != nullptr;
    const size_t dbg_row = (size_t)layer * P.max_batch + t;

    for (int e = threadIdx.x; e < E; e += kWgThreads) cnt[e] = 0;
    auto route = [&](auto per_lane, auto groups) {
        constexpr int NJ = decltype(per_lane)::value, TG = decltype(groups)::value;
        const int l = lane & 15;
        for (int b0 = wave * 4; b0 < B; b0 += TG * 4 * kWaves) {
            int id[TG];
            float val[TG];
            rows_topk<NJ, TG>(P.router_logits, E, forced ? 0 : K, b0, 4 * kWaves, B, id, val, [&](int u, int e, float v) {
                if (dbg && b0 + u * 4 * kWaves + (lane >> 4) == t) as_global(P.dbg_logits)[dbg_row * E + e] = v;
            });
#pragma unroll
            for (int u = 0; u < TG; ++u) {
                const int b = b0 + u * 4 * kWaves + (lane >> 4);
                int my_id = id[u];
                float my_v = val[u];
                if (forced && b < B && l < K) {
                    my_id = gld_i32(P.forced_topk + ((size_t)layer * P.max_batch + b) * K + l);
                    my_v = ld_f32(P.router_logits + (size_t)b * E + my_id);
                }
                float wgt = row_softmax(my_v, K);
                if (b < B && l < K) {
                    ids_s[b * K + l] = my_id;
                    if (b == t) {
                        if (forced_w) wgt = *as_global(P.forced_w + ((size_t)layer * P.max_batch + b) * K + l);
                        st_i32(P.topk_ids + (size_t)t * K + l, my_id);
                        st_f32(P.topk_w + (size_t)t * K + l, wgt);
                        if (dbg) {
                            as_global(P.dbg_topk_ids)[dbg_row * K + l] = my_id;
                            as_global(P.dbg_topk_w)[dbg_row * K + l] = wgt;
                        }
                    }
                }
            }
        }
    };
    if (E <= 128) {
        if (B <= 4 * kWaves) route(std::integral_constant<int, 8>(), std::integral_constant<int, 1>());
        else route(std::integral_constant<int, 8>(), std::integral_constant<int, 2>());
    } else route(std::integral_constant<int, 16>(), std::integral_constant<int, 1>());
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += kWgThreads)
        __hip_atomic_fetch_add(cnt + ids_s[i], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    // Exclusive sums of pairs (low half) and row tiles (high half) over the experts, by one wavefront, four experts a lane: at most
    // 1024 of each.  (A loop over the experts before its own in every thread took 3.5 us longer a layer, 128 experts.)
    if (wave == 0) {
        static_assert(kMaxExperts == 4 * 64 && kMaxBatch * kMaxTopK < (1 << 15), "four experts a lane, 16-bit sums");
        const uint32_t inv = (65536u + (uint32_t)M - 1u) / (uint32_t)M;      // n * inv >> 16 == n / M for n < 65536 / M
        uint32_t own[4], mine = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t c = 4 * lane + j < E ? (uint32_t)cnt[4 * lane + j] : 0u;
            own[j] = c | (((c + (uint32_t)M - 1u) * inv) >> 16) << 16;
            mine += own[j];
        }
        uint32_t incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)incl, off, 64);
            if (lane >= off) incl += o;
        }
        uint32_t at = incl - mine;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = 4 * lane + j;
            if (e < E) { tokp[e] = (int)(at & 0xFFFFu); expp[e] = (int)(at >> 16); }
            at += own[j];
            if (e == E - 1) { tokp[E] = (int)(at & 0xFFFFu); expp[E] = (int)(at >> 16); }
        }
    }
    __syncthreads();

    // the K pairs of this token: stable rank among the pairs of the same expert
    for (int k = wave; k < K; k += kWaves) {
        const int me = t * K + k, e = ids_s[me];
        int c = 0;
        for (int i = lane; i < me; i += 64) c += ids_s[i] == e ? 1 : 0;
        c = wave_sum_i(c);
        if (lane == 0) {
            const int pos = tokp[e] + c;
            st_i32(P.perm + pos, me);
            st_i32(P.inv_perm + me, pos);
            st_i32(P.perm_tok + pos, t);
            if (dbg) as_global(P.dbg_perm)[(size_t)layer * P.max_batch * K + pos] = me;
        }
    }
    if (t == 0) {
        for (int e = threadIdx.x; e <= E; e += kWgThreads) {
            st_i32(P.tok_indptr + e, tokp[e]);
            st_i32(P.exp_indptr + e, expp[e]);
            if (dbg) {
                as_global(P.dbg_tok_indptr)[(size_t)layer * (E + 1) + e] = tokp[e];
                as_global(P.dbg_exp_indptr)[(size_t)layer * (E + 1) + e] = expp[e];
            }
        }
        for (int e = threadIdx.x; e < E; e += kWgThreads) {
            int n = cnt[e], r = expp[e], row = tokp[e];
            for (; n > 0; n -= M, ++r, row += M) {
                st_i32(P.tile_expert + r, e);
                st_i32(P.tile_row0 + r, row);
                st_i32(P.tile_n + r, n < M ? n : M);
            }
        }
    }
    if (P.moe_dd) moe_update_and_trigger(P, layer, t, group_ev, ids_s, cnt, expp);
    __syncthreads();     // the routing scratch in LDS is free again
}

// ---------------------------------------------------------------------------------------------------------
// The MoE layer on its own over a block of T tokens (Sec. 2.4; the token sweep of Sec. 4.2 / 4.5).
// One router tile per token that ranks its pairs against every other token is quadratic in the tokens, so the
// grouping runs as three counting passes over blocks of 64 tokens: (1) top-k of the block's tokens and the
// block's pair count per expert; (2) one scan over experts and blocks: totals, prefix sums, the first grouped row
// of every (block, expert) and the row-tile tables; (3) the stable rank of every pair inside its block.  The
// grouped order is the decoder's: (expert, token, slot).  Still no slot is grabbed with an atomic: the
// permutation is the same in every run and schedule.
// ---------------------------------------------------------------------------------------------------------
constexpr int kMoelBlock = 64;


// 16 tokens: (x_in * gain) split into hi + lo, the row's sum of squares.  A wavefront takes two tokens at a time, a lane 8
// consecutive elements of each per step (16-byte loads and stores), four steps in flight: one round trip for a hidden size
// of 2048.  The residual is kept as it came (bf16): y may overlap x_in, and the combine tasks read it when y is written.
__device__ __noinline__ void moel_load(const Params &P, int blk16)
{
    blk16 = __builtin_amdgcn_readfirstlane(blk16);
    const uint16_t *g2 = (const uint16_t *)as_global(P.weights)[0].g2;
    const int n_oct = P.H / 8, wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int tok0 = blk16 * 16 + 2 * wave;
    if (tok0 >= P.B) return;
    const bool two = tok0 + 1 < P.B;
    const size_t row[2] = {(size_t)tok0 * P.H, (size_t)(two ? tok0 + 1 : tok0) * P.H};
    float total[2] = {0.f, 0.f};
    constexpr int U = 4;
    for (int o0 = lane; o0 - lane < n_oct; o0 += U * 64) {
        u32x4 xa[2][U], ga[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int oct = o0 + u * 64 < n_oct ? o0 + u * 64 : 0;
            ga[u] = gld_16B(g2 + oct * 8);
#pragma unroll
            for (int t = 0; t < 2; ++t) xa[t][u] = gld_16B(P.hidden_in + row[t] + (size_t)oct * 8);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = o0 + u * 64 < n_oct;
            const uint32_t gw[4] = {ga[u].x, ga[u].y, ga[u].z, ga[u].w};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t xw[4] = {xa[t][u].x, xa[t][u].y, xa[t][u].z, xa[t][u].w};
                uint32_t hw[4], lw[4];
                float s = 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v0 = bf16_bits_to_f32(xw[q] & 0xFFFFu), v1 = bf16_bits_to_f32(xw[q] >> 16);
                    uint16_t h0, l0, h1, l1;
                    split_bf16(v0 * bf16_bits_to_f32(gw[q] & 0xFFFFu), h0, l0);
                    split_bf16(v1 * bf16_bits_to_f32(gw[q] >> 16), h1, l1);
                    hw[q] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                    lw[q] = (uint32_t)l0 | ((uint32_t)l1 << 16);
                    s += v0 * v0 + v1 * v1;
                }
                if (live) {
                    total[t] += s;
                    const uint32_t at = (uint32_t)(o0 + u * 64) * 16u;
                    buf_st_16B(buf_of(P.x_copy + row[t]), at, xa[t][u]);
                    buf_st_16B(buf_of(P.xmg_hi + row[t]), at, u32x4{hw[0], hw[1], hw[2], hw[3]});
                    buf_st_16B(buf_of(P.xmg_lo + row[t]), at, u32x4{lw[0], lw[1], lw[2], lw[3]});
                }
            }
        }
    }
    // the whole row's sum of squares: one part per token (a consumer that gathers its columns would otherwise fetch
    // hidden / 16 scattered words for each of them)
    total[0] = wave_sum(total[0]);
    total[1] = wave_sum(total[1]);
    if (lane == 0) {
        st_f32(P.ssq_xmid + tok0, total[0]);
        if (two) st_f32(P.ssq_xmid + tok0 + 1, total[1]);
    }
}

// Block of 64 tokens: top-k ids (larger logit first, equal logits: lower expert first) and routing weights
// (softmax over the selected logits) of each token; the block's pair count per expert.
__device__ __noinline__ void moel_topk(const Params &P, int blk, float *sm)
{
    blk = __builtin_amdgcn_readfirstlane(blk);
    const int wave = wave_id(), lane = lane_id();
    const int E = P.E, K = P.topk;
    ETC_AS_LDS int32_t *cnt = reinterpret_cast<ETC_AS_LDS int32_t *>(as_lds(sm));      // [E]
    const int forced_bits = P.forced_mask != nullptr ? (int)*as_global(P.forced_mask) : 0;
    const bool forced = (forced_bits & 1) != 0, forced_w = forced && (forced_bits & 2) != 0 && P.forced_w != nullptr;
    const bool dbg = (P.debug_flags & 4u) != 0 && P.dbg_logits != nullptr;
    for (int e = threadIdx.x; e < E; e += kWgThreads) cnt[e] = 0;
    __syncthreads();
    const int n_here = min(kMoelBlock, P.B - blk * kMoelBlock);      // <= 0: a block beyond the bound tokens
    auto route = [&](auto per_lane, auto groups) {
        constexpr int NJ = decltype(per_lane)::value, TG = decltype(groups)::value;
        const int l = lane & 15, t0 = blk * kMoelBlock;
        for (int i0 = wave * 4; i0 < n_here; i0 += TG * 4 * kWaves) {
            int id[TG];
            float val[TG];
            rows_topk<NJ, TG>(P.router_logits, E, forced ? 0 : K, t0 + i0, 4 * kWaves, P.B, id, val, [&](int u, int e, float v) {
                if (dbg) as_global(P.dbg_logits)[(size_t)(t0 + i0 + u * 4 * kWaves + (lane >> 4)) * E + e] = v;
            });
#pragma unroll
            for (int u = 0; u < TG; ++u) {
                const int i = i0 + u * 4 * kWaves + (lane >> 4), b = t0 + i;
                const bool live = i < n_here && l < K;
                int my_id = id[u];
                float my_v = val[u];
                if (forced && live) {
                    my_id = gld_i32(P.forced_topk + (size_t)b * K + l);
                    my_v = ld_f32(P.router_logits + (size_t)b * E + my_id);
                }
                float wgt = row_softmax(my_v, K);
                if (live) {
                    if (forced_w) wgt = *as_global(P.forced_w + (size_t)b * K + l);
                    st_i32(P.topk_ids + (size_t)b * K + l, my_id);
                    st_f32(P.topk_w + (size_t)b * K + l, wgt);
                    if (dbg) {
                        as_global(P.dbg_topk_ids)[(size_t)b * K + l] = my_id;
                        as_global(P.dbg_topk_w)[(size_t)b * K + l] = wgt;
                    }
                    __hip_atomic_fetch_add(cnt + my_id, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);      // integer count: order-free
                }
            }
        }
    };
    if (E <= 128) {
        if (n_here <= 4 * kWaves) route(std::integral_constant<int, 8>(), std::integral_constant<int, 1>());
        else route(std::integral_constant<int, 8>(), std::integral_constant<int, 2>());
    } else route(std::integral_constant<int, 16>(), std::integral_constant<int, 1>());
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kWgThreads) st_i32(P.moel_hist + (size_t)blk * E + e, cnt[e]);
    __syncthreads();
}

// One task: pairs per expert, prefix sums over the experts (pairs and row tiles), the first grouped row of every
// (block, expert), the row-tile tables.  Under the dynamic scheduler it also takes the surplus row-tile slots of the
// static grids out of the counts that were fixed before the routing was known (as tile 0 does in a decoder).
// Alone on the critical path, bound by its round trips: all threads count (two or four to an expert, 16 loads each in flight; the
// counts stay in registers for the second use), and the prefix sums are a wavefront's each.
__device__ __noinline__ void moel_scan(const Params &P, float *sm)
{
    const int E = P.E, M = P.tile_m, n_blk = (P.B + kMoelBlock - 1) / kMoelBlock;
    constexpr int kRow = kMaxExperts + 1, kClasses = 4;
    ETC_AS_LDS int32_t *shares = reinterpret_cast<ETC_AS_LDS int32_t *>(as_lds(sm));   // [parts][EW] pairs of a part's token blocks
    ETC_AS_LDS int32_t *tokp = shares + kWgThreads;                                    // [E+1] pairs; row tiles; row blocks of each class
    ETC_AS_LDS int32_t *expp = tokp + kRow, *clsp = expp + kRow;                       //   (then their exclusive sums, the total last)
    // A GroupGEMM task takes a row BLOCK of up to row_merge row tiles of one expert: the weights are streamed once for all its columns.
    // Static grids: the blocks fill the first slots, the longest first (by what they cost: more than 64, 32, 16 columns and the
    // others), so that what a queue gets last is short; the other slots are left without rows.  Where the grid is by XCD
    // (moe_slots_by_xcd) and enough slots are left over, neighbours in that order go in pairs to every eighth slot: the tasks of a
    // slot go to the workgroups of one XCD (first_dim_by_xcd).
    // Qwen3-30B-A3B layer of 2000 / 4001 tokens: 670 / 1160 us with the blocks in the experts' order and everywhere, 635 / 1162 by XCD, 630 / 1117 now.
    // Dynamic scheduler: an expert's tasks are released as the slots of its row tiles, so its blocks take the first of them.
    const int MB = M * P.row_merge;
    auto class_of = [](int n) { return n > 64 ? 0 : (n > 32 ? 1 : (n > 16 ? 2 : 3)); };
    const bool dbg = (P.debug_flags & 4u) != 0 && P.dbg_logits != nullptr;
    const int EW = E <= 128 ? 128 : 256, parts = kWgThreads / EW, part = (int)threadIdx.x / EW, e = (int)threadIdx.x % EW;
    const int per = (n_blk + parts - 1) / parts, b_first = part * per, b_end = min(n_blk, b_first + per);
    int h[16], own = 0;
    auto load_counts = [&](int b0) {
#pragma unroll
        for (int u = 0; u < 16; ++u) h[u] = e < E && b0 + u < b_end ? ld_i32(P.moel_hist + (size_t)(b0 + u) * E + e) : 0;
    };
    for (int b0 = b_first; b0 < b_end; b0 += 16) {
        load_counts(b0);
#pragma unroll
        for (int u = 0; u < 16; ++u) own += h[u];
    }
    shares[threadIdx.x] = own;
    __syncthreads();
    int n = 0, before = 0;                                 // pairs of the expert; those of the token blocks of the parts before this one
    if (e < E)
        for (int p = 0; p < parts; ++p) {
            const int c = shares[p * EW + e];
            n += c;
            before += p < part ? c : 0;
        }
    const int full = n / MB, rest = n % MB;                // row blocks
    if (part == 0 && e < E) {
        tokp[e] = n;
        expp[e] = (n + M - 1) / M;
#pragma unroll
        for (int c = 0; c < kClasses; ++c) clsp[c * kRow + e] = (c == class_of(MB) ? full : 0) + (rest > 0 && c == class_of(rest) ? 1 : 0);
    }
    __syncthreads();
    if (wave_id() < 2 + kClasses) {                        // exclusive sums of one quantity, four experts a lane
        static_assert(kMaxExperts == 4 * 64 && 2 + kClasses <= kWaves, "four experts a lane, a wavefront for each quantity");
        ETC_AS_LDS int32_t *q = tokp + wave_id() * kRow;
        const int lane = lane_id();
        int own4[4], mine = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            own4[j] = 4 * lane + j < E ? q[4 * lane + j] : 0;
            mine += own4[j];
        }
        int incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        int at = incl - mine;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (4 * lane + j < E) q[4 * lane + j] = at;
            at += own4[j];
            if (4 * lane + j == E - 1) q[E] = at;
        }
    }
    __syncthreads();
    int class0[kClasses], n_blocks = 0;                    // first block of each class
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
        class0[c] = n_blocks;
        n_blocks += clsp[c * kRow + E];
    }
    const int n_tiles = expp[E];
    const bool by_xcd = P.slots_by_xcd != 0 && (n_blocks + 2 * kXcds - 1) / (2 * kXcds) * (2 * kXcds) <= n_tiles;
    if (!P.moe_dd)
        for (int r = threadIdx.x; r < n_tiles; r += kWgThreads) {
            const int depth = r / kXcds, q = by_xcd ? 2 * (depth / 2 * kXcds + r % kXcds) + depth % 2 : r;
            if (q >= n_blocks) st_i32(P.tile_n + r, 0);
        }
    if (e < E) {
        int row = tokp[e] + before;
        for (int b0 = b_first; b0 < b_end; b0 += 16) {
            if (per > 16) load_counts(b0);
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if (b0 + u < b_end) st_i32(P.moel_base + (size_t)(b0 + u) * E + e, row);
                row += h[u];
            }
        }
    }
    if (part == 0 && e < E) {
        st_i32(P.moel_count + e, n);
        const int c_full = class_of(MB), c_rest = class_of(rest);
        for (int j = 0; j * MB < n; ++j) {
            const bool whole = j < full;
            int c_first = 0, c_before = 0;
#pragma unroll
            for (int c = 0; c < kClasses; ++c)
                if (c == (whole ? c_full : c_rest)) { c_first = class0[c]; c_before = clsp[c * kRow + e]; }
            const int q = c_first + c_before + (whole ? j : (c_rest == c_full ? full : 0));
            const int slot = P.moe_dd ? expp[e] + j : (by_xcd ? (q / 2 / kXcds * 2 + q % 2) * kXcds + q / 2 % kXcds : q);
            st_i32(P.tile_expert + slot, e);
            st_i32(P.tile_row0 + slot, tokp[e] + j * MB);
            st_i32(P.tile_n + slot, (whole ? MB : rest) | (n > MB ? kTileShared : 0));
        }
        if (P.moe_dd)
            for (int r = expp[e] + (n + MB - 1) / MB; r < expp[e + 1]; ++r) st_i32(P.tile_n + r, 0);
    }
    for (int i = threadIdx.x; i <= E; i += kWgThreads) {
        st_i32(P.tok_indptr + i, tokp[i]);
        st_i32(P.exp_indptr + i, expp[i]);
        if (dbg) {
            as_global(P.dbg_tok_indptr)[i] = tokp[i];
            as_global(P.dbg_exp_indptr)[i] = expp[i];
        }
    }
    if (P.moe_dd && wave_id() == 0) {
        const int lane = lane_id(), G = P.moe_groups_gu, Gd = P.moe_groups_down;
        const int live = expp[E], dead = P.moe_rmax - live;
        const int ev_slot0 = gld_i32(P.moe_layer_events), ev_y = gld_i32(P.moe_layer_events + 1);
        for (int r = live + lane; r < P.moe_rmax; r += 64) st_i32(ev_counter(P, ev_slot0 + r), 0);
        ev_drop_producers(P, ev_y, live * Gd, P.moe_rmax * Gd);
        if (lane == 0 && dead > 0) {
            __hip_atomic_fetch_sub(as_global(P.ev_disp_cur + ((size_t)(ev_y & kEvIndex) << P.ev_shift)), dead * Gd, __ATOMIC_RELAXED, ETC_SCOPE);
            __hip_atomic_fetch_add(as_global(P.q_ctrl_cur + kQDone), dead * (G + Gd), __ATOMIC_RELAXED, ETC_SCOPE);
        }
    }
    __syncthreads();
}

// Data-dependent event update and task triggering (Sec. 2.4) of the stand-alone layer, dynamic scheduler only: the
// block adds its pair count of every expert to the expert's event at once; the total per expert is known since the
// scan, so the update that completes it has fired the event and releases the expert's GroupGEMM-1 tiles, the
// row-tile slots [exp_indptr[e], exp_indptr[e+1]), to the ready queue.
__device__ __forceinline__ void moel_update_and_trigger(const Params &P, int blk, int group_ev)
{
    drain_vmem();            // this block's share of the permutation is written
    __syncthreads();
    if (wave_id() != 0) return;
    const int lane = lane_id(), E = P.E, G = P.moe_groups_gu;
    const int c0 = __builtin_amdgcn_readfirstlane(gld_i32(P.ev_consumers + group_ev));
    for (int e0 = 0; e0 < E; e0 += 64) {
        const int e = e0 + lane;
        const int h = e < E ? ld_i32(P.moel_hist + (size_t)blk * E + e) : 0;
        const int before = h > 0 ? __hip_atomic_fetch_sub(as_global(P.exp_event + e), h, __ATOMIC_RELAXED, ETC_SCOPE) : 0;
        const bool fired = h > 0 && before - h == -ld_i32(P.moel_count + e);
        int first = 0, n_rel = 0;
        if (fired) {
            st_i32(P.exp_event + e, 0);
            const int r0 = ld_i32(P.exp_indptr + e), r1 = ld_i32(P.exp_indptr + e + 1);
            first = r0 * G;
            n_rel = (r1 - r0) * G;
        }
        drain_vmem();        // the fired counters are back at zero before the tasks they release are published
        const int total = wave_sum_i(n_rel);
        if (total == 0) continue;
        const int base = q_reserve_wave(P, total);
        if (base < 0) return;
        int off = 0;
        uint64_t m = __ballot(fired);
        while (m) {
            const int src = __builtin_ctzll(m);
            m &= m - 1;
            const int s0 = __shfl(first, src, 64), n = __shfl(n_rel, src, 64);
            for (int i = lane; i < n; i += 64)
                __hip_atomic_store(as_global(P.q_slots + base + off + i),
                                   q_slot_word(P, gld_i32(P.consumer_ids + c0 + s0 + i) & 0xFFFFFF), __ATOMIC_RELAXED, ETC_SCOPE);
            off += n;
        }
    }
}

// Block of 64 tokens: every pair's grouped row = first row of (block, expert) + its rank among the block's earlier
// pairs of the same expert (pairs in token, slot order).
__device__ __noinline__ void moel_place(const Params &P, int blk, int group_ev, float *sm)
{
    blk = __builtin_amdgcn_readfirstlane(blk);
    group_ev = notify_event(__builtin_amdgcn_readfirstlane(group_ev));
    const int E = P.E, K = P.topk;
    const int n_tok = P.B - blk * kMoelBlock < kMoelBlock ? P.B - blk * kMoelBlock : kMoelBlock;
    ETC_AS_LDS int32_t *ids_s = reinterpret_cast<ETC_AS_LDS int32_t *>(as_lds(sm));    // [64 * K]
    ETC_AS_LDS int32_t *base_s = ids_s + kMoelBlock * kMaxTopK;                        // [E]
    ETC_AS_LDS int32_t *grp = base_s + kMaxExperts;                                    // [groups of 64 pairs][kMaxExperts] pairs per expert
    static_assert(kMaxExperts == 256 && kMoelBlock * kMaxTopK == 16 * 64, "eight bits of an expert, 16 groups");
    const bool dbg = (P.debug_flags & 4u) != 0 && P.dbg_logits != nullptr;
    if (n_tok > 0) {
        const int n_pairs = n_tok * K, pair0 = blk * kMoelBlock * K;
        for (int p = threadIdx.x; p < n_pairs; p += kWgThreads) ids_s[p] = ld_i32(P.topk_ids + pair0 + p);
        for (int e = threadIdx.x; e < E; e += kWgThreads) base_s[e] = ld_i32(P.moel_base + (size_t)blk * E + e);
        for (int i = threadIdx.x; i < (n_pairs + 63) / 64 * kMaxExperts; i += kWgThreads) grp[i] = 0;
        __syncthreads();
        // Rank among the block's earlier pairs of the same expert: the pairs are taken 64 to a wavefront, at most 16 such groups; a
        // group counts its pairs per expert, and a pair adds the counts of the groups before its own and the lower lanes of its
        // group that share its expert (found by eight ballots over the expert's bits).
        const int n_groups = (n_pairs + 63) / 64;
        for (int g = wave_id(); g < n_groups; g += kWaves) {
            const int p = g * 64 + lane_id();
            if (p < n_pairs) __hip_atomic_fetch_add(grp + g * kMaxExperts + ids_s[p], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        for (int g = wave_id(); g < n_groups; g += kWaves) {
            const int p = g * 64 + lane_id();
            const bool live = p < n_pairs;
            const int e = live ? ids_s[p] : 0;
            uint64_t same = __ballot(live);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const uint64_t with = __ballot((e >> bit) & 1);
                same &= (e >> bit) & 1 ? with : ~with;
            }
            int rank = __popcll(same & ((1ull << lane_id()) - 1ull));
            for (int q = 0; q < g; ++q) rank += grp[q * kMaxExperts + e];
            if (!live) continue;
            const int pos = base_s[e] + rank, pair = pair0 + p;
            st_i32(P.perm + pos, pair);
            st_i32(P.inv_perm + pair, pos);
            st_i32(P.perm_tok + pos, pair / K);
            if (dbg) as_global(P.dbg_perm)[pos] = pair;
        }
    }
    if (P.moe_dd) moel_update_and_trigger(P, blk, group_ev);
    __syncthreads();
}

// Combine tile (token b, 512 consecutive elements): x = x_mid + sum_k w[b,k] * y[row of pair (b,k)],
// slots in ascending order.  Like every producer of the residual stream it also prepares the next
// layer's projection operand (x * gain, split) and the partial sums of squares per 16 elements.
__device__ __forceinline__ void moe_combine(const Params &P, const Task &t)
{
    const int b = t.c0, h = t.c1 * kWgThreads + (int)threadIdx.x;
    if (h >= P.H) return;
    const int K = P.topk;
    float acc = 0.f;
    const size_t o = (size_t)b * P.H + h;
    const float x0 = ld_f32(P.x_mid + o);
    constexpr int SL = 8;
    for (int k0 = 0; k0 < K; k0 += SL) {               // the look-ups of 8 slots in one round trip, their rows in the next
        int pos[SL];
        float wk[SL], y[SL];
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            const size_t p = (size_t)b * K + (k0 + k < K ? k0 + k : K - 1);
            pos[k] = ld_i32(P.inv_perm + p);
            wk[k] = ld_f32(P.topk_w + p);
        }
#pragma unroll
        for (int k = 0; k < SL; ++k) y[k] = ld_f32(P.ey + (size_t)pos[k] * P.H + h);
#pragma unroll
        for (int k = 0; k < SL; ++k)
            if (k0 + k < K) acc += wk[k] * y[k];
    }
    const float v = x0 + acc;
    st_f32(P.x + o, v);
    const bool last = (t.flags & TF_LAST_LAYER) != 0;
    if (last && P.hidden_out) gst_u16(P.hidden_out + o, f32_to_bf16_bits(v));
    if (!last || P.vocab > 0) {       // operand of the next projection: the next layer's QKV, or the vocabulary projection
        const uint16_t *g1 = last ? P.gf : (const uint16_t *)as_global(P.weights)[t.layer + 1].g1;
        uint16_t hi, lo;
        split_bf16(v * bf16_bits_to_f32(gld_u16(g1 + h)), hi, lo);
        st_u16(P.xg_hi + o, hi);
        st_u16(P.xg_lo + o, lo);
        float s = v * v;          // 16 consecutive lanes hold one 16-element part
        s = lanes_sum<16>(s);
        if ((threadIdx.x & 15) == 0) st_f32(P.ssq_x + (size_t)(h >> 4) * kMaxBatch + b, s);
    }
    if (P.debug_flags & 2u) gst_f32(P.layer_hidden + ((size_t)t.layer * kMaxBatch + b) * P.H + h, v);
}

// Combine of the stand-alone layer: task (block of `n_tok` tokens starting at tok0, 2048 consecutive elements).  One
// task per token and 512 elements would be 16 384 tasks of two dependent load rounds each at 4096 tokens (415 us for
// 320 MB); here a thread takes 4 consecutive elements (16-byte loads) of a token, with the rows of up to 8 slots in
// flight together.  The layer's output is y; no fp32 residual is kept.
__device__ __forceinline__ void moel_combine(const Params &P, int tok0, int n_tok, int chunk)
{
    const int h = (chunk * kWgThreads + (int)threadIdx.x) * 4;
    if (h >= P.H) return;
    const int K = P.topk;
    const int end = tok0 + n_tok < P.B ? tok0 + n_tok : P.B;
    constexpr int SL = 8;
    for (int b = tok0; b < end; ++b) {
        const uint64_t xw = ld_u64(P.x_copy + (size_t)b * P.H + h);
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < K; k0 += SL) {             // slots in ascending order
            int pos[SL];
            float wk[SL];
            u32x4 y[SL];
#pragma unroll
            for (int k = 0; k < SL; ++k) {               // slots beyond K read the last one, weight 0, and are not added
                const size_t p = (size_t)b * K + (k0 + k < K ? k0 + k : K - 1);
                pos[k] = ld_i32(P.inv_perm + p);
                wk[k] = ld_f32(P.topk_w + p);
            }
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const int row = __builtin_amdgcn_readfirstlane(pos[k]);
                y[k] = buf_ld_16B(buf_of(P.ey + (size_t)row * P.H), (uint32_t)h * 4u, 0);
            }
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                if (k0 + k < K) {                        // uniform
                    sum[0] += wk[k] * __uint_as_float(y[k].x);
                    sum[1] += wk[k] * __uint_as_float(y[k].y);
                    sum[2] += wk[k] * __uint_as_float(y[k].z);
                    sum[3] += wk[k] * __uint_as_float(y[k].w);
                }
            }
        }
        if (P.hidden_out) {
            uint64_t v = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float x = bf16_bits_to_f32((uint32_t)(xw >> (16 * q)) & 0xFFFFu);
                v |= (uint64_t)f32_to_bf16_bits(x + sum[q]) << (16 * q);
            }
            *as_global(reinterpret_cast<uint64_t *>(P.hidden_out + (size_t)b * P.H + h)) = v;
        }
    }
}

}  // namespace etc
