// Paged decode attention (split-KV):
//   attn_chunk  (sequence b, kv head, chunk): online-softmax partial (m, l, o) of the group's query
//               heads over the chunk's keys, K/V rows gathered through the page table;
//               the chunk that arrives last at its (sequence, kv head) combines the partials in ascending order.
// Scores and maxima are kept times log2(e), so that every exponential is one exp2.
// Cached K/V rows are read-only during the launch (ordinary loads).  The row appended by this step is
// not read back from the cache (where it is bf16) but taken in fp32 from the projection's scratch copy,
// so the new token enters its own attention unrounded; that copy, the queries and the partials cross
// tasks and are accessed with device-scope loads / stores.
#pragma once
#include <type_traits>

#include "device_rt.hip.h"

namespace etc {

// Per-wavefront partial results of a chunk in LDS: kWaves entries, and one more for the step's own token:
// [entry][g] m, l, then [entry][g][D] o.
constexpr int kAttnEnt = kWaves + 1;
template <int GRP> constexpr int kAttnOff = (2 * kAttnEnt * GRP + 3) & ~3;      // floats in front of the o rows (which are read 16 bytes at a time)
constexpr int kAttnScratch = 40 * 1024;             // bytes in front of the wavefronts' V tiles (behind those: kAttnPages page ids)

__device__ __forceinline__ float exp2_f(float x) { return __builtin_amdgcn_exp2f(x); }

template <int D, int GRP> __device__ __forceinline__ void attn_merge_chunks(const Params &P, int b, int kvh, int nc);

// Keys per chunk of sequence b, and the chunk a slot of the attention grid stands for.  The grid has max_slots slots per
// KV head; a step of P.B sequences gives each max_slots / P.B of them and splits it evenly, in whole pages and not finer than
// the caller's chunk: the slots of one sequence are equally long, and a batch below the sampled one uses all of them.  With
// chunks of a fixed number of keys (the longest sequence cut into the sampled batch's slots) a sequence of 1.5 chunks left
// half of its second slot idle, and a batch of 5 in the plan of 8 three eighths of the queues.  The chunk bounds, and so the
// order of a sequence's sums, follow P.B.
__device__ __forceinline__ int attn_chunk_keys(const Params &P, int n_keys)
{
    const int slots = P.attn_grid / P.B;
    const int pages = (n_keys + P.page - 1) >> P.page_shift;
    const int even = ((pages + slots - 1) / slots) << P.page_shift;
    return even > P.kv_chunk ? even : P.kv_chunk;
}

// The end of a chunk task: the first n_ent LDS entries (complete, behind a barrier) are reduced to the chunk's result,
// which is the attention output itself or one of the sequence's partial results.
template <int D, int GRP>
__device__ __forceinline__ void attn_finish(const Params &P, int b, int kvh, int ch, int chunk, int n_keys, int n_ent, float *sm, int task_id)
{
    ETC_AS_LDS float *s_m = as_lds(sm);
    ETC_AS_LDS float *s_l = s_m + kAttnEnt * GRP;
    ETC_AS_LDS float *s_o = s_m + kAttnOff<GRP>;
    // A sequence that is one chunk long needs no partial results, no arrival count and no merge: what a merge of one
    // chunk would compute is exactly num / den below (three memory round trips less at the end of the task).
    const int nc = (n_keys + chunk - 1) / chunk;
    const bool whole = nc == 1 && P.attn_arrive != nullptr;
    for (int idx = threadIdx.x; idx < GRP * D / 4; idx += kWgThreads) {      // four consecutive elements per thread: 8-byte stores
        const int g = idx / (D / 4), i = (idx % (D / 4)) * 4;
        float m = -INFINITY;
        for (int wv = 0; wv < n_ent; ++wv) m = fmaxf(m, s_m[wv * GRP + g]);
        float num[4] = {0.f, 0.f, 0.f, 0.f}, den = 0.f;
        for (int wv = 0; wv < n_ent; ++wv) {
            const float wm = s_m[wv * GRP + g];
            const float sc = (wm == -INFINITY) ? 0.f : exp2_f(wm - m);
            const f32x4 ov = *reinterpret_cast<ETC_AS_LDS const f32x4 *>(s_o + (size_t)(wv * GRP + g) * D + i);
#pragma unroll
            for (int q = 0; q < 4; ++q) num[q] += sc * ov[q];
            den += sc * s_l[wv * GRP + g];
        }
        const int h = kvh * GRP + g;
        if (whole) {               // the sequence's only chunk: this is the attention output (operand of the O projection)
            uint16_t hi[4], lo[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) split_bf16(num[q] / den, hi[q], lo[q]);
            const size_t o1 = (size_t)b * (size_t)(P.nq * D) + (size_t)h * D + i;
            st_u64(P.attn_hi + o1, (uint64_t)hi[0] | ((uint64_t)hi[1] << 16) | ((uint64_t)hi[2] << 32) | ((uint64_t)hi[3] << 48));
            st_u64(P.attn_lo + o1, (uint64_t)lo[0] | ((uint64_t)lo[1] << 16) | ((uint64_t)lo[2] << 32) | ((uint64_t)lo[3] << 48));
        } else {
            const size_t pidx = ((size_t)b * P.nq + h) * (size_t)P.max_chunks + ch;
            st_u64(P.part_o + pidx * D + i, (uint64_t)__float_as_uint(num[0]) | ((uint64_t)__float_as_uint(num[1]) << 32));
            st_u64(P.part_o + pidx * D + i + 2, (uint64_t)__float_as_uint(num[2]) | ((uint64_t)__float_as_uint(num[3]) << 32));
            if (i == 0) { st_f32(P.part_m + pidx, m); st_f32(P.part_l + pidx, den); }
        }
    }
    // The chunk task that arrives last at its (sequence, KV head) merges the chunks itself: the merge is no stage of
    // its own, one all-to-all hand-over less per layer.  Arrival is counted with one returning atomic per task (behind
    // the drain of the partial results); the last one puts the counter back for the next launch.  Every chunk task
    // still notifies the one event of the attention block, the merging one after its merge.
    trace_mark(P, task_id, 3);
    if (P.attn_arrive != nullptr && !whole) {
        ETC_AS_LDS int32_t *s_last = reinterpret_cast<ETC_AS_LDS int32_t *>(s_o + (size_t)kAttnEnt * GRP * D);
        drain_vmem();
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t *ctr = P.attn_arrive + (size_t)b * P.nkv + kvh;
            const int last = __hip_atomic_fetch_add(as_global(ctr), 1, __ATOMIC_RELAXED, ETC_SCOPE) + 1 == nc;
            if (last) st_i32(ctr, 0);
            *s_last = last;
        }
        __syncthreads();
        if (*s_last) attn_merge_chunks<D, GRP>(P, b, kvh, nc);
    }
}

// Two neighbouring values to bf16 (round to nearest even), and back.
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ float bf16_low(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_high(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Part `part` of (a, b) as bf16: part 0 the rounded value, part 1 what that leaves, part 2 what both leave, then nothing: the
// three add up to all 24 bits of a value.  What part 1 of 8 heads leaves has no column of its own and goes to `rest`.
template <int GRP>
__device__ __forceinline__ uint32_t bf16_part(float a, float b, int part, uint32_t &rest)
{
    const uint32_t h = pack_bf16(a, b);
    const float a1 = a - bf16_low(h), b1 = b - bf16_high(h);
    const uint32_t l = pack_bf16(a1, b1);
    const uint32_t l2 = pack_bf16(a1 - bf16_low(l), b1 - bf16_high(l));
    rest = GRP == 8 && part == 1 ? l2 : 0u;
    return part == 0 ? h : (part == 1 ? l : (part == 2 ? l2 : 0u));
}

// Across the four lane groups of 16: the same value in all of them.
__device__ __forceinline__ float groups_max(float v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float groups_sum(float v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// A chunk on the matrix cores (one head per KV head: long ones only, see attn_chunk_one_head).  A wavefront takes 32 (NBLK = 1: 16)
// keys per step:
//   scores   S^T[key][column] = K[key][:] . Q[column][:]   A = K rows, read as fragments (lane (key % 16, kg): 16 bytes of its
//            key's row) from a wavefront-private LDS tile, B = the queries as sums of bf16 parts.  The 16 columns hold the parts side by
//            side: column n is part n / GRP of head n % GRP (three parts, all 24 bits of a query), so one product per
//            fragment does for all parts and the columns of a head are added across lanes.  (8 heads fill the columns with two
//            parts: a second product adds the third one to the columns of the second.  Without it their queries and probabilities had
//            16 bits: 8.8e-6 instead of 2.1e-6 off where scores spread by tens, and 0.3 to 1 us a layer less.)  The result lands as lane (column, kg) <- keys blk * 16 + kg * 4 + r: eight keys of one head per lane, and in exactly the order
//            the next product wants its A fragment in;
//   softmax  per lane over its 8 keys, the maximum across the four lane groups by two row swaps, the running sum kept
//            per lane until the end;
//   output   O[row][d] += P[row][key] . V[key][d]   rows are parts and heads as the columns above (their sums are taken once, at
//            the end), A = P as it stands in the lanes, B = V with eight KEYS per lane: the V rows go through a
//            wavefront-private LDS tile, read back transposed (ds_read_b64_tr_b16).
// K and V rows of the next step are in flight while a step computes; the step's own token goes into an LDS entry of its own,
// next to the wavefronts' partial results.  Rows are loaded whole (a load of 64-byte pieces of 16 rows, the A fragment as it
// stands, made a task alone on the chip 112 us long instead of 73, 8192 keys) and past the caches (70B shape, batch 32: 1133 ->
// 1103 us per two layers); K and V pass through the same tile, one after the other.
// What bounds it is HBM: 8192 (2048) keys of each of 32 sequences take 175 (50) us a layer, 6.1 TB/s, with 4 and with 8 heads per
// KV head.  With vector code for up to 4 heads (4500 cycles of a SIMD per 32 keys) and 16 two-byte reads per V fragment for 8 it
// was 210 (64) and 233 (82).
// NBLK: blocks of 16 keys in a step.  A chunk of at most 128 keys is one step of 16 (all wavefronts have some) and no loop.  Longer
// chunks take 32, 128 KB in flight per compute unit, and have their callee clobber the caller's vector registers instead of saving
// them (see frame_anchor in gemm_tiles_chunked; 8B batch 16 / 48, two layers: 305 / 456 -> 300 / 440 us).  In the staged-only
// instances, whose task loop keeps values in vector registers over the call, that costs the 8B iteration 4 %, and the 33 saved
// registers of every lane cost more than the longer steps give (8B shape, chunks of 171 to 352 keys, two layers: 234 us against 228
// with steps of 16; chunks of 2048 keys, a layer: 63 against 59), so they take steps of 16 throughout.
//
// ev0 / ev1: the events the task waits on (the queries and this step's K / V row of the KV head).  The cached K / V
// rows do not depend on them: page ids and the rows of a wavefront's first step are requested BEFORE the wait, like a projection
// task's weights, so that after the wait only the queries are a round trip away.
template <int D, int GRP, int NBLK, bool LOOP>
__device__ __noinline__ void attn_chunk(const Params &P, int layer, int b, int kvh, int ch, int chunk, float *sm, int ev0, int ev1, int task_id,
                                        int *frame_anchor)
{
    constexpr int KK = D / 32, DB = D / 16;              // steps of 32 elements of a head, blocks of 16
    constexpr bool REST = GRP == 8;                      // a second product for the third parts
    constexpr int VS = 2 * D + 32;                       // bytes between two rows of a tile: transposed reads of 8 rows hit every bank once
    constexpr int LPR = D / 8, RPI = 64 / LPR, STEP = 16 * NBLK, NI = STEP / RPI;      // lanes per row, rows per load, keys of a step, loads
    static_assert((GRP & (GRP - 1)) == 0 && GRP <= 8 && (D == 64 || D == 128), "heads and parts fill at most 16 columns");
    static_assert((kAttnOff<GRP> + kAttnEnt * GRP * D) * 4 + 4 <= kAttnScratch && kAttnScratch + kWaves * 32 * VS + kAttnPages * 4 <= kLdsBytes, "LDS");
    task_id = __builtin_amdgcn_readfirstlane(task_id);
    if (NBLK > 1 && task_id == -0x7FFFFFFF) *frame_anchor = 1;       // never true: keeps the call from being a tail call (see gemm_tiles_chunked)
    layer = __builtin_amdgcn_readfirstlane(layer);       // uniform arguments back into scalar registers
    b = __builtin_amdgcn_readfirstlane(b);
    kvh = __builtin_amdgcn_readfirstlane(kvh);
    ch = __builtin_amdgcn_readfirstlane(ch);
    chunk = __builtin_amdgcn_readfirstlane(chunk);
    ev0 = __builtin_amdgcn_readfirstlane(ev0);
    ev1 = __builtin_amdgcn_readfirstlane(ev1);
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int n16 = lane & 15, kg = lane >> 4;
    const int n_keys = __builtin_amdgcn_readfirstlane(gld_i32(P.kv_len + b)) + 1;
    const int j0 = ch * chunk;
    const int j1 = j0 + min(n_keys - j0, chunk);
    const int jc1 = min(j1, n_keys - 1);                 // cached keys of the chunk: [j0, jc1), the step's own token is not read back
    const int32_t *pages = P.page_ids + __builtin_amdgcn_readfirstlane(gld_i32(P.page_indptr + b));
    const size_t lbase = (size_t)layer * (size_t)P.pool_layer_stride + (size_t)kvh * D;
    const float qscale = 1.44269504088896f / sqrtf((float)D);      // and log2(e)
    const int psh = P.page_shift, pmask = P.page - 1;    // pages hold a power of two of tokens
    ETC_AS_LDS float *s_m = as_lds(sm);                  // [kAttnEnt][GRP]
    ETC_AS_LDS float *s_l = s_m + kAttnEnt * GRP;        // [kAttnEnt][GRP]
    ETC_AS_LDS float *s_o = s_m + kAttnOff<GRP>;         // [kAttnEnt][GRP][D]
    // (The base of the dynamic LDS is a table look-up in a function that is no kernel, and the compiler repeats that
    // load where the pointer is used: inside the key loop it would drain the K / V loads in flight.  An empty asm
    // statement makes the value opaque: it is computed once.)
    uint32_t tiles = (uint32_t)(uintptr_t)(reinterpret_cast<ETC_AS_LDS char *>(as_lds(sm)) + kAttnScratch);
    asm volatile("" : "+v"(tiles));
    ETC_AS_LDS char *vt = reinterpret_cast<ETC_AS_LDS char *>(tiles) + wave * (32 * VS);      // this wavefront's V tile [32 keys][VS]
    ETC_AS_LDS int *s_pg = reinterpret_cast<ETC_AS_LDS int *>(tiles + kWaves * 32 * VS);

    // Page ids of the keys [w0, w1) sit in LDS: all of the chunk's, unless it is longer than kAttnPages pages.
    int w0 = j0, w1 = LOOP ? attn_window_end(j0, jc1, psh) : jc1;      // (j0 is a whole number of pages)
    auto load_pages = [&](int first) {
        for (int i = first + (int)threadIdx.x; i < attn_window_pages(w0, w1, psh); i += kWgThreads) s_pg[i] = gld_i32(pages + (w0 >> psh) + i);
    };
    // K and V rows of a step, whole rows per load: this lane has piece lane % LPR of the rows of the keys base + i * RPI +
    // lane / LPR; beyond the window: its last key again, weight 0
    u32x4 kr[NI], vr[NI];
    uint32_t at[NI];                                     // row of the pool: page * page size + place
    const int lr = lane / LPR, lp = lane % LPR;
    const uint32_t row_len = (uint32_t)__builtin_amdgcn_readfirstlane(P.nkv * D);
    auto row_offsets = [&](int base, bool from_lds) {
        int jc[NI], page[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int j = base + i * RPI + lr;
            jc[i] = j < w1 ? j : max(w1 - 1, w0);            // (a chunk of the new token alone: that token's place, not used)
            page[i] = from_lds ? s_pg[(jc[i] - w0) >> psh] : gld_i32(pages + (jc[i] >> psh));
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
            at[i] = ((uint32_t)page[i] << psh) + (uint32_t)(jc[i] & pmask);
    };
    auto request = [&](const uint16_t *pool, u32x4 (&r)[NI]) {
#pragma unroll
        for (int i = 0; i < NI; ++i) r[i] = gld_16B_nt(pool + lbase + (size_t)at[i] * row_len + lp * 8);
    };
    auto to_tile = [&](const u32x4 (&r)[NI]) {
#pragma unroll
        for (int i = 0; i < NI; ++i) *reinterpret_cast<ETC_AS_LDS u32x4 *>(vt + (i * RPI + lr) * VS + lp * 16) = r[i];
    };
    // In front of the wait: page ids, the first step's K rows and, in steps of 16 keys, its V rows.  (The poll queues behind what
    // its wavefront has requested, so no more than that; nor may it wait for a page id behind the rows.)
    int page_id = 0;
    if (LOOP) page_id = gld_i32(pages + (w0 >> psh) + min((int)threadIdx.x, max((w1 - w0 - 1) >> psh, 0)));
    row_offsets(w0 + wave * STEP, false);
    request(P.kpool, kr);
    if (NBLK == 1) request(P.vpool, vr);
    if (LOOP) {
        s_pg[threadIdx.x] = page_id;
        load_pages(kWgThreads);
    }
    if (ev0 < 0 && ev1 < 0) __syncthreads();             // the wait has a barrier
    wg_wait(P, ev0, ev1, FN_ATTN);
    trace_mark(P, task_id, 1);

    // ---- queries, and for the step's own token its K and V row: one round trip ----------------------------------
    // Lane (column n16, kg) holds elements kk * 32 + kg * 8 .. + 8 of head n16 % GRP.
    const int g_own = n16 & (GRP - 1), part = n16 / GRP, head = kvh * GRP + g_own;
    const bool takes_new = j1 == n_keys && wave == kWaves - 1;
    auto sum_of_squares = [&](int hd, f32x4 (&t)[D / 64]) {      // qk_norm models: the sums the head's projection tasks left
        const __amdgpu_buffer_rsrc_t sq_b = buf_of(P.qk_ssq);
#pragma unroll
        for (int i = 0; i < D / 64; ++i)
            t[i] = __builtin_bit_cast(f32x4, buf_ld_16B(sq_b, ((uint32_t)(b * (P.nq + P.nkv) + hd) * (D / 16) + 4 * i) * 4u, 0));
    };
    auto rnorm = [&](const f32x4 (&t)[D / 64]) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < D / 64; ++i) s += (t[i][0] + t[i][1]) + (t[i][2] + t[i][3]);
        return 1.0f / sqrtf(s / (float)D + P.eps);
    };
    f32x4 qf[KK][2], kn[KK][2], q_sq[D / 64], k_sq[D / 64];
    float vn[D / 64];
    {
        const __amdgpu_buffer_rsrc_t q_b = buf_of(P.qbuf), k_b = buf_of(P.knew);
        const uint32_t q_at = ((uint32_t)(b * P.nq + head) * D + kg * 8) * 4u, k_at = ((uint32_t)(b * P.nkv + kvh) * D + kg * 8) * 4u;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int h = 0; h < 2; ++h) qf[kk][h] = __builtin_bit_cast(f32x4, buf_ld_16B(q_b, q_at + kk * 128 + h * 16, 0));
        if (P.qk_norm) sum_of_squares(head, q_sq);
        if (takes_new) {
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int h = 0; h < 2; ++h) kn[kk][h] = __builtin_bit_cast(f32x4, buf_ld_16B(k_b, k_at + kk * 128 + h * 16, 0));
            if (P.qk_norm) sum_of_squares(P.nq + kvh, k_sq);
#pragma unroll
            for (int i = 0; i < D / 64; ++i) vn[i] = ld_f32(P.vnew + ((size_t)b * P.nkv + kvh) * D + i * 64 + lane);
        }
    }
    const float qs = P.qk_norm ? qscale * rnorm(q_sq) : qscale;
    bf16x8 qp[KK], qr[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        uint32_t w[4], r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            qf[kk][i >> 1][(2 * i) & 3] *= qs;
            qf[kk][i >> 1][(2 * i + 1) & 3] *= qs;
            w[i] = bf16_part<GRP>(qf[kk][i >> 1][(2 * i) & 3], qf[kk][i >> 1][(2 * i + 1) & 3], part, r[i]);
        }
        qp[kk] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
        qr[kk] = __builtin_bit_cast(bf16x8, u32x4{r[0], r[1], r[2], r[3]});
    }
    // ---- the token of this step: an LDS entry of its own (m = its score, l = 1, o = its V row), by the last wavefront, which
    // ---- has no step of its own in the shortest chunks
    if (takes_new) {
        const float rk = P.qk_norm ? rnorm(k_sq) : 1.f;
        float dot = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float k0 = kn[kk][i >> 1][(2 * i) & 3] * rk, k1 = kn[kk][i >> 1][(2 * i + 1) & 3] * rk;
                dot += qf[kk][i >> 1][(2 * i) & 3] * k0 + qf[kk][i >> 1][(2 * i + 1) & 3] * k1;
                w[i] = pack_bf16(k0, k1);
            }
            // K-Norm + RoPE + CacheAppend (Sec. 4.3): the key's norm is complete here, and so is its cache row (which nobody
            // reads in this launch)
            if (P.qk_norm && n16 == 0)
                *as_global(reinterpret_cast<u32x4 *>(P.kpool + lbase + (size_t)gld_i32(P.kv_slot + b) * (size_t)(P.nkv * D) + kk * 32 + kg * 8)) = u32x4{w[0], w[1], w[2], w[3]};
        }
        dot = groups_sum(dot);
        if (lane < GRP) { s_m[kWaves * GRP + lane] = dot; s_l[kWaves * GRP + lane] = 1.f; }
#pragma unroll
        for (int g = 0; g < GRP; ++g)
#pragma unroll
            for (int i = 0; i < D / 64; ++i) s_o[(size_t)(kWaves * GRP + g) * D + i * 64 + lane] = vn[i];
    }
    if (NBLK > 1) {                                      // here the registers of the queries are free
        __builtin_amdgcn_sched_barrier(0);
        request(P.vpool, vr);
    }

    // ---- the wavefront's steps: 16 NBLK keys each -------------------------------------------------------------------
    f32x4 oacc[DB];                                      // O[row kg * 4 + r][db * 16 + n16]
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x4{0, 0, 0, 0};
    float mrun = -INFINITY, lrun = 0.f;                  // of the head, over the keys this lane has seen
    ETC_AS_LDS const char *k_out = vt + n16 * VS + kg * 16;
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    ETC_AS_LDS char *v_out = vt + (kg * 4 + (n16 >> 2)) * VS + (n16 & 3) * 8;
    // One step; MORE (known to the compiler: a branch around a load would make the waits behind it drain all loads in flight):
    // there is another one, whose rows are requested on the way.
    auto step = [&](int base, auto more_c) {
        constexpr bool more = decltype(more_c)::value;
        if (more) row_offsets(base + kWaves * STEP, true);
        to_tile(kr);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 sacc[NBLK], srest[NBLK];
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk) sacc[blk] = srest[blk] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk) {
                const bf16x8 kf = *reinterpret_cast<ETC_AS_LDS const bf16x8 *>(k_out + blk * 16 * VS + kk * 64);
                sacc[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qp[kk], sacc[blk], 0, 0, 0);
                if constexpr (REST) srest[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qr[kk], srest[blk], 0, 0, 0);
            }
        // The registers: rows in flight 64, output 32, queries 16; a refill waits until the fragments read back from the tile are
        // used up, so that nothing a caller keeps in registers has to be saved.
        __builtin_amdgcn_sched_barrier(0);
        if (more) request(P.kpool, kr);
        __builtin_amdgcn_sched_barrier(0);
        to_tile(vr);                                 // behind the reads of the K rows
        __builtin_amdgcn_sched_barrier(0);
        if (more) request(P.vpool, vr);
        __builtin_amdgcn_sched_barrier(0);
        // softmax over this lane's keys (blk * 16 + kg * 4 + r) of its head
        float sv[4 * NBLK];
        float mloc = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4 * NBLK; ++j) {
            const int key = base + (j >> 2) * 16 + kg * 4 + (j & 3);
            // An infinite element of a key decides its score (-inf: weight 0) through the leading parts of a query; the lower ones, zero
            // or of the other sign, would make it a NaN.
            float v = sacc[j >> 2][j & 3], low = v;
            if constexpr (REST) low += srest[j >> 2][j & 3];
            v = part == 0 ? v : (__builtin_isfinite(low) ? low : 0.f);
            v += dpp_f32<0x128>(v);                  // the columns of a head: rotations of the row by 8, 4, 2, 1
            if constexpr (GRP <= 4) v += dpp_f32<0x124>(v);
            if constexpr (GRP <= 2) v += dpp_f32<0x122>(v);
            if constexpr (GRP == 1) v += dpp_f32<0x121>(v);
            sv[j] = key < w1 ? v : -INFINITY;
            mloc = fmaxf(mloc, sv[j]);
        }
        const float nm = fmaxf(mrun, groups_max(mloc));
        const float ref = fmaxf(nm, -1e30f);         // scores of -inf alone: exp2(-inf - ref) = 0 instead of exp2(nan)
        const float sc = exp2_f(mrun - ref);
        float psum = 0.f;
        uint32_t pw[2 * NBLK], pr[2 * NBLK];
#pragma unroll
        for (int j = 0; j < 4 * NBLK; j += 2) {
            const float p0 = exp2_f(sv[j] - ref), p1 = exp2_f(sv[j + 1] - ref);
            psum += p0 + p1;
            pw[j >> 1] = bf16_part<GRP>(p0, p1, part, pr[j >> 1]);
        }
        lrun = lrun * sc + psum;
        mrun = nm;
        // running output: rows kg * 4 + r, whose rescale factors sit in lanes kg * 4 + r
        if (__builtin_amdgcn_ballot_w64(sc != 1.0f) != 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float scr = __int_as_float(__builtin_amdgcn_ds_bpermute((kg * 4 + r) * 4, __float_as_int(sc)));
#pragma unroll
                for (int db = 0; db < DB; ++db) oacc[db][r] *= scr;
            }
        }
        // O += P . V: lane (column n16 of block db, kg) takes keys (j >> 2) * 16 + kg * 4 + (j & 3), j = 0 .. 4 NBLK, from the tile
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ETC_AS_LDS s16x4 *>(v_out + db * 32));
            if constexpr (NBLK == 1) {
                oacc[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, u32x2{pw[0], pw[1]}), lo, oacc[db], 0, 0, 0);
                if constexpr (REST) oacc[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, u32x2{pr[0], pr[1]}), lo, oacc[db], 0, 0, 0);
            } else {
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ETC_AS_LDS s16x4 *>(v_out + 16 * VS + db * 32));
                const u32x2 a = __builtin_bit_cast(u32x2, lo), c = __builtin_bit_cast(u32x2, hi);
                const bf16x8 vf = __builtin_bit_cast(bf16x8, u32x4{a.x, a.y, c.x, c.y});
                oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u32x4{pw[0], pw[1], pw[2], pw[3]}), vf, oacc[db], 0, 0, 0);
                if constexpr (REST) oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u32x4{pr[0], pr[1], pr[2], pr[3]}), vf, oacc[db], 0, 0, 0);
            }
            if (db % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (;;) {
        if (w0 + wave * STEP < w1) {                     // uniform per wavefront
            int base = w0 + wave * STEP;
            if constexpr (LOOP)
                for (; base + kWaves * STEP < w1; base += kWaves * STEP) step(base, std::true_type());
            step(base, std::false_type());
        }
        if (!LOOP || w1 >= jc1) break;               // uniform
        w0 = w1;
        w1 = attn_window_end(w0, jc1, psh);
        __syncthreads();                                 // every wavefront is done with the page ids
        load_pages(0);
        __syncthreads();
        row_offsets(w0 + wave * STEP, true);
        request(P.kpool, kr);
        request(P.vpool, vr);
    }
    trace_mark(P, task_id, 2);

    // ---- the wavefront's partial result: entry `wave` of the LDS table ----
    lrun = groups_sum(lrun);                             // the four lane groups saw different keys
    if (lane < GRP) { s_m[wave * GRP + lane] = mrun; s_l[wave * GRP + lane] = lrun; }
#pragma unroll
    for (int db = 0; db < DB; ++db) {                    // the parts of a head: rows GRP apart, kg * 4 + r of lane group kg
        ETC_AS_LDS float *dst = s_o + (size_t)wave * GRP * D + db * 16 + n16;
        if constexpr (GRP == 8) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = oacc[db][r] + __shfl_xor(oacc[db][r], 32, 64);
                if (kg < 2) dst[(kg * 4 + r) * D] = v;
            }
        } else if constexpr (GRP == 4) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = groups_sum(oacc[db][r]);
                if (kg == r) dst[r * D] = v;
            }
        } else if constexpr (GRP == 2) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float v = groups_sum(oacc[db][r] + oacc[db][r + 2]);
                if (kg == r) dst[r * D] = v;
            }
        } else {
            const float v = groups_sum((oacc[db][0] + oacc[db][1]) + (oacc[db][2] + oacc[db][3]));
            if (kg == 0) dst[0] = v;
        }
    }
    __syncthreads();
    attn_finish<D, GRP>(P, b, kvh, ch, chunk, n_keys, j1 == n_keys ? kWaves + 1 : kWaves, sm, task_id);
}

// One head per KV head, in fp32 on the vector units: D / 8 lanes to a key, 16 keys of a wavefront at a time.  On the matrix cores one
// column in 16 of a product has work there, and a step of 16 keys is bound by the chain through it (two LDS round trips, products, row
// swaps: a microsecond), where vector code needs a sum over 16 lanes and no LDS.  So it takes what goes in steps of 16, chunks of at
// most 128 keys and all of the staged-only instances, and chunks of at most kOneHeadKeys, which are one step of 32 there.  Eight layers,
// hidden 2048, 16 heads, batch 1 of 8192 / 8 of 500 / 8 of 2048 / 32 of 120 keys: 435 / 429 / 532 / 779 us on the matrix cores, 407 / 395 /
// 502 / 751 here.  In steps of 32, batch 64 of 250 / 500 / 1000 / 2048 keys at most: 1159 / 1260 / 1496 / 2026 there, 1123 here, 1247 /
// 1575 / 2195 with vector code for all.
// Everything else is as in attn_chunk: windows of page ids, rows requested ahead of the wait, the new token from its fp32 row.
constexpr int kOneHeadKeys = 256;
template <int D, bool LOOP>
__device__ __noinline__ void attn_chunk_one_head(const Params &P, int layer, int b, int kvh, int ch, int chunk, float *sm, int ev0, int ev1, int task_id)
{
    constexpr int LPK = D / 8, KPL = 64 / LPK, BATCH = 4, STEP = KPL * BATCH;      // lanes per key, keys per load, loads and keys of a step
    static_assert((kAttnOff<1> + kAttnEnt * D) * 4 + 4 <= kAttnScratch && kAttnScratch + kAttnPages * 4 <= kLdsBytes, "LDS");
    task_id = __builtin_amdgcn_readfirstlane(task_id);
    layer = __builtin_amdgcn_readfirstlane(layer);       // uniform arguments back into scalar registers
    b = __builtin_amdgcn_readfirstlane(b);
    kvh = __builtin_amdgcn_readfirstlane(kvh);
    ch = __builtin_amdgcn_readfirstlane(ch);
    chunk = __builtin_amdgcn_readfirstlane(chunk);
    ev0 = __builtin_amdgcn_readfirstlane(ev0);
    ev1 = __builtin_amdgcn_readfirstlane(ev1);
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id(), tq = lane / LPK, dl = lane % LPK;
    const int n_keys = __builtin_amdgcn_readfirstlane(gld_i32(P.kv_len + b)) + 1;
    const int j0 = ch * chunk;
    const int j1 = j0 + min(n_keys - j0, chunk);
    const int jc1 = min(j1, n_keys - 1);                 // cached keys of the chunk: [j0, jc1)
    const int32_t *pages = P.page_ids + __builtin_amdgcn_readfirstlane(gld_i32(P.page_indptr + b));
    const size_t lbase = (size_t)layer * (size_t)P.pool_layer_stride + (size_t)kvh * D;
    const float qscale = 1.44269504088896f / sqrtf((float)D);      // and log2(e)
    const int psh = P.page_shift, pmask = P.page - 1;
    ETC_AS_LDS float *s_m = as_lds(sm), *s_l = s_m + kAttnEnt, *s_o = s_m + kAttnOff<1>;      // [kAttnEnt], [kAttnEnt], [kAttnEnt][D]
    uint32_t pg_base = (uint32_t)(uintptr_t)(reinterpret_cast<ETC_AS_LDS char *>(as_lds(sm)) + kAttnScratch);
    asm volatile("" : "+v"(pg_base));                    // computed once (see attn_chunk)
    ETC_AS_LDS int *s_pg = reinterpret_cast<ETC_AS_LDS int *>(pg_base);

    int w0 = j0, w1 = LOOP ? attn_window_end(j0, jc1, psh) : jc1;
    auto load_pages = [&](int first) {
        for (int i = first + (int)threadIdx.x; i < attn_window_pages(w0, w1, psh); i += kWgThreads) s_pg[i] = gld_i32(pages + (w0 >> psh) + i);
    };
    // rows of a step: this lane has piece dl of the rows of the keys base + u * KPL + tq; beyond the window: its last key again, weight 0
    u32x4 kr[BATCH], vr[BATCH];
    const uint32_t row_len = (uint32_t)__builtin_amdgcn_readfirstlane(P.nkv * D);
    auto request = [&](int base, bool from_lds) {
        int jc[BATCH], page[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int j = base + u * KPL + tq;
            jc[u] = j < w1 ? j : max(w1 - 1, w0);            // (a chunk of the new token alone: that token's place, not used)
            page[u] = from_lds ? s_pg[(jc[u] - w0) >> psh] : gld_i32(pages + (jc[u] >> psh));
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const size_t off = lbase + (size_t)(((uint32_t)page[u] << psh) + (uint32_t)(jc[u] & pmask)) * row_len + dl * 8;
            kr[u] = gld_16B(P.kpool + off);
            vr[u] = gld_16B(P.vpool + off);
        }
    };
    auto widen = [](u32x4 r, float (&f)[8]) {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) { f[2 * i] = bf16_low(w[i]); f[2 * i + 1] = bf16_high(w[i]); }
    };
    int page_id = 0;
    if (LOOP) page_id = gld_i32(pages + (w0 >> psh) + min((int)threadIdx.x, max((w1 - w0 - 1) >> psh, 0)));
    request(w0 + wave * STEP, false);
    if (LOOP) {
        s_pg[threadIdx.x] = page_id;
        load_pages(kWgThreads);
    }
    if (ev0 < 0 && ev1 < 0) __syncthreads();             // the wait has a barrier
    wg_wait(P, ev0, ev1, FN_ATTN);
    trace_mark(P, task_id, 1);

    // ---- the query, and for the step's own token its K and V row: one round trip ----------------------------------
    const bool takes_new = j1 == n_keys && wave == 0;
    float q[8], kn[8], vn[8], q_sq[D / 16], k_sq[D / 16];
    auto row_of = [&](const float *p, float (&f)[8]) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) ld_f32x2(p + dl * 8 + i, f[i], f[i + 1]);
    };
    auto sum_of_squares = [&](int hd, float (&t)[D / 16]) {      // qk_norm models: the sums the head's projection tasks left
#pragma unroll
        for (int i = 0; i < D / 16; ++i) t[i] = ld_f32(P.qk_ssq + ((size_t)b * (P.nq + P.nkv) + hd) * (size_t)(D / 16) + i);
    };
    auto rnorm = [&](const float (&t)[D / 16]) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < D / 16; ++i) s += t[i];
        return 1.0f / sqrtf(s / (float)D + P.eps);
    };
    row_of(P.qbuf + ((size_t)b * P.nq + kvh) * D, q);
    if (P.qk_norm) sum_of_squares(kvh, q_sq);
    if (takes_new) {
        row_of(P.knew + ((size_t)b * P.nkv + kvh) * D, kn);
        row_of(P.vnew + ((size_t)b * P.nkv + kvh) * D, vn);
        if (P.qk_norm) sum_of_squares(P.nq + kvh, k_sq);
    }
    const float qs = P.qk_norm ? qscale * rnorm(q_sq) : qscale;
    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { q[i] *= qs; o[i] = 0.f; }
    if (takes_new) {                                     // the first key of lane group 0 of wavefront 0: weight 1
        const float rk = P.qk_norm ? rnorm(k_sq) : 1.f;
        float sc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) { kn[i] *= rk; sc += q[i] * kn[i]; }
        sc = lanes_sum<LPK>(sc);
        if (tq == 0) {
            m = sc;
            l = 1.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = vn[i];
            if (P.qk_norm)       // K-Norm + RoPE + CacheAppend (Sec. 4.3): the key's norm is complete here, and so is its cache row
                *as_global(reinterpret_cast<u32x4 *>(P.kpool + lbase + (size_t)gld_i32(P.kv_slot + b) * row_len + dl * 8)) =
                    u32x4{pack_bf16(kn[0], kn[1]), pack_bf16(kn[2], kn[3]), pack_bf16(kn[4], kn[5]), pack_bf16(kn[6], kn[7])};
        }
    }

    // ---- the wavefront's steps: all scores, one new maximum and one rescale, then the weighted rows ------------------
    auto fold = [&](int base) {
        float p[BATCH], nm = m;
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            float kf[8], sc = 0.f;
            widen(kr[u], kf);
#pragma unroll
            for (int i = 0; i < 8; ++i) sc += q[i] * kf[i];
            sc = lanes_sum<LPK>(sc);
            p[u] = base + u * KPL + tq < w1 ? sc : -INFINITY;
            nm = fmaxf(nm, p[u]);
        }
        const float ref = fmaxf(nm, -1e30f);             // scores of -inf alone: exp2(-inf - ref) = 0 instead of exp2(nan)
        const float sc = exp2_f(m - ref);
        l *= sc;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] *= sc;
        m = nm;
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            float vf[8];
            widen(vr[u], vf);
            p[u] = exp2_f(p[u] - ref);
            l += p[u];
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] += p[u] * vf[i];
        }
    };
    for (;;) {
        int base = w0 + wave * STEP;
        if (base < w1) fold(base);                       // uniform per wavefront
        if constexpr (LOOP)
            for (base += kWaves * STEP; base < w1; base += kWaves * STEP) {
                request(base, true);
                fold(base);
            }
        if (!LOOP || w1 >= jc1) break;                   // uniform
        w0 = w1;
        w1 = attn_window_end(w0, jc1, psh);
        __syncthreads();                                 // every wavefront is done with the page ids
        load_pages(0);
        __syncthreads();
        request(w0 + wave * STEP, true);
    }
    trace_mark(P, task_id, 2);

    // ---- the wavefront's partial result: its lane groups saw different keys; entry `wave` of the LDS table ----
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
        const float om = __shfl_xor(m, off, 64), ol = __shfl_xor(l, off, 64), nm = fmaxf(m, om), ref = fmaxf(nm, -1e30f);
        const float sa = exp2_f(m - ref), sb = exp2_f(om - ref);
        l = l * sa + ol * sb;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = o[i] * sa + __shfl_xor(o[i], off, 64) * sb;
        m = nm;
    }
    if (tq == 0) {
        if (dl == 0) { s_m[wave] = m; s_l[wave] = l; }
#pragma unroll
        for (int i = 0; i < 8; ++i) s_o[(size_t)wave * D + dl * 8 + i] = o[i];
    }
    __syncthreads();
    attn_finish<D, 1>(P, b, kvh, ch, chunk, n_keys, kWaves, sm, task_id);
}

// Merge of the chunk partials of (sequence b, KV head kvh): ascending chunk order, whoever runs it.
template <int D, int GRP>
__device__ __forceinline__ void attn_merge_chunks(const Params &P, int b, int kvh, int nc)
{
    for (int idx = threadIdx.x; idx < GRP * D; idx += kWgThreads) {
        const int g = idx / D, i = idx % D;
        const int h = kvh * GRP + g;
        const size_t p0 = ((size_t)b * P.nq + h) * (size_t)P.max_chunks;
        // one pass in ascending chunk order, 16 chunks' loads in flight at a time, running max rescaling
        float m = -INFINITY, num = 0.f, den = 0.f;
        for (int c0 = 0; c0 < nc; c0 += 16) {
            float pm[16], pl[16], po[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int c = c0 + u < nc ? c0 + u : nc - 1;
                pm[u] = ld_f32(P.part_m + p0 + c);
                pl[u] = ld_f32(P.part_l + p0 + c);
                po[u] = ld_f32(P.part_o + (p0 + c) * D + i);
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if (c0 + u < nc) {
                    const float nm = fmaxf(m, pm[u]);
                    const float sa = exp2_f(m - nm), sb = exp2_f(pm[u] - nm);
                    num = num * sa + sb * po[u];
                    den = den * sa + sb * pl[u];
                    m = nm;
                }
            }
        }
        uint16_t hi, lo;                               // operand of the O projection: split bf16
        split_bf16(num / den, hi, lo);
        const size_t o = (size_t)b * (size_t)(P.nq * D) + (size_t)h * D + i;
        st_u16(P.attn_hi + o, hi);
        st_u16(P.attn_lo + o, lo);
    }
}

}  // namespace etc
