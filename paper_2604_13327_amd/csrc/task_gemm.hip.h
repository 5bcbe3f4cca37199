// Projection tile task: 16 weight rows x K against up to 64 activation columns, bf16 MFMA with
// fp32 accumulation (v_mfma_f32_16x16x32_bf16), weights streamed from HBM exactly once.
//
// Work split (small batches; the out-of-line paths have their own).  The 8 wavefronts of the workgroup split K; each
// streams its slice of all 16 rows with 16-byte non-temporal loads of whole lines (unit_row), keeping PF loads (PF KB per
// wave, 128 KB per CU) in flight.  The first of them are issued BEFORE the task waits on its events (weight prefetch, paper Sec. 3.4 / 4.3), so
// HBM keeps streaming while the dependency resolves.
//
// Activation operand.  Activations reach the MFMA as bf16, which alone would cost ~2^-9 relative error
// per projection and break the 2e-2 parity bar after a few dozen layers.  The PRODUCER of an activation
// therefore stores it as two bf16 numbers, hi + lo (16 mantissa bits), and the tile issues two MFMAs per
// weight fragment (hi and lo); the matrix pipe is <10 % busy in this HBM-bound regime, so this is free.
// RMSNorm is folded in the same way: the producer stores (x * gain) split, plus one partial sum of
// squares per 16-row tile; the consumer sums the partials in a fixed order and scales its accumulator
// by 1/sqrt(mean(x^2)+eps) in the epilogue (the norm factor is a per-column scalar, so it commutes
// with the contraction).  No separate norm task, no extra event hop.
//
// The 16 rows of a tile are two groups of 8 (rowsA, rowsB): a RoPE tile takes rows i..i+7 and
// i+d/2..i+d/2+7 of one head (8 rotation pairs), a SwiGLU tile takes 8 gate rows and the 8 matching
// up rows, plain tiles take 16 consecutive rows.  Partial tiles of the 8 waves are reduced through LDS
// in a fixed order (deterministic), then the epilogue runs on 8 x columns threads.
#pragma once
#include <type_traits>

#include "device_rt.hip.h"

namespace etc {

struct GemmTile {
    const uint16_t *rowsA, *rowsB;   // bf16 weights, first row of each 8-row group
    int ldw;                         // weight row stride (elements)
    int K;                           // reduction length, multiple of 256
    const uint16_t *b_hi, *b_lo;     // activation operand, split bf16, [rows, ldb]
    int ldb;
    const int32_t *col_rows;         // optional gather: column n reads operand row col_rows[n]
    int n_cols;                      // valid columns (batch rows or routed tokens), <= 64
    const float *ssq_parts;          // RMSNorm: partial sums of squares [n_parts][ssq_stride], or null
    int n_parts;
    int ssq_stride;
    float eps;
    int n_tiles;                     // consecutive 16-row tiles this task streams back to back
    int tile_rows;                   // rows between consecutive tiles inside each 8-row group (8 or 16)
    int w_shared;                    // GroupGEMM: other row blocks stream the same weights (they may stay in the caches)
};

constexpr uint16_t EPF_DUMP_LAYER = 0x8000;   // epilogue also records the layer's hidden state

enum EpiKind : int { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_STORE_F32 = 3, EPI_MOE_ACT = 4, EPI_MOE_Y = 5,
                     EPI_PARTIAL = 6, EPI_LOGITS = 7 };   // PARTIAL: fp32 sums over one slice of K, [row tile][kMaxBatch][16], outf = the slice's block

struct Epilogue {
    int kind;
    int layer;
    uint16_t flags;
    int row0;                 // first output row (RESID / STORE), first f (SWIGLU), first pair index (QKV)
    int head;                 // QKV: global head index (q heads, then k heads, then v heads)
    const float *resid;       // RESID: [*, ld] fp32 added to the result
    float *outf;              // fp32 destination
    uint16_t *out_hi, *out_lo;// split-bf16 destination (operand of the consuming projection)
    const uint16_t *next_gain;// RESID: gain the consumer's RMSNorm applies (null: no operand is prepared)
    float *ssq_out;           // RESID: this tile's partial sums of squares [kMaxBatch]
    int ld;                   // destination row stride
    int col0;                 // MoE: first destination row (permuted row of column 0)
    ETC_AS_LDS unsigned long long *lds_best;   // LOGITS: the task's running maxima per column, in LDS (set by the projection path)
};

// What an epilogue thread needs from memory, fetched before the streaming loop so that the epilogue
// itself issues no load (a load issued behind the weight stream returns only after it: memory
// operations of a wavefront complete in order).
struct EpiPre {
    float a, b;       // RESID: the two residual values; QKV: cos and sin of the rotation angle
    float ga, gb;     // RESID: gains of the two rows for the consumer's operand
    int slot;         // QKV (k / v heads): KV slot of the appended row (page * page_size + position in the page)
};
__device__ __forceinline__ EpiPre epilogue_preload(const Params &P, const Epilogue &e, int col, int mp);
template <bool LM>
__device__ __forceinline__ void apply_epilogue(const Params &P, const Epilogue &e, int col, int mp, float lo, float hi,
                                               const EpiPre &pre);
__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }

constexpr int PF = 16;                            // weight loads in flight per lane (16 KB per wave)

__device__ __forceinline__ u32x4 load16_nt(const uint16_t *p) { return gld_16B_nt(p); }
__device__ __forceinline__ void ld_f32x2_pair(const float *p, float &a, float &b) { a = ld_f32(p); b = ld_f32(p + 8); }

// Waits of a projection task.  per_wave: wave w waits on ev0 + w (its own K slice) on its own.
struct TaskWaits {
    int ev0, ev1, fn;
    bool per_wave;
    int op_key;          // identifies the operand a staged copy in LDS holds (-1: never reuse a copy)
};

// State a persistent workgroup carries from task to task (uniform across the workgroup).
struct WgState {
    int zero0, zero1;    // events already seen at zero in this launch (they never re-arm inside a launch)
    int staged_key;      // operand currently staged in LDS (-1: none)
    int routed_layer;    // MoE layer whose routing tables this workgroup has already seen complete (-1: none)
};

__device__ __forceinline__ void wg_state_init(WgState &st)
{
    st.zero0 = st.zero1 = -1;
    st.staged_key = -1;
    st.routed_layer = -1;
}

__device__ __forceinline__ bool event_known_zero(const WgState &st, int ev) { return ev < 0 || ev == st.zero0 || ev == st.zero1; }

// Whole lines of weights per load.  The A fragment of the 16x16x32 product is 16 rows x 64 bytes: loaded as it stands, every
// load touches 16 half lines, and streamed non-temporally that costs a fifth of the rate (256 workgroups, 16 loads in
// flight per lane: 5.6 - 5.9 TB/s; 8 rows x 128 bytes per load 6.9, contiguous memory 7.0).  So a load takes 8 rows x one
// UNIT of 64 elements of K: lane (x = lane % 16, kg = lane / 16) the 16-byte piece 2 kg + x % 2 of row x / 2.  In the
// product, rows x of one parity then hold the pieces of that parity, so the operand is given in the same way: its column
// n holds the pieces 2 kg + n % 2 of batch column n / 2, and the product of equal parities is the sum over those pieces
// (the other half of the product is not used).  8 batch columns per product instead of 16: the matrix pipe has room for
// that up to 16 columns or so, and the operand fragment serves both 8-row groups of a tile.
constexpr int kUnitK = 64;
__device__ __forceinline__ const uint16_t *unit_row(const uint16_t *rows, int ldw)
{
    const int x = lane_id() & 15, kg = lane_id() >> 4;
    return rows + (size_t)(x >> 1) * (size_t)ldw + (kg * 2 + (x & 1)) * 8;
}
// Sums of the two parities: lane (n, kg) gets rows 2 kg and 2 kg + 1 of group n % 2 (0: rowsA, 1: rowsB) for batch column
// n / 2 of the group of 8.  acc register i of lane (n, kg) is product row 4 kg + i: row 2 kg + i / 2 of its 8, parity i % 2.
__device__ __forceinline__ void unit_sums(const f32x4 &accA, const f32x4 &accB, float (&v)[2])
{
    const bool odd = (lane_id() & 1) != 0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float give = odd ? accA[2 * j + 1] : accB[2 * j], keep = odd ? accB[2 * j + 1] : accA[2 * j];
        v[j] = keep + dpp_f32<0xB1>(give);               // neighbouring lane (quad_perm [1,0,3,2])
    }
}
// Units of K a wavefront takes when the 8 of them split K / 64 units: [first, first + count).
__device__ __forceinline__ void wave_units(int K, int wave, int &first, int &count)
{
    const int n = K / kUnitK;
    first = n * wave / kWaves;
    count = n * (wave + 1) / kWaves - first;
}

// Workgroup wait with a two-entry cache of events already known to have fired.
__device__ __forceinline__ void wg_wait_cached(const Params &P, WgState &st, int ev0, int ev1, int fn)
{
    const bool need0 = ev0 >= 0 && ev0 != st.zero0 && ev0 != st.zero1;
    const bool need1 = ev1 >= 0 && ev1 != st.zero0 && ev1 != st.zero1;
    if (!need0 && !need1) return;
    wg_wait(P, need0 ? ev0 : -1, need1 ? ev1 : -1, fn);
    if (need0) { st.zero1 = st.zero0; st.zero0 = ev0; }
    if (need1) { st.zero1 = st.zero0; st.zero0 = ev1; }
}

// Latency-critical path (at most 16 columns whose whole operand fits in LDS).  The operand (all columns,
// full K, hi and lo) is copied into LDS once per stage with device-scope loads and reused by every
// tile of that stage this workgroup runs.  A task streams its n_tiles row tiles back to back through a
// ring of PF weight fragments per lane that never drains between tiles; each wave parks its partial
// tile in LDS; one barrier, one reduction and one epilogue per task.
//
// Order of memory operations.  A wavefront's loads return in order, so anything issued behind the
// weight stream waits for it.  The first PF weight loads are issued BEFORE the task waits on its events
// (weight prefetch, Sec. 3.4); the epilogue's inputs are fetched before the streaming loop, so the
// epilogue issues no load.  Measured alternatives that lost: streaming the NEXT task's first fragments
// during the tail of the loop (the epilogue's loads and the drain before the notify then queue behind that
// stream: +10 % per step); keeping the polling wavefront's queue free of weight loads until the event is
// seen (+2 %); one control wavefront that polls, stages and runs the epilogue while seven wavefronts
// stream (+10 %: the compute unit's read rate follows the bytes it keeps in flight, and the gap between
// two stages is longer than what its registers can buffer either way).
//
// Shape of the streaming loop.  The task's weights are ONE linear stream of (tile, unit) pairs; an issue cursor
// runs PF / 2 units ahead of the consume cursor.  The compiler places wait counts per basic block, and what it
// cannot follow it answers with a full drain of the loads in flight, so the loop is written for it:
//   - the steady state (whole revolutions of the ring whose look-ahead units all exist) has no branch around
//     a load, and so have the common endings (one revolution left; one and a half);
//   - a ring slot is refilled BEHIND the MFMAs that read it, so the new fragment can land in the same
//     registers: refilled in front of them it needs other registers, and the copy back at the loop's end
//     waits for every load of the revolution.
// With both, every step waits for exactly the oldest of the PF loads (4.08 -> 3.94 ms per 8B step).
template <int PRE, int NG, bool LM>
__device__ __forceinline__ void gemm_tiles_staged(const Params &P, const GemmTile &g, const Epilogue &e, const TaskWaits &w,
                                                  float *sm, WgState &st, int task_id)
{
    // PRE: ring units requested before the wait; NG: groups of 8 columns (1 or 2)
    constexpr int PU = PF / 2;                        // a ring unit is two loads: rows A and rows B
    static_assert(PRE >= 1 && PRE <= PU && (NG == 1 || NG == 2), "ring units requested before the wait, column groups");
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int n16 = lane & 15, kg = lane >> 4;
    int unit0, n_it;                                  // this wavefront's units of K
    wave_units(g.K, wave, unit0, n_it);
    const size_t tile_step = (size_t)g.tile_rows * (size_t)g.ldw;

    // What a later task may find again (norm factors, operand) lies in front of what depends on this task's tile count: the
    // tasks of a stage share the operand, and the last one of the vocabulary projection has fewer tiles than the others.
    ETC_AS_LDS float *rs = as_lds(sm);
    ETC_AS_LDS uint16_t *op_hi = reinterpret_cast<ETC_AS_LDS uint16_t *>(rs + kRsFloats);
    const int Kp = g.K + kOpPad;                        // column stride of the operand in LDS
    ETC_AS_LDS uint16_t *op_lo = op_hi + (size_t)g.n_cols * Kp;
    ETC_AS_LDS float *red = reinterpret_cast<ETC_AS_LDS float *>(op_lo + (size_t)g.n_cols * Kp);      // [tile][wave][col][16 rows]

    const int key = w.op_key;
    const bool restage = key < 0 || key != st.staged_key;
    // Gathered columns: lane n has the operand row of column n (16 at most).  Known since the routing, requested ahead of the weights:
    // behind them every look-up is a round trip under load.
    const bool gathered = g.col_rows != nullptr;
    int lane_row = lane & 15;
    if (gathered) lane_row = max(ld_i32(g.col_rows + ((lane & 15) < g.n_cols ? lane & 15 : g.n_cols - 1)), 0);
    // The task's weights are one linear stream of (tile, unit) pairs: unit s of tile t sits t * tile_step + 64 s behind the
    // first one.  The issue cursor runs PU units ahead of the consume cursor through that stream.
    const int total = g.n_tiles * n_it;
    const long long tile_jump = (long long)tile_step - (long long)n_it * kUnitK;
    const uint16_t *ipA = unit_row(g.rowsA, g.ldw) + unit0 * kUnitK;      // next unit to request
    const uint16_t *ipB = unit_row(g.rowsB, g.ldw) + unit0 * kUnitK;
    int is = 0;                                       // its place inside its tile
    auto advance_issue = [&]() {
        ++is;
        const bool wrap = is == n_it;
        const long long by = kUnitK + (wrap ? tile_jump : 0);
        ipA += by;
        ipB += by;
        is = wrap ? 0 : is;
    };
    u32x4 wr[PF];
    // Of the PU ring units, PRE are requested before the task waits on its events and the rest behind the operand once the
    // events have fired: the poll and the operand queue behind whatever was prefetched, which costs the workgroup that
    // arrives last (and sets the stage's end) what it gains the early ones.  Measured: 8B step (staged-only instance)
    // 4 / 5 / 6 / 7 / 8 units = 3.95 / 3.88 / 3.88 / 3.95 / 3.92 ms; the MoE step is 5 % faster with all 8 (its tasks are
    // small and many), so the count is a parameter of the instance.
    auto prefetch_range = [&](int j0, int j1) {
#pragma unroll
        for (int j = 0; j < PU; ++j) {
            if (j >= j0 && j < j1) {
                if (j < total) {
                    wr[2 * j] = load16_nt(ipA);
                    wr[2 * j + 1] = load16_nt(ipB);
                    advance_issue();
                } else {
                    wr[2 * j] = wr[2 * j + 1] = u32x4{0, 0, 0, 0};
                }
            }
        }
    };
    auto prefetch = [&]() { prefetch_range(0, PU); };
    // A task that has nothing to wait for (its events are already known to have fired, or it runs without
    // events in the kernel-by-kernel comparator) issues its operand loads first and the weight stream right
    // behind them: loads return in order, so the operand would otherwise arrive a full round trip under load
    // later.  A task that has to wait prefetches first.  (Deciding this with one extra poll at task start was
    // measured: the round trip it adds on every workgroup costs more than it saves on the last one.)
    const bool will_wait = restage ? (!event_known_zero(st, w.ev0) || w.per_wave || !event_known_zero(st, w.ev1))
                                   : !event_known_zero(st, w.ev1);
    const bool fired = !will_wait;
    if (!fired) prefetch_range(0, PRE);

    // What the epilogue will need (single pass of the epilogue loop only) is requested right behind the operand:
    // it is back by the time the operand sits in LDS, and the streaming loop starts without another round trip.
    const int per_tile = g.n_cols * 8;
    const int n_out = g.n_tiles * per_tile;
    const bool pre_ok = n_out <= kWgThreads;
    EpiPre pre{};
    auto request_epilogue_inputs = [&]() {
        if (pre_ok && (int)threadIdx.x < n_out) {
            const int ti = (int)threadIdx.x / per_tile, r = (int)threadIdx.x - ti * per_tile;
            Epilogue et = e;
            et.row0 = e.row0 + ti * g.tile_rows;
            pre = epilogue_preload(P, et, r >> 3, r & 7);
        }
    };

    if (restage) {
        // ---- E.wait() ---------------------------------------------------------------------------
        if (fired) {
            if (!w.per_wave && !event_known_zero(st, w.ev0)) { st.zero1 = st.zero0; st.zero0 = w.ev0; }
            if (!event_known_zero(st, w.ev1)) { st.zero1 = st.zero0; st.zero0 = w.ev1; }
        } else if (w.per_wave) {    // the staged copy needs every K slice: lanes 0..7 of wave 0 poll one slice each
            if (wave == 0 && lane < kWaves) spin_until_zero(P, w.ev0 + lane, w.fn);
            if (wave_id() == 0) spin_event(P, w.ev1, w.fn);
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        } else {
            wg_wait_cached(P, st, w.ev0, w.ev1, w.fn);
        }
        trace_mark(P, task_id, 1);
        // ---- stage the operand: all loads of a thread in flight at once ---------------------------
        constexpr int U = 4;
        const int ppc = g.K >> 3;                           // 16-byte pieces per column
        const int total_p = g.n_cols * ppc;
        const __amdgpu_buffer_rsrc_t hi_b = buf_of(g.b_hi), lo_b = buf_of(g.b_lo);
        float sq[8];                                        // RMSNorm: this lane's partial sums of squares of column `wave`
        const bool one_col_per_wave = g.ssq_parts != nullptr && g.n_cols <= kWaves && g.n_parts <= 512;
        auto request_norm = [&]() {
            if (one_col_per_wave && wave < g.n_cols) {
                const int row = gathered ? __builtin_amdgcn_readlane(lane_row, wave) : wave;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int pt = lane + 64 * j;
                    sq[j] = pt < g.n_parts ? ld_f32(g.ssq_parts + (size_t)pt * (size_t)g.ssq_stride + row) : 0.f;
                }
            }
        };
        u32x4 vh[U], vl[U];
        uint32_t at[U];
        int i0 = threadIdx.x;
        auto load_pieces = [&]() {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int idx = i0 + u * kWgThreads;
                const int col = idx < total_p ? idx / ppc : 0, q = idx - col * ppc;
                const int row = gathered ? __shfl(lane_row, col, 64) : col;
                at[u] = (uint32_t)(col * Kp + q * 8);
                const uint32_t off = idx < total_p ? ((uint32_t)row * (uint32_t)g.ldb + (uint32_t)q * 8u) * 2u : kBufNone;
                vh[u] = buf_ld_16B(hi_b, off, 0);
                vl[u] = buf_ld_16B(lo_b, off, 0);
            }
        };
        auto store_pieces = [&]() {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u * kWgThreads < total_p) {
                    *reinterpret_cast<ETC_AS_LDS u32x4 *>(op_hi + at[u]) = vh[u];
                    *reinterpret_cast<ETC_AS_LDS u32x4 *>(op_lo + at[u]) = vl[u];
                }
            }
        };
        for (int left = total_p; left > U * kWgThreads; left -= U * kWgThreads) {
            load_pieces();
            store_pieces();
            i0 += U * kWgThreads;
        }
        load_pieces();       // everything else the task needs is requested behind its last pieces, without a branch around it
        request_norm();
        request_epilogue_inputs();
        if (fired) prefetch(); else prefetch_range(PRE, PU);
        store_pieces();
        if (g.ssq_parts) {       // RMSNorm factor of every column: fixed-order sum of the producers' partial sums of squares
            if (one_col_per_wave) {
                if (wave < g.n_cols) {
                    float s = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
                    s = wave_sum(s);
                    if (lane == 0) rs[wave] = 1.0f / sqrtf(s / (float)g.K + g.eps);
                }
            } else {
                for (int col = wave; col < g.n_cols; col += kWaves) {
                    const int row = gathered ? __builtin_amdgcn_readlane(lane_row, col) : col;
                    float s = 0.f;
                    for (int pt = lane; pt < g.n_parts; pt += 64) s += ld_f32(g.ssq_parts + (size_t)pt * (size_t)g.ssq_stride + row);
                    s = wave_sum(s);
                    if (lane == 0) rs[col] = 1.0f / sqrtf(s / (float)g.K + g.eps);
                }
            }
        }
        st.staged_key = key;
        __syncthreads();
    } else {
        if (fired) {
            if (!event_known_zero(st, w.ev1)) { st.zero1 = st.zero0; st.zero0 = w.ev1; }
            request_epilogue_inputs();
            prefetch();
        } else {
            wg_wait_cached(P, st, w.ev1, -1, w.fn);
            request_epilogue_inputs();
            prefetch_range(PRE, PU);
        }
    }
    trace_mark(P, task_id, 2);

    // operand fragments: column n16 / 2 of each group of 8, pieces 2 kg + n16 % 2; columns beyond n_cols read column 0's
    // operand (never stored)
    ETC_AS_LDS const uint16_t *sh[NG], *sl[NG];
#pragma unroll
    for (int ng = 0; ng < NG; ++ng) {
        const int col = ng * 8 + (n16 >> 1), c = col < g.n_cols ? col : 0;
        sh[ng] = op_hi + (size_t)c * (size_t)Kp + unit0 * kUnitK + (kg * 2 + (n16 & 1)) * 8;
        sl[ng] = op_lo + (size_t)c * (size_t)Kp + unit0 * kUnitK + (kg * 2 + (n16 & 1)) * 8;
    }
    // Consume cursor: unit sc of tile tc.
    f32x4 accA[NG], accB[NG];
#pragma unroll
    for (int ng = 0; ng < NG; ++ng) accA[ng] = accB[ng] = f32x4{0, 0, 0, 0};
    int sc = 0, tc = 0;
    auto store_tile = [&](int t) {      // rows 2 kg, 2 kg + 1 of group n16 % 2, this wavefront's share of K
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) {
            float v[2];
            unit_sums(accA[ng], accB[ng], v);
            const int col = ng * 8 + (n16 >> 1);
            if (col < g.n_cols) {
                ETC_AS_LDS float *dst = red + ((size_t)(t * kWaves + wave) * g.n_cols + col) * 16 + (n16 & 1) * 8 + 2 * kg;
                dst[0] = v[0];
                dst[1] = v[1];
            }
            accA[ng] = accB[ng] = f32x4{0, 0, 0, 0};
        }
    };
#define ETC_STAGED_UNIT(j, RELOAD)                                                                               \
    {                                                                                                             \
        const bf16x8 a0 = __builtin_bit_cast(bf16x8, wr[2 * (j)]), a1 = __builtin_bit_cast(bf16x8, wr[2 * (j) + 1]); \
        _Pragma("unroll") for (int ng = 0; ng < NG; ++ng) {                                                       \
            const bf16x8 bh = __builtin_bit_cast(bf16x8, *reinterpret_cast<ETC_AS_LDS const u32x4 *>(sh[ng] + sc * kUnitK)); \
            const bf16x8 bl = __builtin_bit_cast(bf16x8, *reinterpret_cast<ETC_AS_LDS const u32x4 *>(sl[ng] + sc * kUnitK)); \
            accA[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bh, accA[ng], 0, 0, 0);                        \
            accB[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bh, accB[ng], 0, 0, 0);                        \
            accA[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bl, accA[ng], 0, 0, 0);                        \
            accB[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bl, accB[ng], 0, 0, 0);                        \
        }                                                                                                         \
        if (RELOAD) {           /* behind the MFMAs that read the slots: the loads can land in the same registers */ \
            wr[2 * (j)] = load16_nt(ipA);                                                                         \
            wr[2 * (j) + 1] = load16_nt(ipB);                                                                     \
            advance_issue();                                                                                      \
        }                                                                                                         \
        if (++sc == n_it) {     /* tile done */                                                                   \
            store_tile(tc);                                                                                       \
            sc = 0;                                                                                               \
            ++tc;                                                                                                 \
        }                                                                                                         \
    }
    // Steady state: whole ring revolutions whose look-ahead units all exist.  No branch around a load here: the
    // compiler places its wait counts per basic block, and a conditional load turns the waits behind it into full
    // drains of the ring.
    int q = 0;
    for (; q + 2 * PU <= total; q += PU) {
#pragma unroll
        for (int j = 0; j < PU; ++j) ETC_STAGED_UNIT(j, true)
    }
    if (total - q == PU) {                           // one whole revolution left: nothing to request, nothing to test
#pragma unroll
        for (int j = 0; j < PU; ++j) ETC_STAGED_UNIT(j, false)
        q = total;
    } else if (total - q == PU + PU / 2) {           // one and a half (K = 3.5 revolutions per tile, one tile)
#pragma unroll
        for (int j = 0; j < PU / 2; ++j) ETC_STAGED_UNIT(j, true)
#pragma unroll
        for (int j = PU / 2; j < PU; ++j) ETC_STAGED_UNIT(j, false)
#pragma unroll
        for (int j = 0; j < PU / 2; ++j) ETC_STAGED_UNIT(j, false)
        q = total;
    }
    for (; q < total; q += PU) {                     // the last revolutions of any other length
#pragma unroll
        for (int j = 0; j < PU; ++j) {
            if (q + j < total) {
                if (q + j + PU < total) ETC_STAGED_UNIT(j, true)
                else ETC_STAGED_UNIT(j, false)
            }
        }
    }
#undef ETC_STAGED_UNIT
    if (n_it == 0)                                   // K of fewer units than wavefronts: this one has none
        for (int t = 0; t < g.n_tiles; ++t) store_tile(t);

    // ---- one reduction (fixed wave order) and one epilogue for all tiles of the task -------------
    trace_mark(P, task_id, 3);
    ETC_AS_LDS unsigned long long *lbest = reinterpret_cast<ETC_AS_LDS unsigned long long *>(rs + kRsFloats / 2);   // [16]
    const bool to_best = LM && e.kind == EPI_LOGITS;
    if (to_best && (int)threadIdx.x < g.n_cols) lbest[threadIdx.x] = 0ull;
    __syncthreads();
    for (int idx = threadIdx.x; idx < n_out; idx += kWgThreads) {
        const int ti = idx / per_tile, r = idx - ti * per_tile;
        const int col = r >> 3, mp = r & 7;
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int wv = 0; wv < kWaves; ++wv) {
            ETC_AS_LDS const float *base = red + ((size_t)(ti * kWaves + wv) * g.n_cols + col) * 16;
            lo += base[mp];
            hi += base[mp + 8];
        }
        if (g.ssq_parts) {
            const float rn = rs[col];
            lo *= rn;
            hi *= rn;
        }
        Epilogue et = e;
        et.row0 = e.row0 + ti * g.tile_rows;
        et.lds_best = lbest;
        if (e.ssq_out) et.ssq_out = e.ssq_out + (size_t)ti * kMaxBatch;
        if (!pre_ok) pre = epilogue_preload(P, et, col, mp);
        apply_epilogue<LM>(P, et, col, mp, lo, hi, pre);
    }
    if (to_best) {       // the task's maxima join the sequences' running maxima
        __syncthreads();
        if ((int)threadIdx.x < g.n_cols)
            __hip_atomic_fetch_max(as_global(P.best + threadIdx.x), lbest[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Out-of-line path of tasks of at most 4 row tiles whose operand does not fit a whole copy in LDS (batches above 16
// columns, QKV above all).  The operand is walked in chunks of KC elements of K: a chunk of ALL columns (hi and lo) sits
// in LDS, double buffered; while the wavefronts run the MFMAs of chunk c out of one buffer, every thread already
// has its 16-byte pieces of chunk c+1 in flight into registers (8-byte ones ran at 41 GB/s per compute unit, these at 67)
// and drops them into the other buffer at the end of the chunk: one barrier per chunk.  Within a chunk a wavefront owns 32
// of every 256 elements of K (S = KC / 256 MFMA steps); a task streams T row tiles against one pass over the operand,
// which every task has to read in full, with a ring of PFC weight fragments in flight per lane running over
// (chunk, step, tile) triples.  Register budget decides the shape: accumulators take T x NB x 4 registers,
// the ring 4 PFC, the operand pieces in flight COLS x KC / 512 - so 16 columns keep the full ring of 16, 32
// columns a ring of 8, 64 columns a ring of 4.  Nothing may spill inside the loop: a
// register reload is a memory load that queues behind the whole ring.
//
// The steady state of the loop is free of branches.  The compiler places its wait counts per basic block;
// a branch around a load (a dead tile slot, a column beyond the batch, a chunk beyond K) makes every later
// wait a full drain of the loads in flight, which halves the streaming rate.  So the steady state always
// moves T tiles (slots beyond n_tiles stream the last live tile again and are never stored), columns beyond
// n_cols read row 0, and only the last ring revolutions, whose look-ahead leaves K, run the conditional code.

// Arguments of the out-of-line path travel through LDS: passed by value they fill the argument registers and
// spill to the stack, i.e. every lane writes and reads its own copy of the same descriptors through scratch memory.
struct ChunkedArgs {
    GemmTile g;
    Epilogue e;
    TaskWaits w;
    int task_id;
};
__device__ __forceinline__ ChunkedArgs *chunked_args_slot()
{
    __shared__ ChunkedArgs slot;
    return &slot;
}

// `frame_anchor` points into the caller's stack frame and is there for the compiler alone.  A call that could be a
// tail call makes the callee save and restore every callee-saved vector register it uses, through scratch memory,
// on every call: 112 registers per lane here, at batch 64 twenty times the bytes the tasks produce.  A callee whose
// call sites all hand it a piece of the caller's frame cannot be tail-called; the compiler then tells the callers
// what the callee clobbers instead, and the callers (the task loop) have next to nothing live across the call.
template <int NB, int T, bool BUF16>
__device__ __noinline__ void gemm_tiles_chunked(const Params &P, const ChunkedArgs *args, float *sm, int *frame_anchor)
{
    const ChunkedArgs a = lds_get_uniform(args);
    if (a.task_id == -0x7FFFFFFF) *frame_anchor = 1;      // never true (task ids are >= -1)
    const GemmTile &g = a.g;
    const Epilogue &e = a.e;
    const TaskWaits &w = a.w;
    const int task_id = a.task_id;
    static_assert(T == 1 || T == 2 || T == 4, "row tiles per pass");
    constexpr int PFC = NB == 1 ? (T >= 4 ? PF : 8) : (NB == 2 ? 8 : 4);   // weight loads in flight per lane, as the registers allow
    constexpr int COLS = NB * 16;
    constexpr int S = (4 / NB) < (PFC / T) ? (4 / NB) : (PFC / T);   // MFMA steps per wavefront, chunk and tile
    constexpr int KC = 256 * S;                    // K elements per chunk
    constexpr int STRIDE = KC + 8;                 // LDS column stride in elements: 16 columns cover all banks
    constexpr int PE = BUF16 ? 8 : 4;              // elements of a piece
    constexpr int PPC = KC / PE;                   // pieces per column and half
    constexpr int U = COLS * PPC / kWgThreads;     // pieces per thread, chunk and half
    constexpr int BUF = 2 * COLS * STRIDE;         // elements of one buffer: hi columns, then lo columns
    constexpr int CPR = PFC / (T * S);              // chunks per revolution of the ring
    static_assert(COLS * PPC == U * kWgThreads, "every thread moves U pieces of each half");
    static_assert(CPR >= 1 && CPR * T * S == PFC, "the ring holds whole chunks");
    static_assert((size_t)2 * BUF * 2 + (64 + 512) * 4 <= (size_t)kLdsBytes, "two operand buffers and the norm scratch fit");
    static_assert((size_t)kWaves * NB * 256 * 4 <= (size_t)BUF * 2, "the reduction buffer aliases one operand buffer");
    const int wave = wave_id(), lane = lane_id();
    const int m = lane & 15, kg = lane >> 4;
    const int K = __builtin_amdgcn_readfirstlane(g.K);
    const int n_chunks = (K + KC - 1) / KC;        // K is a multiple of 256; the last chunk may be partial
    const int n_full = K / KC;                     // chunks that lie inside K with all their steps
    const int n_tiles = __builtin_amdgcn_readfirstlane(g.n_tiles);
    const size_t tile_step = (size_t)g.tile_rows * (size_t)g.ldw;
    const uint16_t *wbase = (m < 8 ? g.rowsA + (size_t)m * (size_t)g.ldw : g.rowsB + (size_t)(m - 8) * (size_t)g.ldw) +
                            wave * 32 + kg * 8;
    // The steady state of the streaming loop has no branch (a branch around a load makes every later wait
    // a full drain of the loads in flight): it always moves T row tiles, slots beyond n_tiles stream the
    // last live tile again and are never stored; columns beyond n_cols read row 0.
    uint32_t toff[T];                              // uniform element offsets of the tiles: scalar registers
#pragma unroll
    for (int ti = 0; ti < T; ++ti)
        toff[ti] = __builtin_amdgcn_readfirstlane((uint32_t)((size_t)(ti < n_tiles ? ti : n_tiles - 1) * tile_step));

    ETC_AS_LDS uint16_t *buf0 = reinterpret_cast<ETC_AS_LDS uint16_t *>(as_lds(sm));
    ETC_AS_LDS float *red = as_lds(sm);                                  // after the last chunk
    ETC_AS_LDS float *rs = reinterpret_cast<ETC_AS_LDS float *>(buf0 + 2 * BUF);
    ETC_AS_LDS float *rs_part = rs + 64;                                  // [8][64]

    // ring slot j <-> (chunk j / (S*T) of the revolution, step (j / T) % S, tile j % T)
    auto step_live = [&](int c, int sidx) { return c * KC + sidx * 256 < K; };
    // ---- weight prefetch before the wait ---------------------------------------------------------------
    u32x4 wr[PFC];
#pragma unroll
    for (int j = 0; j < PFC; ++j) {
        const int c = j / (S * T), sidx = (j / T) % S, ti = j % T;
        if (step_live(c, sidx)) wr[j] = gld_16B(wbase + toff[ti] + c * KC + sidx * 256);
        else wr[j] = u32x4{0, 0, 0, 0};
    }
    // ---- E.wait(): the operand is needed in full, so every K slice event is waited for ---------------
    if (w.per_wave) {
        if (wave == 0 && lane < kWaves) spin_until_zero(P, w.ev0 + lane, w.fn);
        if (wave_id() == 0) spin_event(P, w.ev1, w.fn);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
        wg_wait(P, w.ev0, w.ev1, w.fn);
    }
    trace_mark(P, task_id, 1);

    // this thread's pieces of every chunk: piece tid + 512u = (column, piece of the column's chunk)
    using Piece = typename std::conditional<BUF16, u32x4, uint64_t>::type;
    const __amdgpu_buffer_rsrc_t hi_b = buf_of(g.b_hi), lo_b = buf_of(g.b_lo);
    int rows[U], pcs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int idx = (int)threadIdx.x + kWgThreads * u;
        const int col = idx / PPC;
        pcs[u] = idx - col * PPC;
        rows[u] = 0;
        if (col < g.n_cols) rows[u] = g.col_rows ? ld_i32(g.col_rows + col) : col;
        if (rows[u] < 0) rows[u] = 0;
        if (BUF16)                                 // byte offset from here on; a column beyond n_cols loads nothing
            rows[u] = col < g.n_cols ? (int)(((uint32_t)rows[u] * (uint32_t)g.ldb + (uint32_t)pcs[u] * PE) * 2u) : (int)kBufNone;
    }
    Piece vh[U], vl[U];
    auto fetch_piece = [&](int u, int c) {
        if constexpr (BUF16) {
            vh[u] = buf_ld_16B(hi_b, (uint32_t)rows[u], (uint32_t)c * (KC * 2));
            vl[u] = buf_ld_16B(lo_b, (uint32_t)rows[u], (uint32_t)c * (KC * 2));
        } else {
            const size_t off = (size_t)rows[u] * (size_t)g.ldb + (size_t)c * KC + pcs[u] * PE;
            vh[u] = ld_u64(g.b_hi + off);
            vl[u] = ld_u64(g.b_lo + off);
        }
    };
    auto fetch_chunk = [&](int c) {                // any chunk: pieces beyond K are left out
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vh[u] = vl[u] = Piece{};
            if (c * KC + pcs[u] * PE < K) fetch_piece(u, c);
        }
    };
    auto fetch_full_chunk = [&](int c) {           // a chunk inside K: no conditions, and not sunk towards its use
#pragma unroll
        for (int u = 0; u < U; ++u) fetch_piece(u, c);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto park_chunk = [&](int b) {
        ETC_AS_LDS uint16_t *hi = buf0 + b * BUF, *lo = hi + COLS * STRIDE;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = (int)threadIdx.x + kWgThreads * u;
            const int col = idx / PPC;
            *reinterpret_cast<ETC_AS_LDS Piece *>(hi + col * STRIDE + pcs[u] * PE) = vh[u];
            *reinterpret_cast<ETC_AS_LDS Piece *>(lo + col * STRIDE + pcs[u] * PE) = vl[u];
        }
    };
    fetch_chunk(0);

    // ---- RMSNorm factors: thread (column, group) sums every 8th partial sum of squares, groups meet in LDS ----
    if (g.ssq_parts) {
        const int col = threadIdx.x & 63;
        int row = -1;
        if (col < g.n_cols) row = g.col_rows ? ld_i32(g.col_rows + col) : col;
        float s = 0.f;
        for (int p0 = wave; p0 < g.n_parts; p0 += 8 * 16) {
            float t[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int pt = p0 + 8 * j;
                t[j] = (pt < g.n_parts && row >= 0) ? ld_f32(g.ssq_parts + (size_t)pt * (size_t)g.ssq_stride + row) : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) s += t[j];
        }
        rs_part[wave * 64 + col] = s;
    }
    park_chunk(0);
    __syncthreads();
    if (g.ssq_parts && threadIdx.x < 64) {
        float s = 0.f;
#pragma unroll
        for (int gq = 0; gq < 8; ++gq) s += rs_part[gq * 64 + threadIdx.x];
        rs[threadIdx.x] = 1.0f / sqrtf(s / (float)g.K + g.eps);
    }
    trace_mark(P, task_id, 2);

    f32x4 acc[T][NB];
#pragma unroll
    for (int ti = 0; ti < T; ++ti)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[ti][nb] = f32x4{0, 0, 0, 0};

    // one MFMA step of all T tiles out of ring slots j0 .. j0+T-1; RELOAD: the slots are refilled for chunk cn
#define ETC_CHUNK_STEP(hi, lo, sidx, cc, cn, RELOAD)                                                             \
    {                                                                                                             \
        u32x4 fb[NB];                                                                                             \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                         \
            fb[nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(hi + nb * 16 * STRIDE + (sidx) * 256);            \
        _Pragma("unroll") for (int ti = 0; ti < T; ++ti) {                                                        \
            const bf16x8 a = __builtin_bit_cast(bf16x8, wr[((cc) * S + (sidx)) * T + ti]);                        \
            _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) acc[ti][nb] =                                       \
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, fb[nb]), acc[ti][nb], 0, 0, 0); \
        }                                                                                                         \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                         \
            fb[nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(lo + nb * 16 * STRIDE + (sidx) * 256);            \
        _Pragma("unroll") for (int ti = 0; ti < T; ++ti) {                                                        \
            const int j = ((cc) * S + (sidx)) * T + ti;                                                           \
            const bf16x8 a = __builtin_bit_cast(bf16x8, wr[j]);                                                   \
            if (RELOAD) wr[j] = gld_16B(wbase + toff[ti] + (size_t)(cn) * KC + (sidx) * 256);                   \
            _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) acc[ti][nb] =                                       \
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, fb[nb]), acc[ti][nb], 0, 0, 0); \
        }                                                                                                         \
    }
    int c0 = 0;
    for (; c0 + 2 * CPR <= n_full; c0 += CPR) {    // steady state: this revolution, the next chunk and the chunks
#pragma unroll                                     // the ring is refilled for all lie inside K: no conditions
        for (int cc = 0; cc < CPR; ++cc) {
            const int c = c0 + cc, b = c & 1;
            fetch_full_chunk(c + 1);
            ETC_AS_LDS const uint16_t *hi = buf0 + b * BUF + m * STRIDE + wave * 32 + kg * 8;
            ETC_AS_LDS const uint16_t *lo = hi + COLS * STRIDE;
#pragma unroll
            for (int sidx = 0; sidx < S; ++sidx) ETC_CHUNK_STEP(hi, lo, sidx, cc, c + CPR, true)
            park_chunk(b ^ 1);
            __syncthreads();
        }
    }
    for (; c0 < n_chunks; c0 += CPR) {             // the last revolutions: every load and step is conditional
#pragma unroll
        for (int cc = 0; cc < CPR; ++cc) {
            const int c = c0 + cc;
            if (c < n_chunks) {                    // uniform
                const int b = c & 1;
                if (c + 1 < n_chunks) fetch_chunk(c + 1);
                ETC_AS_LDS const uint16_t *hi = buf0 + b * BUF + m * STRIDE + wave * 32 + kg * 8;
                ETC_AS_LDS const uint16_t *lo = hi + COLS * STRIDE;
#pragma unroll
                for (int sidx = 0; sidx < S; ++sidx) {
                    if (step_live(c, sidx)) {      // uniform
                        if (step_live(c + CPR, sidx)) ETC_CHUNK_STEP(hi, lo, sidx, cc, c + CPR, true)
                        else ETC_CHUNK_STEP(hi, lo, sidx, cc, c + CPR, false)
                    }
                }
                if (c + 1 < n_chunks) park_chunk(b ^ 1);
                __syncthreads();
            }
        }
    }
#undef ETC_CHUNK_STEP

    // ---- per tile: partials of the 8 wavefronts through LDS, fixed order, epilogue ----------------------
    trace_mark(P, task_id, 3);
    ETC_AS_LDS unsigned long long *lbest = reinterpret_cast<ETC_AS_LDS unsigned long long *>(rs_part);   // [64]: the norm scratch is free by now
    const bool to_best = e.kind == EPI_LOGITS;
    if (to_best && (int)threadIdx.x < g.n_cols) lbest[threadIdx.x] = 0ull;      // ordered by the barrier behind the first tile's partials
#pragma unroll
    for (int ti = 0; ti < T; ++ti) {
        if (ti < n_tiles) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                *reinterpret_cast<ETC_AS_LDS f32x4 *>(red + ((size_t)(wave * NB + nb) * 64 + lane) * 4) = acc[ti][nb];
            __syncthreads();
            Epilogue et = e;
            et.row0 = e.row0 + ti * g.tile_rows;
            et.lds_best = lbest;
            if (e.ssq_out) et.ssq_out = e.ssq_out + (size_t)ti * kMaxBatch;
            for (int idx = threadIdx.x; idx < g.n_cols * 8; idx += kWgThreads) {
                const int col = idx >> 3, mp = idx & 7;
                const int nb = col >> 4, n = col & 15;
                float lo = 0.f, hi = 0.f;
#pragma unroll
                for (int wv = 0; wv < kWaves; ++wv) {
                    ETC_AS_LDS const float *base = red + (size_t)(wv * NB + nb) * 256;
                    lo += base[(n + 16 * (mp >> 2)) * 4 + (mp & 3)];
                    hi += base[(n + 16 * ((mp + 8) >> 2)) * 4 + (mp & 3)];
                }
                if (g.ssq_parts) {
                    const float r = rs[col];
                    lo *= r;
                    hi *= r;
                }
                apply_epilogue<true>(P, et, col, mp, lo, hi, epilogue_preload(P, et, col, mp));
            }
            __syncthreads();
        }
    }
    if (to_best && (int)threadIdx.x < g.n_cols)       // behind the last tile's barrier
        __hip_atomic_fetch_max(as_global(P.best + threadIdx.x), lbest[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits of the task's events (with the weights of its first steps already requested), as in the paths above.
__device__ __forceinline__ void gemm_wait(const Params &P, const TaskWaits &w)
{
    if (w.per_wave) {
        if (wave_id() == 0 && lane_id() < kWaves) spin_until_zero(P, w.ev0 + lane_id(), w.fn);
        if (wave_id() == 0) spin_event(P, w.ev1, w.fn);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
        wg_wait(P, w.ev0, w.ev1, w.fn);
    }
}

// RMSNorm factors of the columns, first half: thread (column, group) leaves its share of the column's sum of squares in
// rs_part [512 / NCOL][NCOL].  Behind a barrier norm_factors() adds the shares.  norm_request: the loads of its first 16 parts.
template <int NCOL>
__device__ __forceinline__ int norm_row(const GemmTile &g)      // operand row of this thread's column, -1: none
{
    const int col = (int)threadIdx.x % NCOL;
    if (g.col_rows) {
        const int row = ld_i32(g.col_rows + (col < g.n_cols ? col : g.n_cols - 1));
        return col < g.n_cols ? row : -1;
    }
    return col < g.n_cols ? col : -1;
}
template <int NCOL>
__device__ __forceinline__ void norm_request(const GemmTile &g, int row, float (&t)[16])
{
    constexpr int GRPS = kWgThreads / NCOL;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int pt = (int)threadIdx.x / NCOL + GRPS * j;
        t[j] = (pt < g.n_parts && row >= 0) ? ld_f32(g.ssq_parts + (size_t)pt * (size_t)g.ssq_stride + row) : 0.f;
    }
}
template <int NCOL>
__device__ __forceinline__ void norm_shares(const GemmTile &g, int row, float (&t)[16], ETC_AS_LDS float *rs_part)
{
    constexpr int GRPS = kWgThreads / NCOL;
    const int col = (int)threadIdx.x % NCOL, grp = (int)threadIdx.x / NCOL;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) s += t[j];
    for (int p0 = grp + GRPS * 16; p0 < g.n_parts; p0 += GRPS * 16) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int pt = p0 + GRPS * j;
            t[j] = (pt < g.n_parts && row >= 0) ? ld_f32(g.ssq_parts + (size_t)pt * (size_t)g.ssq_stride + row) : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) s += t[j];
    }
    rs_part[grp * NCOL + col] = s;
}
template <int NCOL>
__device__ __forceinline__ void norm_shares(const GemmTile &g, ETC_AS_LDS float *rs_part)
{
    float t[16];
    const int row = norm_row<NCOL>(g);
    norm_request<NCOL>(g, row, t);
    norm_shares<NCOL>(g, row, t, rs_part);
}
template <int NCOL>
__device__ __forceinline__ void norm_factors(const GemmTile &g, ETC_AS_LDS float *rs, const ETC_AS_LDS float *rs_part)
{
    if (threadIdx.x >= NCOL) return;
    float s = 0.f;
#pragma unroll
    for (int gq = 0; gq < kWgThreads / NCOL; ++gq) s += rs_part[gq * NCOL + threadIdx.x];
    rs[threadIdx.x] = 1.0f / sqrtf(s / (float)g.K + g.eps);
}

// Four gate rows and the four matching up rows of a column -> silu(gate) * up, split, 8 bytes each to hi and lo.
__device__ __forceinline__ void store_swiglu4(__amdgpu_buffer_rsrc_t hi_b, __amdgpu_buffer_rsrc_t lo_b, uint32_t off, const f32x4 &gate,
                                              const f32x4 &up, float r)
{
    uint16_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_bf16(silu_f(gate[i] * r) * (up[i] * r), h[i], l[i]);
    buf_st_8B(hi_b, off, u32x2{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)});
    buf_st_8B(lo_b, off, u32x2{(uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16)});
}

// Epilogues that need no other thread's rows run straight from the accumulators of a 16-row tile: a lane holds rows
// 4 kg .. 4 kg + 3 of column nb * 16 + m.  SwiGLU pairs gate row r with up row r + 8, two lane groups further: lanes
// kg < 2 finish the even column blocks and lanes kg >= 2 the odd ones, after one exchange.
__device__ __forceinline__ constexpr bool epilogue_is_direct(int kind)
{
    return kind == EPI_SWIGLU || kind == EPI_MOE_ACT || kind == EPI_PARTIAL || kind == EPI_MOE_Y;
}
template <int NB>
__device__ __forceinline__ void epilogue_direct(const Epilogue &e, int row0, int n_cols, const f32x4 (&acc)[NB],
                                                const ETC_AS_LDS float *rs, bool normed)
{
    const int lane = lane_id(), m = lane & 15, kg = lane >> 4;
    if (e.kind == EPI_SWIGLU || e.kind == EPI_MOE_ACT) {
        const size_t first = e.kind == EPI_MOE_ACT ? (size_t)e.col0 * e.ld : 0;
        const __amdgpu_buffer_rsrc_t hi_b = buf_of(e.out_hi + first), lo_b = buf_of(e.out_lo + first);
        const bool lower = kg < 2;
        const uint32_t f = (uint32_t)(row0 + (kg & 1) * 4);
        if constexpr (NB == 1) {
            f32x4 up;
#pragma unroll
            for (int i = 0; i < 4; ++i) up[i] = __shfl_xor(acc[0][i], 32, 64);
            if (lower && m < n_cols) store_swiglu4(hi_b, lo_b, ((uint32_t)m * (uint32_t)e.ld + f) * 2u, acc[0], up, normed ? rs[m] : 1.f);
        } else {
#pragma unroll
            for (int nb = 0; nb < NB; nb += 2) {
                f32x4 gate, up;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float got = __shfl_xor(lower ? acc[nb + 1][i] : acc[nb][i], 32, 64);
                    gate[i] = lower ? acc[nb][i] : got;
                    up[i] = lower ? got : acc[nb + 1][i];
                }
                const int col = (lower ? nb : nb + 1) * 16 + m;
                if (col < n_cols) store_swiglu4(hi_b, lo_b, ((uint32_t)col * (uint32_t)e.ld + f) * 2u, gate, up, normed ? rs[col] : 1.f);
            }
        }
    } else {
        const bool partial = e.kind == EPI_PARTIAL;
        const __amdgpu_buffer_rsrc_t out_b = buf_of(partial ? e.outf : e.outf + (size_t)e.col0 * e.ld);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int col = nb * 16 + m;
            const uint32_t o = partial ? (uint32_t)(((row0 >> 4) * kMaxBatch + col) * 16 + 4 * kg)
                                       : (uint32_t)col * (uint32_t)e.ld + (uint32_t)(row0 + 4 * kg);
            if (col < n_cols) buf_st_16B(out_b, o * 4u, __builtin_bit_cast(u32x4, acc[nb]));
        }
    }
}

// The same from the sums of unit_sums(): lane (n16, kg) has rows 2 kg, 2 kg + 1 of group n16 % 2 of column ng * 8 + n16 / 2;
// SwiGLU pairs them with the neighbouring lane's, the same rows of the other group.
template <int NG>
__device__ __forceinline__ void epilogue_direct_units(const Epilogue &e, int row0, int n_cols, const float (&sums)[NG][2],
                                                      const ETC_AS_LDS float *rs, bool normed)
{
    const int lane = lane_id(), n16 = lane & 15, kg = lane >> 4;
    if (e.kind == EPI_SWIGLU || e.kind == EPI_MOE_ACT) {
        const size_t first = e.kind == EPI_MOE_ACT ? (size_t)e.col0 * e.ld : 0;
        const __amdgpu_buffer_rsrc_t hi_b = buf_of(e.out_hi + first), lo_b = buf_of(e.out_lo + first);
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) {
            const int col = ng * 8 + (n16 >> 1);
            const float r = normed ? rs[col] : 1.f;
            const float v0 = sums[ng][0] * r, v1 = sums[ng][1] * r;
            const float u0 = dpp_f32<0xB1>(v0), u1 = dpp_f32<0xB1>(v1);
            if ((n16 & 1) == 0 && col < n_cols) {
                uint16_t h0, l0, h1, l1;
                split_bf16(silu_f(v0) * u0, h0, l0);
                split_bf16(silu_f(v1) * u1, h1, l1);
                const uint32_t o = ((uint32_t)col * (uint32_t)e.ld + (uint32_t)(row0 + 2 * kg)) * 2u;
                buf_st_4B(hi_b, o, (uint32_t)h0 | ((uint32_t)h1 << 16));
                buf_st_4B(lo_b, o, (uint32_t)l0 | ((uint32_t)l1 << 16));
            }
        }
    } else {
        const bool partial = e.kind == EPI_PARTIAL;
        const __amdgpu_buffer_rsrc_t out_b = buf_of(partial ? e.outf : e.outf + (size_t)e.col0 * e.ld);
        const int r = (n16 & 1) * 8 + 2 * kg;
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) {
            const int col = ng * 8 + (n16 >> 1);
            const uint32_t o = partial ? (uint32_t)(((row0 >> 4) * kMaxBatch + col) * 16 + r) : (uint32_t)col * (uint32_t)e.ld + (uint32_t)(row0 + r);
            if (col < n_cols) buf_st_8B(out_b, o * 4u, u32x2{__float_as_uint(sums[ng][0]), __float_as_uint(sums[ng][1])});
        }
    }
}

// The epilogues that need other threads' rows, tile by tile out of LDS (the caller has written the tiles, no barrier yet).
template <int NB>
__device__ __forceinline__ void tiles_epilogue(const Params &P, const ChunkedArgs &a, const ETC_AS_LDS float *tb, const ETC_AS_LDS float *rs,
                                               ETC_AS_LDS float *rs_part, int n_tiles)
{
    const GemmTile &g = a.g;
    const Epilogue &e = a.e;
    ETC_AS_LDS unsigned long long *lbest = reinterpret_cast<ETC_AS_LDS unsigned long long *>(rs_part);
    const bool to_best = e.kind == EPI_LOGITS;
    if (to_best && (int)threadIdx.x < g.n_cols) lbest[threadIdx.x] = 0ull;
    __syncthreads();
    for (int ti = 0; ti < n_tiles; ++ti) {
        Epilogue et = e;
        et.row0 = e.row0 + ti * g.tile_rows;
        et.lds_best = lbest;
        if (e.ssq_out) et.ssq_out = e.ssq_out + (size_t)ti * kMaxBatch;
        const int idx = threadIdx.x;
        if (idx < g.n_cols * 8) {
            const int col = idx >> 3, mp = idx & 7;
            const int nb = col >> 4, n = col & 15;
            ETC_AS_LDS const float *base = tb + (size_t)(ti * NB + nb) * 256;
            float lo = base[(n + 16 * (mp >> 2)) * 4 + (mp & 3)];
            float hi = base[(n + 16 * ((mp + 8) >> 2)) * 4 + (mp & 3)];
            if (g.ssq_parts) {
                const float r = rs[col];
                lo *= r;
                hi *= r;
            }
            apply_epilogue<true>(P, et, col, mp, lo, hi, epilogue_preload(P, et, col, mp));
        }
    }
    __syncthreads();                               // the next pass parks its operand over the tiles
    if (to_best && (int)threadIdx.x < g.n_cols)
        __hip_atomic_fetch_max(as_global(P.best + threadIdx.x), lbest[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wide path: decoder tasks of 5 or more row tiles at 33 .. 64 columns.  The chunked path splits K over the 8 wavefronts, so
// every wavefront holds accumulators for all tiles of the pass (at 64 columns a pass is 4 tiles: the operand, hi and lo, is
// read again for every 256 KB of weights) and the tiles meet in a reduction across wavefronts.  Here the wavefronts split
// the OUTPUT: a pair of them owns TW row tiles of the pass, each half of every chunk of K (which halves the operand reads
// from LDS, 27 us of a 56 us gate/up stage of the 8B shape when every wavefront took the whole operand); the operand chunk
// in LDS (double buffered) is shared by all of them, a pass is 4 x TW tiles, and the pair exchanges half of its sums.
// What bounds it is bytes through the fabric: at 64 columns the operand is as large as the weights of a task (43 us for 1 MB
// of each at 24 + 24 GB/s per compute unit; this loop takes 50 - 54, before 56).  Loaded past the caches the half lines of
// its fragments cost 5 %, so these loads may allocate.  Up to 32 columns: gemm_tiles_lines.
template <int TW>
__device__ __noinline__ void gemm_tiles_wide(const Params &P, const ChunkedArgs *args, float *sm, int *frame_anchor)
{
    const ChunkedArgs a = lds_get_uniform(args);
    if (a.task_id == -0x7FFFFFFF) *frame_anchor = 1;      // never true; see gemm_tiles_chunked
    const GemmTile &g = a.g;
    const Epilogue &e = a.e;
    const TaskWaits &w = a.w;
    const int task_id = a.task_id;
    constexpr int NB = 4, KH = 2;                  // column blocks of 16; wavefronts per row group
    constexpr int COLS = 16 * NB, KC = 256, KS = KC / 32, STRIDE = KC + 8;
    constexpr int PPC = KC / 8;                    // 16-byte pieces per column and half
    constexpr int U = COLS * PPC / kWgThreads;     // pieces per thread, chunk and half
    constexpr int BUF = 2 * COLS * STRIDE;         // elements of one operand buffer: hi columns, then lo columns
    constexpr int PASS = kWaves / KH * TW;         // row tiles per pass
    constexpr int KSW = KS / KH;                   // k steps of a chunk that one wavefront takes: kh * KSW on (whole 128-byte lines)
    constexpr int RD = KSW * TW >= 16 ? 1 : 16 / (KSW * TW);      // chunks of weights in flight
    constexpr int RING = KSW * TW * RD;            // weight fragments in flight per lane
    constexpr int NCOL = COLS < 64 ? 64 : COLS, GRPS = kWgThreads / NCOL;      // norm factors: threads (column, group)
    static_assert(TW == 2 || TW == 4, "tiles per pair of wavefronts");
    static_assert(U >= 1 && COLS * PPC == U * kWgThreads && RD <= 2, "every thread moves U pieces of each half");
    static_assert((size_t)2 * BUF * 2 + (NCOL + kWgThreads) * 4 <= (size_t)kLdsBytes, "two operand buffers and the norm scratch fit");
    static_assert((size_t)PASS * NB * 256 * 4 <= (size_t)2 * BUF * 2, "the tiles' accumulators alias the operand buffers");
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int rg = wave / KH, kh = wave % KH;      // row group and share of K of this wavefront
    const int m = lane & 15, kg = lane >> 4;
    const int K = __builtin_amdgcn_readfirstlane(g.K);
    const int n_chunks = K / KC;                   // K is a multiple of 256
    const int n_tiles = __builtin_amdgcn_readfirstlane(g.n_tiles);      // <= PASS
    const size_t tile_step = (size_t)g.tile_rows * (size_t)g.ldw;
    const uint16_t *wbase = (m < 8 ? g.rowsA + (size_t)m * (size_t)g.ldw : g.rowsB + (size_t)(m - 8) * (size_t)g.ldw) + kg * 8 + kh * (KSW * 32);
    // a wavefront whose tile lies beyond n_tiles streams the last live tile again and never stores it: no branch in the loop
    uint32_t toff[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t) {
        const int ti = rg * TW + t;
        toff[t] = __builtin_amdgcn_readfirstlane((uint32_t)((size_t)(ti < n_tiles ? ti : n_tiles - 1) * tile_step));
    }
    ETC_AS_LDS uint16_t *buf0 = reinterpret_cast<ETC_AS_LDS uint16_t *>(as_lds(sm));
    ETC_AS_LDS float *tb = as_lds(sm);                                    // after the last chunk: [PASS][NB][64 lanes][4]
    ETC_AS_LDS float *rs = reinterpret_cast<ETC_AS_LDS float *>(buf0 + 2 * BUF);
    ETC_AS_LDS float *rs_part = rs + NCOL;                                // [GRPS][NCOL]

    // ---- weight prefetch before the wait: the fragments of the first RD chunks -------------------------------
    u32x4 wr[RING];
#pragma unroll
    for (int j = 0; j < RING; ++j) {
        const int k = (j / TW / KSW) * KC + (j / TW % KSW) * 32;               // beyond K (one chunk, two in the ring): the last one again, never used
        wr[j] = gld_16B(wbase + toff[j % TW] + (RD == 1 || k < K ? k : 0));
    }
    if (w.per_wave) {
        if (wave == 0 && lane < kWaves) spin_until_zero(P, w.ev0 + lane, w.fn);
        if (wave_id() == 0) spin_event(P, w.ev1, w.fn);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
        wg_wait(P, w.ev0, w.ev1, w.fn);
    }
    trace_mark(P, task_id, 1);

    const __amdgpu_buffer_rsrc_t hi_b = buf_of(g.b_hi), lo_b = buf_of(g.b_lo);
    uint32_t off[U];                               // byte offset of this thread's pieces in chunk 0
    const int pc = (int)threadIdx.x % PPC;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
        int row = 0;
        if (col < g.n_cols) row = g.col_rows ? ld_i32(g.col_rows + col) : col;
        if (row < 0) row = 0;
        off[u] = col < g.n_cols ? ((uint32_t)row * (uint32_t)g.ldb + (uint32_t)pc * 8u) * 2u : kBufNone;
    }
    u32x4 vh[U], vl[U];                            // pieces of the next chunk in flight
    auto fetch_chunk = [&](int c) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vh[u] = buf_ld_16B(hi_b, off[u], (uint32_t)c * (KC * 2));
            vl[u] = buf_ld_16B(lo_b, off[u], (uint32_t)c * (KC * 2));
        }
    };
    auto park_chunk = [&](int b) {
        ETC_AS_LDS uint16_t *hi = buf0 + b * BUF, *lo = hi + COLS * STRIDE;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
            *reinterpret_cast<ETC_AS_LDS u32x4 *>(hi + col * STRIDE + pc * 8) = vh[u];
            *reinterpret_cast<ETC_AS_LDS u32x4 *>(lo + col * STRIDE + pc * 8) = vl[u];
        }
    };
    fetch_chunk(0);
    if (g.ssq_parts) {       // RMSNorm factors, as in the chunked path
        const int col = (int)threadIdx.x % NCOL, grp = (int)threadIdx.x / NCOL;
        int row = -1;
        if (col < g.n_cols) row = g.col_rows ? ld_i32(g.col_rows + col) : col;
        float s = 0.f;
        for (int p0 = grp; p0 < g.n_parts; p0 += GRPS * 16) {
            float t[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int pt = p0 + GRPS * j;
                t[j] = (pt < g.n_parts && row >= 0) ? ld_f32(g.ssq_parts + (size_t)pt * (size_t)g.ssq_stride + row) : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) s += t[j];
        }
        rs_part[grp * NCOL + col] = s;
    }
    park_chunk(0);
    __syncthreads();
    if (g.ssq_parts && threadIdx.x < NCOL) {
        float s = 0.f;
#pragma unroll
        for (int gq = 0; gq < GRPS; ++gq) s += rs_part[gq * NCOL + threadIdx.x];
        rs[threadIdx.x] = 1.0f / sqrtf(s / (float)g.K + g.eps);
    }
    trace_mark(P, task_id, 2);

    f32x4 acc[TW][NB];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[t][nb] = f32x4{0, 0, 0, 0};
    // Chunk c out of ring part r: KS steps of 32 elements of K, hi and lo products in turn.  RELOAD: a slot is refilled for
    // chunk c + RD behind its use.  The scheduling barriers keep the order as written: left to itself the compiler sinks
    // the loads of the next chunk to the end of this one, next to their use, and the LDS reads to the products that need
    // them; here the fragments of the next half step are read while the products of this one run.
#define ETC_WIDE_CHUNK(c, r, RELOAD)                                                                              \
    {                                                                                                             \
        ETC_AS_LDS const uint16_t *hi = buf0 + ((c) & 1) * BUF + m * STRIDE + kg * 8 + kh * (KSW * 32);                             \
        ETC_AS_LDS const uint16_t *lo = hi + COLS * STRIDE;                                                       \
        u32x4 fh[NB], fl[NB];                                                                                     \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                         \
            fh[nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(hi + nb * 16 * STRIDE);                          \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        _Pragma("unroll") for (int kk = 0; kk < KSW; ++kk) {                                                       \
            _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                     \
                fl[nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(lo + nb * 16 * STRIDE + kk * 32);             \
            _Pragma("unroll") for (int t = 0; t < TW; ++t) {                                                      \
                const bf16x8 av = __builtin_bit_cast(bf16x8, wr[((r) * KSW + kk) * TW + t]);                       \
                _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) acc[t][nb] =                                    \
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, fh[nb]), acc[t][nb], 0, 0, 0); \
            }                                                                                                     \
            __builtin_amdgcn_sched_barrier(0);                                                                    \
            if (kk + 1 < KSW) {                                                                                    \
                _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                 \
                    fh[nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(hi + nb * 16 * STRIDE + (kk + 1) * 32);   \
            }                                                                                                     \
            _Pragma("unroll") for (int t = 0; t < TW; ++t) {                                                      \
                const int j = ((r) * KSW + kk) * TW + t;                                                           \
                const bf16x8 av = __builtin_bit_cast(bf16x8, wr[j]);                                              \
                _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) acc[t][nb] =                                    \
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, fl[nb]), acc[t][nb], 0, 0, 0); \
            }                                                                                                     \
            __builtin_amdgcn_sched_barrier(0);                                                                    \
            if (RELOAD) {                                                                                         \
                _Pragma("unroll") for (int t = 0; t < TW; ++t) wr[((r) * KSW + kk) * TW + t] =                     \
                    gld_16B(wbase + toff[t] + (size_t)((c) + RD) * KC + kk * 32);                                \
            }                                                                                                     \
        }                                                                                                         \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
    }
    // one chunk of parity p: request the next chunk's operand, compute, park it
#define ETC_WIDE_STEP(c, p, FETCH, RELOAD, PARK)                                                                  \
    {                                                                                                             \
        if (FETCH) fetch_chunk((c) + 1);                                                                          \
        ETC_WIDE_CHUNK(c, (p) % RD, RELOAD)                                                                       \
        if (PARK) {                                                                                               \
            park_chunk(((p) + 1) & 1);                                                                            \
            __syncthreads();                                                                                      \
        }                                                                                                         \
    }
    int c = 0;
    if constexpr (RD == 1) {
        for (; c + 1 < n_chunks; ++c) {            // steady state: the next chunk exists
            fetch_chunk(c + 1);
            ETC_WIDE_CHUNK(c, 0, true)
            park_chunk((c + 1) & 1);
            __syncthreads();
        }
        ETC_WIDE_CHUNK(c, 0, false)
    } else {
        for (; c + 4 <= n_chunks; c += 2) {        // steady state: everything ahead exists; c is even
            ETC_WIDE_STEP(c, 0, true, true, true)
            ETC_WIDE_STEP(c + 1, 1, true, true, true)
        }
        if (n_chunks - c == 3) {
            ETC_WIDE_STEP(c, 0, true, true, true)
            ETC_WIDE_STEP(c + 1, 1, true, false, true)
            ETC_WIDE_STEP(c + 2, 0, false, false, false)
        } else if (n_chunks - c == 2) {
            ETC_WIDE_STEP(c, 0, true, false, true)
            ETC_WIDE_STEP(c + 1, 1, false, false, false)
        } else {
            ETC_WIDE_STEP(c, 0, false, false, false)
        }
    }
#undef ETC_WIDE_STEP
#undef ETC_WIDE_CHUNK
    trace_mark(P, task_id, 3);

    // ---- the two wavefronts of a row group hold sums over half of K each; each finishes half of the tiles ----
    constexpr int TF = TW / KH;                    // tiles a wavefront finishes: rg * TW + kh * TF + t
    f32x4 sum[TF][NB];
    __syncthreads();                           // every wavefront is done with the operand buffers
#pragma unroll
    for (int t = 0; t < TF; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            *reinterpret_cast<ETC_AS_LDS f32x4 *>(tb + ((size_t)((wave * TF + t) * NB + nb) * 64 + lane) * 4) = kh ? acc[t][nb] : acc[TF + t][nb];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TF; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            sum[t][nb] = (kh ? acc[TF + t][nb] : acc[t][nb]) +
                         *reinterpret_cast<ETC_AS_LDS const f32x4 *>(tb + ((size_t)(((wave ^ 1) * TF + t) * NB + nb) * 64 + lane) * 4);
    if (epilogue_is_direct(e.kind)) {
#pragma unroll
        for (int t = 0; t < TF; ++t) {
            const int ti = rg * TW + kh * TF + t;
            if (ti < n_tiles) epilogue_direct<NB>(e, e.row0 + ti * g.tile_rows, g.n_cols, sum[t], rs, g.ssq_parts != nullptr);
        }
        __syncthreads();                           // the next pass parks its operand over these buffers
        return;
    }
    // ---- sums through LDS into the layout of the epilogue threads, then the epilogue tile by tile ----
    __syncthreads();                               // the exchanged halves have been read
#pragma unroll
    for (int t = 0; t < TF; ++t) {
        const int ti = rg * TW + kh * TF + t;
        if (ti < n_tiles) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                *reinterpret_cast<ETC_AS_LDS f32x4 *>(tb + ((size_t)(ti * NB + nb) * 64 + lane) * 4) = sum[t][nb];
        }
    }
    tiles_epilogue<NB>(P, a, tb, rs, rs_part, n_tiles);
}

// The wide path for up to 32 columns (NG groups of 8), with whole lines of weights per load (see unit_row): the same split
// of the output over the wavefronts and the same operand buffers, but a ring entry is 8 rows x one unit of K, streamed
// non-temporally, and the products run on 8 columns each.  Twice the matrix instructions (12 us of a 35 us gate/up stage
// at 32 columns), which is why 64 columns stay with the fragments above.
template <int TW, int NG>
__device__ __noinline__ void gemm_tiles_lines(const Params &P, const ChunkedArgs *args, float *sm, int *frame_anchor)
{
    const ChunkedArgs a = lds_get_uniform(args);
    if (a.task_id == -0x7FFFFFFF) *frame_anchor = 1;      // never true; see gemm_tiles_chunked
    const GemmTile &g = a.g;
    const Epilogue &e = a.e;
    constexpr int COLS = 8 * NG, NB = NG / 2, KC = 256, STRIDE = KC + 16;      // 32 bytes more per column: a fragment read hits every bank once
    constexpr int PPC = KC / 8, U = COLS * PPC / kWgThreads, BUF = 2 * COLS * STRIDE;
    constexpr int PASS = kWaves * TW;
    constexpr int KSW = KC / kUnitK;               // units of a chunk
    constexpr int RD = KSW * TW >= 8 ? 1 : 8 / (KSW * TW);      // chunks of weights in flight
    constexpr int RING = KSW * TW * RD * 2;        // loads in flight per lane: rows A and rows B of every unit
    constexpr int FD = NG == 2 ? 2 : 1;            // chunks of the operand in flight, as the registers allow
    static_assert((NG == 2 || NG == 4) && RD <= 2 && U >= 1 && COLS * PPC == U * kWgThreads, "shapes");
    static_assert((size_t)2 * BUF * 2 + (64 + kWgThreads) * 4 <= (size_t)kLdsBytes, "two operand buffers and the norm scratch fit");
    static_assert((size_t)PASS * NB * 256 * 4 <= (size_t)2 * BUF * 2, "the tiles' sums alias the operand buffers");
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int n16 = lane & 15, kg = lane >> 4;
    const int K = __builtin_amdgcn_readfirstlane(g.K), n_chunks = K / KC;
    const int n_tiles = __builtin_amdgcn_readfirstlane(g.n_tiles);
    const size_t tile_step = (size_t)g.tile_rows * (size_t)g.ldw;
    const uint16_t *wA = unit_row(g.rowsA, g.ldw), *wB = unit_row(g.rowsB, g.ldw);
    uint32_t toff[TW];                             // a tile beyond n_tiles streams the last live one again and is never stored
#pragma unroll
    for (int t = 0; t < TW; ++t) {
        const int ti = wave * TW + t;
        toff[t] = __builtin_amdgcn_readfirstlane((uint32_t)((size_t)(ti < n_tiles ? ti : n_tiles - 1) * tile_step));
    }
    ETC_AS_LDS uint16_t *buf0 = reinterpret_cast<ETC_AS_LDS uint16_t *>(as_lds(sm));
    ETC_AS_LDS float *tb = as_lds(sm);             // after the last chunk
    ETC_AS_LDS float *rs = reinterpret_cast<ETC_AS_LDS float *>(buf0 + 2 * BUF), *rs_part = rs + 64;

    u32x4 wr[RING];
#pragma unroll
    for (int j = 0; j < RING / 2; ++j) {           // ring entry (chunk, unit, tile)
        const int k = (j / TW / KSW) * KC + (j / TW % KSW) * kUnitK;
        const uint32_t o = toff[j % TW] + (uint32_t)(RD == 1 || k < K ? k : 0);      // beyond K (one chunk, two in the ring): never used
        wr[2 * j] = load16_nt(wA + o);
        wr[2 * j + 1] = load16_nt(wB + o);
    }
    gemm_wait(P, a.w);
    trace_mark(P, a.task_id, 1);

    const __amdgpu_buffer_rsrc_t hi_b = buf_of(g.b_hi), lo_b = buf_of(g.b_lo);
    uint32_t off[U];
    const int pc = (int)threadIdx.x % PPC;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
        int row = 0;
        if (col < g.n_cols) row = g.col_rows ? ld_i32(g.col_rows + col) : col;
        if (row < 0) row = 0;
        off[u] = col < g.n_cols ? ((uint32_t)row * (uint32_t)g.ldb + (uint32_t)pc * 8u) * 2u : kBufNone;
    }
    u32x4 vh[FD][U], vl[FD][U];
    auto fetch_chunk = [&](int c, u32x4 (&h)[U], u32x4 (&l)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            h[u] = buf_ld_16B(hi_b, off[u], (uint32_t)c * (KC * 2));
            l[u] = buf_ld_16B(lo_b, off[u], (uint32_t)c * (KC * 2));
        }
    };
    auto park_chunk = [&](int b, const u32x4 (&h)[U], const u32x4 (&l)[U]) {
        ETC_AS_LDS uint16_t *hi = buf0 + b * BUF, *lo = hi + COLS * STRIDE;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
            *reinterpret_cast<ETC_AS_LDS u32x4 *>(hi + col * STRIDE + pc * 8) = h[u];
            *reinterpret_cast<ETC_AS_LDS u32x4 *>(lo + col * STRIDE + pc * 8) = l[u];
        }
    };
    fetch_chunk(0, vh[0], vl[0]);
    if (FD == 2 && n_chunks > 1) fetch_chunk(1, vh[FD - 1], vl[FD - 1]);
    if (g.ssq_parts) norm_shares<64>(g, rs_part);
    park_chunk(0, vh[0], vl[0]);
    __syncthreads();
    if (g.ssq_parts) norm_factors<64>(g, rs, rs_part);        // read behind the barrier after the last chunk
    trace_mark(P, a.task_id, 2);

    f32x4 acc[TW][2][NG];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) acc[t][0][ng] = acc[t][1][ng] = f32x4{0, 0, 0, 0};
    // chunk c out of ring part r, in the order as written (see ETC_WIDE_CHUNK)
#define ETC_LINES_CHUNK(c, r, RELOAD)                                                                             \
    {                                                                                                             \
        ETC_AS_LDS const uint16_t *hi = buf0 + ((c) & 1) * BUF + (n16 >> 1) * STRIDE + (kg * 2 + (n16 & 1)) * 8; \
        ETC_AS_LDS const uint16_t *lo = hi + COLS * STRIDE;                                                       \
        u32x4 fh[NG], fl[NG];                                                                                     \
        _Pragma("unroll") for (int ng = 0; ng < NG; ++ng)                                                         \
            fh[ng] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(hi + ng * 8 * STRIDE);                           \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        _Pragma("unroll") for (int kk = 0; kk < KSW; ++kk) {                                                      \
            _Pragma("unroll") for (int ng = 0; ng < NG; ++ng)                                                     \
                fl[ng] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(lo + ng * 8 * STRIDE + kk * kUnitK);          \
            _Pragma("unroll") for (int t = 0; t < TW; ++t)                                                        \
                _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                   \
                    const bf16x8 av = __builtin_bit_cast(bf16x8, wr[(((r) * KSW + kk) * TW + t) * 2 + h]);        \
                    _Pragma("unroll") for (int ng = 0; ng < NG; ++ng) acc[t][h][ng] =                             \
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, fh[ng]), acc[t][h][ng], 0, 0, 0); \
                }                                                                                                 \
            __builtin_amdgcn_sched_barrier(0);                                                                    \
            if (kk + 1 < KSW) {                                                                                   \
                _Pragma("unroll") for (int ng = 0; ng < NG; ++ng)                                                 \
                    fh[ng] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(hi + ng * 8 * STRIDE + (kk + 1) * kUnitK); \
            }                                                                                                     \
            _Pragma("unroll") for (int t = 0; t < TW; ++t)                                                        \
                _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                   \
                    const bf16x8 av = __builtin_bit_cast(bf16x8, wr[(((r) * KSW + kk) * TW + t) * 2 + h]);        \
                    _Pragma("unroll") for (int ng = 0; ng < NG; ++ng) acc[t][h][ng] =                             \
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, fl[ng]), acc[t][h][ng], 0, 0, 0); \
                }                                                                                                 \
            __builtin_amdgcn_sched_barrier(0);                                                                    \
            if (RELOAD) {                                                                                         \
                _Pragma("unroll") for (int t = 0; t < TW; ++t) {                                                  \
                    const int j = (((r) * KSW + kk) * TW + t) * 2;                                                \
                    const size_t o = toff[t] + (size_t)((c) + RD) * KC + kk * kUnitK;                             \
                    wr[j] = load16_nt(wA + o);                                                                    \
                    wr[j + 1] = load16_nt(wB + o);                                                                \
                }                                                                                                 \
            }                                                                                                     \
        }                                                                                                         \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
    }
    // one chunk of parity p: request the operand FD chunks ahead, compute, park the next chunk's operand
#define ETC_LINES_STEP(c, p, FETCH, RELOAD, PARK)                                                                 \
    {                                                                                                             \
        if (FETCH) fetch_chunk((c) + FD, vh[(p) % FD], vl[(p) % FD]);                                             \
        ETC_LINES_CHUNK(c, (p) % RD, RELOAD)                                                                      \
        if (PARK) {                                                                                               \
            park_chunk((p) ^ 1, vh[((p) + 1) % FD], vl[((p) + 1) % FD]);                                          \
            __syncthreads();                                                                                      \
        }                                                                                                         \
    }
    int c = 0;
    if constexpr (RD == 1 && FD == 1) {
        for (; c + 1 < n_chunks; ++c) {            // steady state: the next chunk exists
            fetch_chunk(c + 1, vh[0], vl[0]);
            ETC_LINES_CHUNK(c, 0, true)
            park_chunk((c + 1) & 1, vh[0], vl[0]);
            __syncthreads();
        }
        ETC_LINES_CHUNK(c, 0, false)
    } else {
        for (; c + 4 <= n_chunks; c += 2) {        // steady state: everything ahead exists; c is even
            ETC_LINES_STEP(c, 0, true, true, true)
            ETC_LINES_STEP(c + 1, 1, true, true, true)
        }
        if (n_chunks - c == 3) {
            ETC_LINES_STEP(c, 0, true, true, true)
            ETC_LINES_STEP(c + 1, 1, FD == 1, RD == 1, true)
            ETC_LINES_STEP(c + 2, 0, false, false, false)
        } else if (n_chunks - c == 2) {
            ETC_LINES_STEP(c, 0, FD == 1, RD == 1, true)
            ETC_LINES_STEP(c + 1, 1, false, false, false)
        } else {
            ETC_LINES_STEP(c, 0, false, false, false)
        }
    }
#undef ETC_LINES_STEP
#undef ETC_LINES_CHUNK
    trace_mark(P, a.task_id, 3);

    // ---- sums: lane (n16, kg) has rows 2 kg, 2 kg + 1 of group n16 % 2 for column ng * 8 + n16 / 2 ----
    float v[TW][NG][2];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) unit_sums(acc[t][0][ng], acc[t][1][ng], v[t][ng]);
    __syncthreads();                               // every wavefront is done with the operand buffers
    if (epilogue_is_direct(e.kind)) {
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            const int ti = wave * TW + t;
            if (ti < n_tiles) epilogue_direct_units<NG>(e, e.row0 + ti * g.tile_rows, g.n_cols, v[t], rs, g.ssq_parts != nullptr);
        }
        __syncthreads();                           // the next pass parks its operand over these buffers
        return;
    }
    // ---- the other epilogues, tile by tile from LDS: [tile][column block][row / 4][column][row % 4] ----
#pragma unroll
    for (int t = 0; t < TW; ++t) {
        const int ti = wave * TW + t, r = (n16 & 1) * 8 + 2 * kg;
        if (ti < n_tiles) {
#pragma unroll
            for (int ng = 0; ng < NG; ++ng) {
                const int n = (ng & 1) * 8 + (n16 >> 1);
                ETC_AS_LDS float *dst = tb + (size_t)(ti * NB + (ng >> 1)) * 256 + ((r >> 2) * 16 + n) * 4 + (r & 3);
                dst[0] = v[t][ng][0];
                dst[1] = v[t][ng][1];
            }
        }
    }
    tiles_epilogue<NB>(P, a, tb, rs, rs_part, n_tiles);
}

// ---- GroupGEMM paths (row blocks of the MoE block: EPI_MOE_ACT, EPI_MOE_Y) -----------------------------------------
// Up to 16 columns, 8 or more row tiles that do not fit the staged path: the whole operand sits in LDS (64 KB for 8 columns of K = 2048) and every
// wavefront streams row tiles of its own (wave, wave + 8, ...) through all of K: one linear stream of weights with 16
// loads in flight that never drains between tiles, no barrier and no reduction behind the staging, the epilogue straight
// from the accumulators.  Bound by HBM.  The staged path splits K over the wavefronts instead and meets in one reduction
// per task, whose buffer limits a task to 16 tiles at 6 columns: a token block of 100 runs three rounds of 1 MB tasks
// there (wait, staging and reduction three times) and one round of 3 MB tasks here.
template <int NG>
__device__ __noinline__ void gemm_tiles_stream(const Params &P, const ChunkedArgs *args, float *sm, int *frame_anchor)
{
    const ChunkedArgs a = lds_get_uniform(args);
    if (a.task_id == -0x7FFFFFFF) *frame_anchor = 1;      // never true; see gemm_tiles_chunked
    const GemmTile &g = a.g;
    const Epilogue &e = a.e;
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int n16 = lane & 15, kg = lane >> 4;
    const int K = __builtin_amdgcn_readfirstlane(g.K), n_tiles = __builtin_amdgcn_readfirstlane(g.n_tiles);
    const int upt = K >> 8;                        // steps of 4 units (256 elements of K) per tile
    const int total = n_tiles > wave ? (n_tiles - wave + kWaves - 1) / kWaves * upt : 0;      // steps of this wavefront
    const size_t tile_step = (size_t)g.tile_rows * (size_t)g.ldw;
    const uint16_t *ipA = unit_row(g.rowsA, g.ldw) + (size_t)wave * tile_step;      // next step to request
    const uint16_t *ipB = unit_row(g.rowsB, g.ldw) + (size_t)wave * tile_step;
    const long long tile_jump = (long long)(kWaves * tile_step) - (long long)K;
    int iu = 0;                                    // its place in its tile
    auto next_step = [&]() {
        const bool wrap = ++iu == upt;
        const long long by = 256 + (wrap ? tile_jump : 0);
        ipA += by;
        ipB += by;
        iu = wrap ? 0 : iu;
    };
    u32x4 wr[16];                                  // two steps of 4 units, rows A and rows B of each
    auto request_weights = [&]() {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h < total) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    wr[h * 8 + 2 * j] = gld_16B_nt(ipA + j * kUnitK);
                    wr[h * 8 + 2 * j + 1] = gld_16B_nt(ipB + j * kUnitK);
                }
                next_step();
            }
        }
    };
    // ---- the operand, hi and lo, whole; its columns K + kOpPad elements apart ----------------------------------
    const int Kp = K + kOpPad, ppc = K >> 3, pieces = g.n_cols * ppc;       // 16-byte pieces
    ETC_AS_LDS float *rs = as_lds(sm), *rs_part = rs + 64;
    ETC_AS_LDS uint16_t *op_hi = reinterpret_cast<ETC_AS_LDS uint16_t *>(rs_part + kWgThreads), *op_lo = op_hi + (size_t)g.n_cols * Kp;
    const __amdgpu_buffer_rsrc_t hi_b = buf_of(g.b_hi), lo_b = buf_of(g.b_lo);
    constexpr int U = 4;
    u32x4 vh[U], vl[U];
    uint32_t at[U];
    int i0 = threadIdx.x;
    auto load_pieces = [&](auto row_of) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kWgThreads;
            const int col = i < pieces ? i / ppc : 0, pc = i - col * ppc;
            at[u] = (uint32_t)(col * Kp + pc * 8);
            const uint32_t off = i < pieces ? ((uint32_t)row_of(col) * (uint32_t)g.ldb + (uint32_t)pc * 8u) * 2u : kBufNone;
            vh[u] = buf_ld_16B(hi_b, off, 0);
            vl[u] = buf_ld_16B(lo_b, off, 0);
        }
    };
    auto store_pieces = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * kWgThreads < pieces) {
                *reinterpret_cast<ETC_AS_LDS u32x4 *>(op_hi + at[u]) = vh[u];
                *reinterpret_cast<ETC_AS_LDS u32x4 *>(op_lo + at[u]) = vl[u];
            }
        }
    };
    auto whole_operand = [&](auto row_of, auto behind) {
        for (int left = pieces; left > U * kWgThreads; left -= U * kWgThreads) {
            load_pieces(row_of);
            store_pieces();
            i0 += U * kWgThreads;
        }
        load_pieces(row_of);
        behind();
        store_pieces();
    };
    if (e.kind == EPI_MOE_ACT) {                   // its events have been seen (the rows depend on the routing): operand ahead of the weights
        const int col_row = norm_row<64>(g);       // of column `lane`
        float t[16];
        whole_operand([&](int col) { return max(__shfl(col_row, col, 64), 0); }, [&]() {
            norm_request<64>(g, col_row, t);
            request_weights();
        });
        norm_shares<64>(g, col_row, t, rs_part);
        trace_mark(P, a.task_id, 1);
    } else {                                       // the activations of its own row block: rows as they stand
        request_weights();
        gemm_wait(P, a.w);
        trace_mark(P, a.task_id, 1);
        whole_operand([](int col) { return col; }, []() {});
    }
    __syncthreads();
    if (g.ssq_parts) {
        norm_factors<64>(g, rs, rs_part);
        __syncthreads();
    }
    trace_mark(P, a.task_id, 2);

    ETC_AS_LDS const uint16_t *sh[NG], *sl[NG];    // columns beyond n_cols read column 0's operand and are never stored
#pragma unroll
    for (int ng = 0; ng < NG; ++ng) {
        const int col = ng * 8 + (n16 >> 1), c = col < g.n_cols ? col : 0;
        sh[ng] = op_hi + (size_t)c * Kp + (kg * 2 + (n16 & 1)) * 8;
        sl[ng] = op_lo + (size_t)c * Kp + (kg * 2 + (n16 & 1)) * 8;
    }
    f32x4 accA[NG], accB[NG];
#pragma unroll
    for (int ng = 0; ng < NG; ++ng) accA[ng] = accB[ng] = f32x4{0, 0, 0, 0};
    int cu = 0, ti = wave;                         // step inside its tile, tile
    auto finish_tile = [&]() {                     // straight from the accumulators
        float v[NG][2];
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) {
            unit_sums(accA[ng], accB[ng], v[ng]);
            accA[ng] = accB[ng] = f32x4{0, 0, 0, 0};
        }
        epilogue_direct_units<NG>(e, e.row0 + ti * g.tile_rows, g.n_cols, v, rs, g.ssq_parts != nullptr);
    };
    // one step out of ring half h; RELOAD: its slots are refilled for the step after the next, behind their use
#define ETC_STREAM_STEP(h, RELOAD)                                                                                \
    {                                                                                                             \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                           \
            const bf16x8 a0 = __builtin_bit_cast(bf16x8, wr[(h) * 8 + 2 * j]), a1 = __builtin_bit_cast(bf16x8, wr[(h) * 8 + 2 * j + 1]); \
            _Pragma("unroll") for (int ng = 0; ng < NG; ++ng) {                                                   \
                const bf16x8 bh = __builtin_bit_cast(bf16x8, *reinterpret_cast<ETC_AS_LDS const u32x4 *>(sh[ng] + cu * 256 + j * kUnitK)); \
                const bf16x8 bl = __builtin_bit_cast(bf16x8, *reinterpret_cast<ETC_AS_LDS const u32x4 *>(sl[ng] + cu * 256 + j * kUnitK)); \
                accA[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bh, accA[ng], 0, 0, 0);                    \
                accB[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bh, accB[ng], 0, 0, 0);                    \
                accA[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bl, accA[ng], 0, 0, 0);                    \
                accB[ng] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bl, accB[ng], 0, 0, 0);                    \
            }                                                                                                     \
            if (RELOAD) {                                                                                         \
                wr[(h) * 8 + 2 * j] = gld_16B_nt(ipA + j * kUnitK);                                               \
                wr[(h) * 8 + 2 * j + 1] = gld_16B_nt(ipB + j * kUnitK);                                           \
                __builtin_amdgcn_sched_barrier(0);                                                                \
            }                                                                                                     \
        }                                                                                                         \
        if (RELOAD) next_step();                                                                                  \
        if (++cu == upt) {                                                                                        \
            finish_tile();                                                                                        \
            cu = 0;                                                                                               \
            ti += kWaves;                                                                                         \
        }                                                                                                         \
    }
    int u = 0;
    for (; u + 4 <= total; u += 2) {
        ETC_STREAM_STEP(0, true)
        ETC_STREAM_STEP(1, true)
    }
    if (total - u == 3) {
        ETC_STREAM_STEP(0, true)
        ETC_STREAM_STEP(1, false)
        ETC_STREAM_STEP(0, false)
    } else if (total - u >= 1) {
        ETC_STREAM_STEP(0, false)
        if (total - u == 2) ETC_STREAM_STEP(1, false)
    }
#undef ETC_STREAM_STEP
    trace_mark(P, a.task_id, 3);
    __syncthreads();                               // the operand in LDS is free again
}
__device__ __forceinline__ bool stream_fits(int n_tiles, int n_cols, int K, int ldb)
{
    return n_cols <= 16 && ldb <= kMaxBufLd && n_tiles >= kWaves && K % 256 == 0 &&
           (long long)(64 + kWgThreads) * 4 + (long long)n_cols * (K + kOpPad) * 4 <= (long long)kLdsBytes;
}

// Row blocks of 33 .. 16 * NB columns (128 at most) against any number of row tiles, 8 * TW per pass (TW per wavefront).
// The operand is walked in chunks through two LDS buffers as in the wide path, but the passes are one stream: the weights
// of the next pass and its first operand chunk are requested while this one ends, and the epilogue needs no LDS, so
// nothing drains between them.  What bounds a large block is bytes through the fabric (40 - 48 GB/s per compute unit) and LDS reads of the
// operand, which every wavefront takes whole; both shrink with the tiles of a pass, so a wavefront takes as many as its
// registers hold (4 x 128 columns: 128 accumulators) and the chunk shrinks instead.
// LINES (not for two tiles per wavefront): weights arrive as whole lines (8 rows x 64 elements of K per load, see unit_row;
// here lane / 8 is the row and lane % 8 the piece) and turn into the product's fragments through 2 KB of LDS per wavefront;
// the ring entry is free for its next load once it is written there.  48 tiles x 64 columns of K = 2048: 185 us with
// fragments loaded as they stand, 161 with whole lines, 126 with whole lines past the caches (NT); the row blocks of an
// expert that has several stream the same rows and find them in the caches, where fragments as they stand do better (32
// tiles x 128 columns: 130 us, through LDS 145).
template <int NB, int TW, bool LINES, bool NT>
__device__ __noinline__ void gemm_tiles_blocks(const Params &P, const ChunkedArgs *args, float *sm, int *frame_anchor)
{
    const ChunkedArgs a = lds_get_uniform(args);
    if (a.task_id == -0x7FFFFFFF) *frame_anchor = 1;      // never true; see gemm_tiles_chunked
    const GemmTile &g = a.g;
    const Epilogue &e = a.e;
    constexpr int PASS = kWaves * TW;
    constexpr int COLS = 16 * NB, KC = (TW == 2 ? 1024 : 512) / NB, KS = KC / 32, STRIDE = KC + 8;
    constexpr int PPC = KC / 8, U = COLS * PPC / kWgThreads, BUF = 2 * COLS * STRIDE;
    constexpr int RING = KS * TW;                  // weight fragments in flight per lane: one chunk
    constexpr int NBH = 4;                         // column blocks of one operand read
    constexpr int NCOL = NB == 4 ? 64 : 128;       // norm factors: threads (column, group)
    constexpr int UNITS = KC / kUnitK;             // LINES: units of a chunk; a ring entry pair is rows A and rows B of one
    static_assert((NB == 4 || NB == 8) && TW >= 2 && TW <= 4 && (!LINES || TW > 2), "column blocks, tiles per wavefront");
    static_assert(U >= 1 && COLS * PPC == U * kWgThreads, "every thread moves U pieces of each half");
    static_assert((size_t)2 * BUF * 2 + (NCOL + kWgThreads) * 4 + (LINES ? kWaves * 2048 : 0) <= (size_t)kLdsBytes, "two operand buffers, the norm scratch and the fragments fit");
    const int wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
    const int m = lane & 15, kg = lane >> 4;
    const int n_tiles = __builtin_amdgcn_readfirstlane(g.n_tiles);
    const int n_chunks = __builtin_amdgcn_readfirstlane(g.K) / KC;
    const int total = (n_tiles + PASS - 1) / PASS * n_chunks;
    const uint32_t tile_step = (uint32_t)g.tile_rows * (uint32_t)g.ldw;
    const uint16_t *wbase = LINES ? g.rowsA + (size_t)(lane >> 3) * (size_t)g.ldw + (lane & 7) * 8
                                  : (m < 8 ? g.rowsA + (size_t)m * (size_t)g.ldw : g.rowsB + (size_t)(m - 8) * (size_t)g.ldw) + kg * 8;
    const uint16_t *wbaseB = LINES ? g.rowsB + (size_t)(lane >> 3) * (size_t)g.ldw + (lane & 7) * 8 : wbase;
    auto load_w = [&](const uint16_t *p) { return NT ? gld_16B_nt(p) : gld_16B(p); };
    // request cursor of the weights: chunk rc of the pass whose first tile of this wavefront is rt (tiles beyond the task
    // stream its last one again and are never stored: no branch in the loop)
    int rc = 0, rt = wave * TW;
    size_t ro[TW];
    auto set_offsets = [&]() {
#pragma unroll
        for (int t = 0; t < TW; ++t) ro[t] = (size_t)(rt + t < n_tiles ? rt + t : n_tiles - 1) * tile_step + (size_t)rc * KC;
    };
    auto next_request = [&]() {
        if (++rc == n_chunks) { rc = 0; rt += PASS; }
        set_offsets();
    };
    set_offsets();
    u32x4 wr[RING];
    auto request_weights = [&]() {
#pragma unroll
        for (int j = 0; j < RING; ++j) {
            if constexpr (LINES) wr[j] = load_w((j & 1 ? wbaseB : wbase) + ro[j / 2 % TW] + (j / 2 / TW) * kUnitK);
            else wr[j] = load_w(wbase + ro[j % TW] + (j / TW) * 32);
        }
        next_request();
    };
    ETC_AS_LDS uint16_t *buf0 = reinterpret_cast<ETC_AS_LDS uint16_t *>(as_lds(sm));
    ETC_AS_LDS float *rs = reinterpret_cast<ETC_AS_LDS float *>(buf0 + 2 * BUF), *rs_part = rs + NCOL;
    ETC_AS_LDS char *turn = reinterpret_cast<ETC_AS_LDS char *>(rs_part + kWgThreads) + wave * 2048;      // LINES: [16 rows][8 pieces], piece p of row r at p ^ (r & 7)
    const __amdgpu_buffer_rsrc_t hi_b = buf_of(g.b_hi), lo_b = buf_of(g.b_lo);
    uint32_t off[U];
    const int pc = (int)threadIdx.x % PPC;
    auto operand_rows = [&](const int (&row)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
            off[u] = col < g.n_cols ? ((uint32_t)row[u] * (uint32_t)g.ldb + (uint32_t)pc * 8u) * 2u : kBufNone;
        }
    };
    u32x4 vh[U], vl[U];
    auto fetch_chunk = [&](int c) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vh[u] = buf_ld_16B(hi_b, off[u], (uint32_t)c * (KC * 2));
            vl[u] = buf_ld_16B(lo_b, off[u], (uint32_t)c * (KC * 2));
        }
    };
    auto park_chunk = [&](int b) {
        ETC_AS_LDS uint16_t *hi = buf0 + b * BUF, *lo = hi + COLS * STRIDE;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
            *reinterpret_cast<ETC_AS_LDS u32x4 *>(hi + col * STRIDE + pc * 8) = vh[u];
            *reinterpret_cast<ETC_AS_LDS u32x4 *>(lo + col * STRIDE + pc * 8) = vl[u];
        }
    };
    int row[U];
    if (e.kind == EPI_MOE_ACT) {                   // its events have been seen (the rows depend on the routing): operand ahead of the weights
        const int n_row = norm_row<NCOL>(g);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = ((int)threadIdx.x + kWgThreads * u) / PPC;
            row[u] = max(ld_i32(g.col_rows + (col < g.n_cols ? col : g.n_cols - 1)), 0);
        }
        float t[16];
        operand_rows(row);
        fetch_chunk(0);
        norm_request<NCOL>(g, n_row, t);
        request_weights();
        park_chunk(0);
        norm_shares<NCOL>(g, n_row, t, rs_part);
        trace_mark(P, a.task_id, 1);
    } else {                                       // the activations of its own row block: rows as they stand
        request_weights();
        gemm_wait(P, a.w);
        trace_mark(P, a.task_id, 1);
#pragma unroll
        for (int u = 0; u < U; ++u) row[u] = ((int)threadIdx.x + kWgThreads * u) / PPC;
        operand_rows(row);
        fetch_chunk(0);
        park_chunk(0);
    }
    __syncthreads();
    if (g.ssq_parts) norm_factors<NCOL>(g, rs, rs_part);      // read behind at least one more barrier (n_chunks > 1) ...
    if (g.ssq_parts && total == 1) __syncthreads();           // ... or this one
    trace_mark(P, a.task_id, 2);

    f32x4 acc[TW][NB];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[t][nb] = f32x4{0, 0, 0, 0};
    };
    clear();
    int ti0 = wave * TW;                           // this wavefront's first tile of the pass being computed
    auto finish_pass = [&]() {
#pragma unroll
        for (int t = 0; t < TW; ++t)
            if (ti0 + t < n_tiles)
                epilogue_direct<NB>(e, e.row0 + (ti0 + t) * g.tile_rows, g.n_cols, acc[t], rs, g.ssq_parts != nullptr);
    };
    // One chunk out of LDS buffer b, in the order as written (see ETC_WIDE_CHUNK): per step of 32 elements of K hi, then lo,
    // of NBH column blocks at a time; the fragments of the next read are requested ahead of this one's products.
    // frag(t, kk): the weight fragment of step kk of the chunk.
#define ETC_BLOCK_READS(b, k0, nk, FRAG, BEHIND)      /* steps k0 .. k0 + nk */                                   \
    {                                                                                                             \
        ETC_AS_LDS const uint16_t *op = buf0 + (b) * BUF + m * STRIDE + kg * 8 + (k0) * 32;                       \
        constexpr int NP = NB / NBH, READS = (nk) * NP * 2;                                                       \
        u32x4 f[2][NBH];                                                                                          \
        _Pragma("unroll") for (int nb = 0; nb < NBH; ++nb)                                                        \
            f[0][nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(op + nb * 16 * STRIDE);                        \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        _Pragma("unroll") for (int q = 0; q < READS; ++q) {      /* q = (step, column part, hi / lo) */           \
            const int kk = q / (2 * NP), part = q / 2 % NP, qn = q + 1;                                           \
            if (qn < READS) {                                                                                     \
                _Pragma("unroll") for (int nb = 0; nb < NBH; ++nb) f[qn & 1][nb] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>( \
                    op + (qn & 1) * (COLS * STRIDE) + ((qn / 2 % NP) * NBH + nb) * 16 * STRIDE + (qn / (2 * NP)) * 32); \
            }                                                                                                     \
            _Pragma("unroll") for (int t = 0; t < TW; ++t) {                                                      \
                const bf16x8 av = __builtin_bit_cast(bf16x8, FRAG);                                               \
                _Pragma("unroll") for (int nb = 0; nb < NBH; ++nb) acc[t][part * NBH + nb] =                      \
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, f[q & 1][nb]), acc[t][part * NBH + nb], 0, 0, 0); \
            }                                                                                                     \
            __builtin_amdgcn_sched_barrier(0);                                                                    \
            if (q % (2 * NP) == 2 * NP - 1) BEHIND                                                                \
        }                                                                                                         \
    }
#define ETC_BLOCK_CHUNK(b, RELOAD)                                                                                \
    if constexpr (LINES) {                                                                                        \
        _Pragma("unroll") for (int un = 0; un < UNITS; ++un) {                                                    \
            u32x4 fr[TW][2];                                                                                      \
            _Pragma("unroll") for (int t = 0; t < TW; ++t) {      /* lines in, fragments out: in order within the wavefront */ \
                const int j = (un * TW + t) * 2;                                                                  \
                *reinterpret_cast<ETC_AS_LDS u32x4 *>(turn + lane_line) = wr[j];                                  \
                *reinterpret_cast<ETC_AS_LDS u32x4 *>(turn + 1024 + lane_line) = wr[j + 1];                       \
                fr[t][0] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(turn + lane_frag0);                        \
                fr[t][1] = *reinterpret_cast<ETC_AS_LDS const u32x4 *>(turn + lane_frag1);                        \
                if (RELOAD) {                                                                                     \
                    wr[j] = load_w(wbase + ro[t] + un * kUnitK);                                                  \
                    wr[j + 1] = load_w(wbaseB + ro[t] + un * kUnitK);                                             \
                }                                                                                                 \
            }                                                                                                     \
            ETC_BLOCK_READS(b, un * 2, 2, fr[t][kk], {})                                                          \
        }                                                                                                         \
        if (RELOAD) next_request();                                                                               \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
    } else {                                                                                                      \
        ETC_BLOCK_READS(b, 0, KS, wr[kk * TW + t], {                                                              \
            if (RELOAD) {                                                                                         \
                _Pragma("unroll") for (int t = 0; t < TW; ++t) wr[kk * TW + t] = load_w(wbase + ro[t] + kk * 32); \
            }                                                                                                     \
        })                                                                                                        \
        if (RELOAD) next_request();                                                                               \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
    }
    const int lane_line = (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 3)) * 16);
    const int lane_frag0 = m * 128 + ((kg ^ (m & 7)) * 16), lane_frag1 = m * 128 + (((4 + kg) ^ (m & 7)) * 16);
    int c = 0, gc = 0;                             // chunk inside the pass, chunk of the task
    auto next_chunk = [&]() { return c + 1 == n_chunks ? 0 : c + 1; };
    auto advance = [&]() {
        ++gc;
        if (++c == n_chunks) {
            finish_pass();
            clear();
            c = 0;
            ti0 += PASS;
        }
    };
    for (; gc + 1 < total;) {
        fetch_chunk(next_chunk());
        ETC_BLOCK_CHUNK(gc & 1, true)
        park_chunk((gc + 1) & 1);
        __syncthreads();
        advance();
    }
    ETC_BLOCK_CHUNK(gc & 1, false)
    finish_pass();
#undef ETC_BLOCK_CHUNK
#undef ETC_BLOCK_READS
    trace_mark(P, a.task_id, 3);
    __syncthreads();                               // the operand buffers are free again
}

// Passes of the wide (33 .. 64 columns) and the lines path (NG groups of 8 columns).
template <int TW, int NG>
__device__ __forceinline__ void gemm_tiles_wide_passes(const Params &PL, ChunkedArgs a, ChunkedArgs *slot, float *sm, int *frame_anchor)
{
    constexpr int PASS = NG == 8 ? kWaves / 2 * TW : kWaves * TW;
    const int total = a.g.n_tiles;
    for (int t0 = 0; t0 < total; t0 += PASS) {
        a.g.n_tiles = total - t0 < PASS ? total - t0 : PASS;
        if (t0 > 0 || a.g.n_tiles != total) {
            __syncthreads();                       // every wavefront has read the slot's current contents
            if (threadIdx.x == 0) lds_put(slot, a);
            __syncthreads();
        }
        if constexpr (NG == 8) gemm_tiles_wide<TW>(PL, slot, sm, frame_anchor);
        else gemm_tiles_lines<TW, NG>(PL, slot, sm, frame_anchor);
        a.g.rowsA += (size_t)PASS * a.g.tile_rows * a.g.ldw;
        a.g.rowsB += (size_t)PASS * a.g.tile_rows * a.g.ldw;
        a.e.row0 += PASS * a.g.tile_rows;
        if (a.e.ssq_out) a.e.ssq_out += (size_t)PASS * kMaxBatch;
        a.w = TaskWaits{-1, -1, a.w.fn, false, -1};
    }
}

// One call per pass over the operand: T row tiles each (the events have been seen after the first pass).
template <int NB, int T, bool BUF16 = true>
__device__ __forceinline__ void gemm_tiles_chunked_passes(const Params &PL, ChunkedArgs a, ChunkedArgs *slot, float *sm, int *frame_anchor)
{
    const int total = a.g.n_tiles;
    for (int t0 = 0; t0 < total; t0 += T) {
        a.g.n_tiles = total - t0 < T ? total - t0 : T;
        if (t0 > 0 || a.g.n_tiles != total) {      // the slot already holds the arguments of a single pass
            __syncthreads();                       // every wavefront has read the slot's current contents (a wavefront that
                                                   // runs ahead must not rewrite them under the others: they would disagree
                                                   // on the number of passes)
            if (threadIdx.x == 0) lds_put(slot, a);
            __syncthreads();
        }
        gemm_tiles_chunked<NB, T, BUF16>(PL, slot, sm, frame_anchor);
        a.g.rowsA += (size_t)T * a.g.tile_rows * a.g.ldw;
        a.g.rowsB += (size_t)T * a.g.tile_rows * a.g.ldw;
        a.e.row0 += T * a.g.tile_rows;
        if (a.e.ssq_out) a.e.ssq_out += (size_t)T * kMaxBatch;
        a.w = TaskWaits{-1, -1, a.w.fn, false, -1};
    }
}

// Entry of the out-of-line paths; the slot holds their arguments.  Tasks of 5 or more row tiles have a loop whose wavefronts
// split the output (wide, lines; row blocks of experts: stream, blocks); the fewer tiles of the others (QKV, narrow plans)
// would leave wavefronts idle there, so they split K (chunked, 1, 2 or 4 tiles: the loop always moves T, so T follows the
// task).  Operand rows longer than kMaxBufLd lie outside one buffer descriptor: split K, a tile at a time, 8-byte loads.
// Measured against 16 x 64-byte fragments and 8-byte operand loads: 8B batch 5 / 16 / 64 686 / 929 / 1314 -> 562 / 817 / 1210 us
// per four layers, the MoE layer at 1024 tokens 808 -> 436.
//
// MOE: a dense instance carries no row blocks of experts.  The task loop saves what a callee may clobber, also the ones it never
// calls: with the bodies of three and four tiles per wavefront behind the one entry the dense instance's loop had 106 accesses to
// scratch memory, without them 40 (8B batch 16 / 64, 70B batch 32: 886 / 1256 / 1306 us with them, 837 / 1213 / 1266 without).
template <bool MOE>
__device__ __noinline__ void gemm_chunked_entry(const Params &PL, ChunkedArgs *slot, float *sm, int *frame_anchor)
{
    const ChunkedArgs a = lds_get_uniform(slot);
    if (a.task_id == -0x7FFFFFFF) *frame_anchor = 1;      // never true; see gemm_tiles_chunked
    int anchor = 0;
#define ETC_CHUNKED(NB_)                                                                         \
    {                                                                                            \
        if (!buf_ok) gemm_tiles_chunked_passes<NB_, 1, false>(PL, a, slot, sm, &anchor);         \
        else if (a.g.n_tiles == 1) gemm_tiles_chunked_passes<NB_, 1>(PL, a, slot, sm, &anchor); \
        else if (a.g.n_tiles == 2) gemm_tiles_chunked_passes<NB_, 2>(PL, a, slot, sm, &anchor); \
        else gemm_tiles_chunked_passes<NB_, 4>(PL, a, slot, sm, &anchor);                        \
    }
    const bool buf_ok = a.g.ldb <= kMaxBufLd;
    if (MOE && buf_ok && (a.e.kind == EPI_MOE_ACT || a.e.kind == EPI_MOE_Y)) {      // row blocks of more than 64 columns exist here only
        if (stream_fits(a.g.n_tiles, a.g.n_cols, a.g.K, a.g.ldb)) {
            if (a.g.n_cols <= 8) gemm_tiles_stream<1>(PL, slot, sm, &anchor);
            else gemm_tiles_stream<2>(PL, slot, sm, &anchor);
            return;
        }
        // as few passes as four tiles per wavefront give, with as few tiles per wavefront as give them
        const int n = a.g.n_tiles, passes = (n + 4 * kWaves - 1) / (4 * kWaves);
        const int tw = n <= passes * 2 * kWaves ? 2 : (n <= passes * 3 * kWaves ? 3 : 4);
#define ETC_BLOCKS(NB_, TW_, L_, NT_) { gemm_tiles_blocks<NB_, TW_, L_, NT_>(PL, slot, sm, &anchor); return; }
        if (a.g.n_cols > 64) {
            if (tw == 2) ETC_BLOCKS(8, 2, false, false)
            if (a.g.w_shared) { if (tw == 3) ETC_BLOCKS(8, 3, false, false) else ETC_BLOCKS(8, 4, false, false) }
            if (tw == 3) ETC_BLOCKS(8, 3, true, true)
            ETC_BLOCKS(8, 4, true, true)
        }
        if (n >= 5 && a.g.n_cols > 32) {       // an expert's only block, or what its full blocks left: streamed once more at most
            if (tw == 2) ETC_BLOCKS(4, 2, false, false)
            if (tw == 3) ETC_BLOCKS(4, 3, true, true)
            ETC_BLOCKS(4, 4, true, true)
        }
#undef ETC_BLOCKS
    }
    if (a.g.n_cols > 32 && a.g.n_tiles >= 16 && buf_ok) gemm_tiles_wide_passes<4, 8>(PL, a, slot, sm, &anchor);
    else if (a.g.n_cols > 32 && a.g.n_tiles >= 5 && buf_ok) gemm_tiles_wide_passes<2, 8>(PL, a, slot, sm, &anchor);
    else if (a.g.n_cols > 32) ETC_CHUNKED(4)
    else if (a.g.n_cols > 16 && a.g.n_tiles >= 9 && buf_ok) gemm_tiles_wide_passes<2, 4>(PL, a, slot, sm, &anchor);   // 9 .. 16 tiles against ONE pass over the operand
    else if (a.g.n_cols > 16 && a.g.n_tiles >= 5 && buf_ok) gemm_tiles_wide_passes<1, 4>(PL, a, slot, sm, &anchor);
    else if (a.g.n_cols > 16) ETC_CHUNKED(2)
    else if (a.g.n_tiles >= 5 && buf_ok) gemm_tiles_wide_passes<1, 2>(PL, a, slot, sm, &anchor);
    else ETC_CHUNKED(1)
#undef ETC_CHUNKED
}

// Second stage of a K-sliced projection: adds the partial sums of the slices in slice order (fixed, so the
// result does not depend on which slice finished first) and runs the projection's own epilogue on the 16
// rows of one row tile.  e is the epilogue of the whole projection; e.row0 = first row of the tile.
__device__ __forceinline__ void kslice_sum(const Params &P, const Epilogue &e, int n_cols, int n_slices, int n_row_tiles)
{
    const size_t slice_stride = (size_t)n_row_tiles * kMaxBatch * 16;
    const float *base = P.kpart + (size_t)(e.row0 >> 4) * kMaxBatch * 16;
    for (int idx = threadIdx.x; idx < n_cols * 8; idx += kWgThreads) {
        const int col = idx >> 3, mp = idx & 7;
        const EpiPre pre = epilogue_preload(P, e, col, mp);
        float a[8], b[8];
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
            a[sl] = b[sl] = 0.f;
            if (sl < n_slices) ld_f32x2_pair(base + (size_t)sl * slice_stride + (size_t)col * 16 + mp, a[sl], b[sl]);
        }
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
            lo += a[sl];
            hi += b[sl];
        }
        apply_epilogue<false>(P, e, col, mp, lo, hi, pre);
    }
}

// cos / sin of the RoPE angle pos * theta^(-2i/d).  The inverse frequencies come from the host in
// double; the angle is reduced to [-pi, pi] in double (positions run into the thousands), the
// hardware sine / cosine then see a small argument.
__device__ __forceinline__ void rope_cos_sin(const Params &P, int pos, int i, float *cs, float *sn)
{
    const double ang = (double)pos * *as_global(P.rope_inv_freq + i);
    const double turns = ang * 0.15915494309189535;          // 1 / (2 pi)
    const float frac = (float)(turns - rint(turns));          // [-0.5, 0.5] turns
    const float r = frac * 6.2831853071795862f;
    *cs = __cosf(r);
    *sn = __sinf(r);
}

// Sort key of (logit, vocabulary id): larger logit first, then lower id.
__device__ __forceinline__ unsigned long long logit_key(float v, int id)
{
    const uint32_t u = __float_as_uint(v);
    const uint32_t ordered = u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
    return ((unsigned long long)ordered << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)id);
}

__device__ __forceinline__ void store_split(uint16_t *hi_p, uint16_t *lo_p, size_t idx, float v)
{
    uint16_t h, l;
    split_bf16(v, h, l);
    st_u16(hi_p + idx, h);
    st_u16(lo_p + idx, l);
}

__device__ __forceinline__ EpiPre epilogue_preload(const Params &P, const Epilogue &e, int col, int mp)
{
    EpiPre pre{};
    if (e.kind == EPI_QKV) {      // both resolved by the step prologue: plain independent loads, no look-up chain
        const int b = col, i = e.row0 + mp;
        if (e.head < P.nq + P.nkv) ld_f32x2(P.rope_cs + ((size_t)b * (P.d >> 1) + i) * 2, pre.a, pre.b);   // q and k heads are rotated
        if (e.head >= P.nq) pre.slot = ld_i32(P.kv_slot + b);
        if (P.qk_norm && e.head < P.nq + P.nkv) {      // gains of the two rows under the per-head norm
            const ETC_AS_GLOBAL LayerWeights *W = as_global(P.weights) + e.layer;
            const uint16_t *gn = (const uint16_t *)(e.head < P.nq ? W->gq : W->gk);
            pre.ga = bf16_bits_to_f32(gld_u16(gn + i));
            pre.gb = bf16_bits_to_f32(gld_u16(gn + i + (P.d >> 1)));
        }
    } else if (e.kind == EPI_RESID) {
        const size_t o0 = (size_t)col * e.ld + e.row0 + mp;
        pre.a = ld_f32(e.resid + o0);
        pre.b = ld_f32(e.resid + o0 + 8);
        if (e.next_gain) {
            pre.ga = bf16_bits_to_f32(gld_u16(e.next_gain + e.row0 + mp));
            pre.gb = bf16_bits_to_f32(gld_u16(e.next_gain + e.row0 + mp + 8));
        }
    }
    return pre;
}

// LM: the instance carries the vocabulary projection's epilogue.
template <bool LM>
__device__ __forceinline__ void apply_epilogue(const Params &P, const Epilogue &e, int col, int mp, float lo, float hi,
                                               const EpiPre &pre)
{
    switch (e.kind) {
    case EPI_QKV: {
        const int b = col, half = P.d >> 1, i = e.row0 + mp;
        float a = lo, c = hi;
        const bool normed = P.qk_norm && e.head < P.nq + P.nkv;
        if (normed) {
            // Per-head RMSNorm before RoPE (Sec. 4.3: Q-Norm / K-Norm).  The head's 1 / rms is a scalar, and the rotation
            // is linear, so it commutes with both: this tile leaves its share of the head's sum of squares (of the
            // raw values), applies the gains and rotates; whoever consumes the head (the attention tasks) sums the
            // tiles' shares and scales by 1 / sqrt(mean + eps).
            float sq = lo * lo + hi * hi;
            sq = lanes_sum<8>(sq);                     // the 8 threads of a column are 8 consecutive lanes
            if (mp == 0) st_f32(P.qk_ssq + ((size_t)b * (P.nq + P.nkv) + e.head) * (size_t)(P.d >> 4) + (e.row0 >> 3), sq);
            lo *= pre.ga;
            hi *= pre.gb;
            a = lo;
            c = hi;
        }
        if (e.head < P.nq + P.nkv) {
            a = lo * pre.a - hi * pre.b;
            c = lo * pre.b + hi * pre.a;
        }
        if (e.head < P.nq) {
            float *q = P.qbuf + (size_t)b * (size_t)(P.nq * P.d) + (size_t)e.head * P.d;
            st_f32(q + i, a);
            st_f32(q + i + half, c);
        } else {
            const bool is_k = e.head < P.nq + P.nkv;
            const int kvh = is_k ? e.head - P.nq : e.head - P.nq - P.nkv;
            const size_t off = (size_t)e.layer * (size_t)P.pool_layer_stride +
                               ((size_t)pre.slot * P.nkv + kvh) * (size_t)P.d;
            uint16_t *dst = (is_k ? P.kpool : P.vpool) + off;
            if (!(is_k && normed)) {       // a normalised key reaches the cache from the attention task that completes its norm
                st_u16(dst + i, f32_to_bf16_bits(a));
                st_u16(dst + i + half, f32_to_bf16_bits(c));
            }
            // this step's attention takes the new row unrounded (the cache keeps bf16)
            float *cur = (is_k ? P.knew : P.vnew) + ((size_t)b * P.nkv + kvh) * (size_t)P.d;
            st_f32(cur + i, a);
            st_f32(cur + i + half, c);
        }
        break;
    }
    case EPI_RESID: {
        const int b = col;
        const size_t o0 = (size_t)b * e.ld + e.row0 + mp, o1 = o0 + 8;
        const float v0 = pre.a + lo, v1 = pre.b + hi;
        st_f32(e.outf + o0, v0);
        st_f32(e.outf + o1, v1);
        if (e.next_gain) {   // operand of the next projection: (value * gain) split
            store_split(e.out_hi, e.out_lo, o0, v0 * pre.ga);
            store_split(e.out_hi, e.out_lo, o1, v1 * pre.gb);
        }
        float s = v0 * v0 + v1 * v1;      // this tile's sum of squares: the 8 threads of a column are 8 consecutive lanes
        s = lanes_sum<8>(s);
        if (mp == 0 && e.ssq_out) st_f32(e.ssq_out + b, s);
        if ((e.flags & TF_LAST_LAYER) && P.hidden_out) {
            gst_u16(P.hidden_out + o0, f32_to_bf16_bits(v0));
            gst_u16(P.hidden_out + o1, f32_to_bf16_bits(v1));
        }
        if (e.flags & EPF_DUMP_LAYER) {
            float *dbg = P.layer_hidden + (size_t)e.layer * (size_t)kMaxBatch * e.ld;
            gst_f32(dbg + o0, v0);
            gst_f32(dbg + o1, v1);
        }
        break;
    }
    case EPI_SWIGLU: {
        store_split(e.out_hi, e.out_lo, (size_t)col * e.ld + e.row0 + mp, silu_f(lo) * hi);
        break;
    }
    case EPI_STORE_F32: {
        st_f32(e.outf + (size_t)col * e.ld + e.row0 + mp, lo);
        st_f32(e.outf + (size_t)col * e.ld + e.row0 + mp + 8, hi);
        break;
    }
    case EPI_LOGITS: {
        if (!LM) break;
        // fp32 logits of 16 vocabulary rows, and the tile's best (logit, id) towards the sequence's running maximum.
        // The key orders like the logit (sign-folded bits) and, among equal logits, like the complement of the id,
        // so that the maximum is the greedy token with ties to the lower id; max is exact and order-free, so the
        // result does not depend on which tile arrives first.
        const int r = e.row0 + mp;
        st_f32(e.outf + (size_t)col * e.ld + r, lo);
        st_f32(e.outf + (size_t)col * e.ld + r + 8, hi);
        unsigned long long key = logit_key(lo, r), k2 = logit_key(hi, r + 8);
        key = k2 > key ? k2 : key;
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {        // the 8 threads of a column are 8 consecutive lanes
            const unsigned long long o = __shfl_xor(key, off, 64);
            key = o > key ? o : key;
        }
        // first into the task's own maxima in LDS: one device-scope atomic per task and column reaches memory
        // (thousands of them on one address are serialised there: 16 ns each, 130 us per 8B-vocabulary step)
        if (mp == 0) __hip_atomic_fetch_max(e.lds_best + col, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        break;
    }
    case EPI_MOE_ACT: {
        store_split(e.out_hi, e.out_lo, (size_t)(e.col0 + col) * e.ld + e.row0 + mp, silu_f(lo) * hi);
        break;
    }
    case EPI_PARTIAL: {
        float *dst = e.outf + ((size_t)(e.row0 >> 4) * kMaxBatch + col) * 16 + mp;
        st_f32(dst, lo);
        st_f32(dst + 8, hi);
        break;
    }
    case EPI_MOE_Y: {
        st_f32(e.outf + (size_t)(e.col0 + col) * e.ld + e.row0 + mp, lo);
        st_f32(e.outf + (size_t)(e.col0 + col) * e.ld + e.row0 + mp + 8, hi);
        break;
    }
    }
}

}  // namespace etc
