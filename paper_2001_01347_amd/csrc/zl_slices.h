// The summed-wait search of larger instances over value cells, in slices of their values.
// Part of the ZipLine library (see zipline.hip); device code for gfx950.
#pragma once
#include "zl_cells.h"

namespace {

// With W(c) = P * c - S(c), S(c) the sum over the rows of their last entries up to c (all relative to the instance's
// smallest entry), and values cut into cells:
//     P * first - S(last)  <=  W(x)  for every entry x of the cell [first, last], and
//     P * last - S(last)   >=  the wait of the last entry up to `last`, a candidate from thr on.
// S at the end of every cell is a prefix sum of what the entries add to it, x less the entry before it in its row, one LDS
// word per cell: no order, no counts, nothing kept per entry.  Cells whose lower bound exceeds the smallest upper bound hold
// no minimum; the rest, a handful per instance, are listed with their lower bounds for the kernels that follow (zl_slices_queue_kernel),
// which evaluate their entries in 64 bits.
//
// zl_slices_kernel: one workgroup per slice of the values from thr to C, the last value that can win (cut_step).  Rows are
// read once, from where a probe finds the slice's first entry in them, and what lies behind C only for its order.
// Predicted rows are not read at all: their entries and indices are arithmetic.
// How wide cells may be follows from the waits: P rows wait with a standard deviation of about T * sqrt(P / 12) for a mean
// iteration time T, a cell blurs a wait by P times its width, and the blur, in standard deviations, decides how many cells are
// left to look at.  A workgroup takes its slice in as many parts of NB cells as that asks for.  Blur of 0.5 / 0.7 / 1.0 / 1.4, us:
// one slice per instance, 1024 of 256 x 1024 922 / 852 / 1017 / 970, predicted 348 / 285 / 359 / 342; eight, 64 of 1024 x 4096
// 749 / 748 / 674 / 670.
// Keys are the values shifted down to 31 bits (ms; 0 for most inputs), where the bounds are P units wider either way.
// Cells are 32-bit sums; that none has passed 2^32 is seen from their total, which the slice's edges give in 64 bits.
constexpr int SLICE_PMAX = 1024;                 // rows whose index ranges LDS holds
constexpr int SLICE_PARTS = 32;                  // parts of a slice at most (then cells are wider)
constexpr float SLICE_BLUR = 0.7f, SLICE_BLUR_MANY = 1.0f;

struct SlicePart {       // what a slice found
    i64 base;
    u64 thr;
    i64 top;             // a wait that some candidate does not exceed
    u64 from, to;        // the slice's values
    u32 cells, shift;    // cells listed, 2^shift values wide
    u32 flags;
    u32 left;            // 1: the list or a cell's sum did not do; the general search takes the slice
    u32 exact, far;      // 1: `least` below is the exact P * first - S at the cell's end; values spread over 2^32 and more
};
struct SliceCell {
    u64 first;
    i64 least;           // no entry of the cell waits less
};
// Instances of which a cell is left to look at, by zl_slices_queue_kernel.
struct SliceQueued {
    u64 best;            // the best wait so far
    u32 cells, at;       // how many cells may win; where the queue holds them
    u32 ended, lowest;   // how many have been looked at; the cell that zl_slices_queue_kernel has looked at (NO_CELL: none)
    u32 many, pad_;      // 1: they are in the list of crowded cells
};
constexpr u32 NO_CELL = 0xffffffffu;
struct SliceQueue {
    u32 cells, rest;     // cells queued; instances left to zl_slices_rest_kernel,
    u32 crowded, wide;   // and cells: of one word per value, others
};
struct SliceBest {
    u64 wait, x;
};
// The workspace.
struct SliceSpace {
    SlicePart* part;         // per slice
    SliceBest* result;       // (zl_slices_rest_kernel)
    SliceQueued* queued;     // per instance
    SliceQueue* queue;
    u32* rest;
    uint2* ranges;           // stored rows: per slice and row the indices of its first entry in the slice and the one behind it
    SliceCell* cell;         // `room` per slice; looked at: the best entry and its wait
    u32* order;              // the queue: their numbers
    u32* crowded;            // those of more entries than a wave takes; from its end the wide ones
    size_t cells;            // of all slices together
};
constexpr size_t SLICE_CELL_BYTES = sizeof(SliceCell) + 2 * sizeof(u32);
ZL_FN size_t slice_space_fixed(i64 B, i64 slices, int rows)
{
    return (size_t)B * ((size_t)slices * (sizeof(SlicePart) + sizeof(SliceBest) + (size_t)rows * sizeof(uint2)) + sizeof(SliceQueued) + sizeof(u32)) + sizeof(SliceQueue) + 16;
}
ZL_FN SliceSpace slice_space(void* at, i64 B, i64 slices, int rows, u32 room)
{
    SliceSpace s;
    s.part = (SlicePart*)at;
    s.result = (SliceBest*)(s.part + B * slices);
    s.queued = (SliceQueued*)(s.result + B * slices);
    s.queue = (SliceQueue*)(s.queued + B);
    s.ranges = (uint2*)(s.queue + 1);
    s.rest = (u32*)(s.ranges + (size_t)(B * slices) * rows);
    s.cell = (SliceCell*)(((uintptr_t)(s.rest + B) + 15) & ~(uintptr_t)15);
    s.order = (u32*)(s.cell + (size_t)(B * slices) * room);
    s.cells = (size_t)(B * slices) * room;
    s.crowded = s.order + s.cells;
    return s;
}

// Results that other workgroups read are stored and loaded at agent scope, past the caches; the count follows once they have arrived.
// An acquire-release count instead writes back and invalidates the whole L2 every time (the cells of 1024 of 256 x 1024 by a
// workgroup each: 3330 us with it, 1180 without).
__device__ __forceinline__ void publish(u64* to, u64 v) { __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u64 published(const u64* from) { return __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u32 count_published(u32* counter)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One row of an instance, stored or predicted, values relative to base.
template <bool PRED> struct SliceRow;
template <> struct SliceRow<false> {
    const i64* row;
    u32 R;
    u64 base, f, l;      // first and last entry
    __device__ __forceinline__ u64 at(u32 i) const { return (u64)row[i] - base; }
    // the first index with an entry of at least v (R: none)
    __device__ __forceinline__ u32 below(u64 v) const { return RowProbe(row, R, base, f, l, v).index(); }
};
template <> struct SliceRow<true> {
    u64 f, step;         // first entry and interval
    u32 R;
    double rcp;
    __device__ __forceinline__ u64 at(u32 i) const { return f + (u64)i * step; }
    __device__ __forceinline__ u32 below(u64 v) const { return predicted_below(f, step, rcp, R, v); }
};

template <int NT, int NB>
struct SlicesSmem {
    u32 cells[NB];
    u32 lo[SLICE_PMAX], hi[SLICE_PMAX];
    u64 red[6 * (NT / WAVE)];
    u32 listed;
};

// Several values reduced over the workgroup in one exchange: each to a place `at` of its own in `red`, a barrier, block_reduced.
template <int NT, class Op>
__device__ __forceinline__ void block_reduce_to(u64* red, int at, u64 v, Op op)
{
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x >> 6;
    const u64 r = wave_scan(v, op);
    if (lane == WAVE - 1) red[at * (NT / WAVE) + wave] = r;
}
template <int NT, class Op>
__device__ __forceinline__ u64 block_reduced(const u64* red, int at, Op op)
{
    u64 r = red[at * (NT / WAVE)];
#pragma unroll
    for (int w = 1; w < NT / WAVE; ++w) r = op(r, red[at * (NT / WAVE) + w]);
    return r;
}

// The entries of one part: every entry's addition to S goes to its cell.  WIDE: keys are shifted.
template <int NT, int NB, bool PRED, bool WIDE, int U = 4>
__device__ __forceinline__ void slice_entries(SlicesSmem<NT, NB>& sm, const i64* __restrict__ inst, const i64* __restrict__ le, const i64* __restrict__ iv,
                                              int P, int R, u64 base, u32 A, u32 E, u32 shk, u32 ms, int lanes_log, bool from_start, int& bad)
{
    const int tid = threadIdx.x;
    const int groups = NT >> lanes_log, group = tid >> lanes_log;
    const u32 span = E - A;
    [[maybe_unused]] const u32 base32 = (u32)base + A;
    [[maybe_unused]] auto pair = [&](i64 before, i64 entry) {
        bad |= entry < before;
        u32 xk, d;                                         // the key from A on, and what it adds
        if (WIDE) {
            const u32 k = (u32)(((u64)entry - base) >> ms);
            xk = k - A;
            d = k - (u32)(((u64)before - base) >> ms);
        } else {
            xk = (u32)entry - base32;
            d = (u32)entry - (u32)before;
        }
        if (xk <= span) atomicAdd(&sm.cells[xk >> shk], d);
    };
    if constexpr (!PRED)
        if (lanes_log == 6) {
            // Whole waves walk rows, U of them at once, each lane two neighbouring entries a step (and the one before them, which
            // the lane before holds: 127 pairs).  All loads of a step are made whether a row is through or not: a branch around them
            // waits for each.  The kernel on 1024 of 256 x 1024, us: an entry a lane and four steps of one row ahead 946, of four
            // rows 867, two entries 694, without branches 545.
            constexpr int NW = NT / WAVE;
            constexpr u32 STEP = 2 * WAVE - 1;
            const u32 lane = tid & (WAVE - 1);
            for (int p0 = (int)uniform((u32)tid >> 6); p0 < P; p0 += U * NW) {
                u32 s[U], to[U];                           // to: the last entry; s: the next step's first
                const i64* row[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int p = p0 + u * NW < P ? p0 + u * NW : P - 1;
                    const u32 i0 = uniform(sm.lo[p]), i1 = p0 + u * NW < P ? uniform(sm.hi[p]) : 0u;
                    s[u] = from_start || i0 == 0 ? 0u : i0 - 1;
                    to[u] = i1 ? i1 - 1 : 0u;
                    row[u] = inst + (size_t)p * R;
                }
                for (;;) {
                    bool more = false;
#pragma unroll
                    for (int u = 0; u < U; ++u) more |= s[u] < to[u];
                    if (!more) break;
                    i64 v[U][2];
#pragma unroll
                    for (int u = 0; u < U; ++u) {          // (of a row that is through: its last two entries again)
                        const u32 i = s[u] + 2 * lane, last = to[u] ? to[u] - 1 : 0u;
                        const i64* e = row[u] + (i < last ? i : last);
                        v[u][0] = e[0];
                        v[u][1] = e[1];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (s[u] < to[u]) {
                            const u32 n = to[u] - s[u];    // the step's entries are 0 .. n, this lane's 2 * lane and the next
                            const i64 before = dpp_take<DPP_WAVE_SHR1, 0xf>((i64)0, v[u][1]);
                            if (2 * lane < n) {
                                if (lane > 0) pair(before, v[u][0]);
                                pair(v[u][0], v[u][1]);
                            } else if (2 * lane == n && lane > 0)
                                pair(before, v[u][1]);     // (its own place is behind the last entry: that is its second)
                            s[u] = n > STEP ? s[u] + STEP : to[u];
                        }
                }
            }
            return;
        }
    for (int p = group; p < P; p += groups) {
        const u32 i0 = sm.lo[p], i1 = sm.hi[p];
        if constexpr (PRED) {
            const u32 lanes = 1u << lanes_log, lane = tid & (lanes - 1);
            const u64 s = (u64)iv[p];
            u32 i = (i0 ? i0 : 1u) + lane;
            const u64 x0 = (u64)le[p] + s - base + (u64)i * s;
            if constexpr (WIDE) {
                u64 x = x0;
                for (; i < i1; i += lanes, x += s << lanes_log) {
                    const u32 xk = (u32)(x >> ms), pk = (u32)((x - s) >> ms);
                    atomicAdd(&sm.cells[(xk - A) >> shk], xk - pk);
                }
            } else {
                const u32 s32 = (u32)s, more = s32 << lanes_log;
                u32 x = (u32)x0 - A;                       // (values up to C fit 31 bits, so do intervals that lead to them)
                for (; i < i1; i += lanes, x += more) atomicAdd(&sm.cells[x >> shk], s32);
            }
        } else {
            const u32 from = from_start || i0 == 0 ? 0u : i0 - 1;
            if (i1 == 0 || i1 - 1 <= from) continue;
            const i64* row = inst + (size_t)p * R;
            const u32 lanes = 1u << lanes_log;
            for (u32 i = from + 1 + (tid & (lanes - 1)); i < i1; i += lanes) pair(row[i - 1], row[i]);
        }
    }
}

// Bound by the one reading of stored rows (64 of 1024 x 4096: 515 us for 2.15 GB, 270 of them for what lies behind C at 5.7 TB/s and
// 130 for the cells, the rest the probes and reductions ahead of them; by windows a partition pass of 485 and a search of 386),
// by the vector ALU and LDS where they are predicted (99 us, 283 by windows).  At two workgroups of a CU the compiler keeps 13
// (predicted: 7) of a thread's registers in memory: mostly the sums of its cells, walked by index where some are listed.
template <int NT, int NB, bool PRED>
__global__ __launch_bounds__(NT, 4) void zl_slices_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, int P, int R, u32 slices,
    void* __restrict__ workspace, u32 room)
{
    constexpr int LOG = __builtin_ctz((unsigned)NB), NW = NT / WAVE, RPT = SLICE_PMAX / NT, STEPS = NB / NT / 4;
    static_assert(NB % (4 * NT) == 0 && SLICE_PMAX % NT == 0, "whole steps");
    __shared__ __align__(16) SlicesSmem<NT, NB> sm;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x / slices;
    const u32 k = blockIdx.x % slices;
    const SliceSpace space = slice_space(workspace, B, slices, PRED ? 0 : P, room);
    const i64* __restrict__ inst = PRED ? nullptr : ts + b * (i64)P * R;
    if (PRED) { le += b * (i64)P; iv += b * (i64)P; }
    if (blockIdx.x == 0 && tid == 0) *space.queue = SliceQueue{0, 0, 0, 0};
    SlicePart out{};
    SliceCell* const list = space.cell + (size_t)blockIdx.x * room;

    // the ends of the thread's rows
    SliceRow<PRED> row[RPT];
    u64 last[RPT];
    i64 mn = INT64_MAX, mxf = INT64_MIN, mxl = INT64_MIN, mnl = INT64_MAX;
    u64 spans = 0;
    int back = 0, wrapped = 0;
    const u64 interval = PRED ? (u64)iv[0] : 0ull;
    int differ = 0;                                        // 1: not all intervals are this one
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int p = tid + r * NT;
        i64 f = INT64_MAX, l = INT64_MIN;
        row[r] = SliceRow<PRED>{};
        last[r] = 0;
        if (p < P) {
            if constexpr (PRED) {
                const u64 s = (u64)iv[p], from = (u64)le[p];
                f = (i64)(from + s);
                l = (i64)(from + (u64)R * s);
                back |= R > 1 && (i64)s < 0;
                wrapped |= l < f;
                differ |= s != interval;
                row[r].step = s;
            } else {
                row[r].row = inst + (size_t)p * R;
                f = row[r].row[0];
                l = row[r].row[R - 1];
                back |= l < f;
            }
            mn = f < mn ? f : mn;
            mxf = f > mxf ? f : mxf;
            mxl = l > mxl ? l : mxl;
            mnl = l < mnl ? l : mnl;
            spans += (u64)l - (u64)f;
            row[r].f = (u64)f;
            last[r] = (u64)l;
        }
    }
    for (int c = tid; c < NB / 4; c += NT) ((uint4*)sm.cells)[c] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) sm.listed = 0;
    {
        constexpr u64 SIGN = 1ull << 63;                   // signed order as unsigned
        u64 v0 = (u64)mn ^ SIGN, v1 = (u64)mxf ^ SIGN, v2 = (u64)mxl ^ SIGN, v3 = (u64)mnl ^ SIGN;
        block_reduce_to<NT>(sm.red, 0, v0, OpMin());
        block_reduce_to<NT>(sm.red, 1, v1, OpMax());
        block_reduce_to<NT>(sm.red, 2, v2, OpMax());
        block_reduce_to<NT>(sm.red, 3, v3, OpMin());
        block_reduce_to<NT>(sm.red, 4, spans, OpAdd());
        const u64 any = (__ballot(back) ? 1ull : 0ull) | (__ballot(wrapped) ? 2ull : 0ull) | (__ballot(differ) ? 4ull : 0ull);
        if (lane == 0) sm.red[5 * NW + wave] = any;
        __syncthreads();
        v0 = block_reduced<NT>(sm.red, 0, OpMin());
        v1 = block_reduced<NT>(sm.red, 1, OpMax());
        v2 = block_reduced<NT>(sm.red, 2, OpMax());
        v3 = block_reduced<NT>(sm.red, 3, OpMin());
        spans = uniform(block_reduced<NT>(sm.red, 4, OpAdd()));
        u64 flags = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) flags |= sm.red[5 * NW + w];
        flags = uniform(flags);
        back = (flags & 1) != 0;
        wrapped = (flags & 2) != 0;
        differ = (flags & 4) != 0;
        __syncthreads();                                   // (they are written again)
        mn = (i64)uniform(v0 ^ SIGN); mxf = (i64)uniform(v1 ^ SIGN); mxl = (i64)uniform(v2 ^ SIGN); mnl = (i64)uniform(v3 ^ SIGN);
    }
    const u64 base = (u64)mn, thr = (u64)mxf - base, range = (u64)mxl - base;
    out.base = mn;
    out.thr = thr;
    out.far = (range >> 32) != 0;
    out.top = INT64_MAX;
    out.flags = back ? (u32)EBSP_STATUS_UNSORTED : 0u;
    if ((!back && wrapped) || range > (u64)INT64_MAX / (u64)P) out.flags |= EBSP_STATUS_OVERFLOW;
    if (out.flags) {                                       // (the same in every slice: nothing below may rely on such rows)
        if (!PRED && !back) {                              // values too far apart: rows out of order are flagged as well
            for (int p = (int)k * NW + wave; p < P; p += (int)slices * NW)
                row_pairs(inst + (size_t)p * R, 0u, (u32)R - 1, 6, [&](i64 a, i64 y) { back |= y < a; });
            if (__syncthreads_or(back)) out.flags |= EBSP_STATUS_UNSORTED;
        }
        if (tid == 0) space.part[blockIdx.x] = out;
        return;
    }
    const u64 min_last = (u64)mnl - base;

    // C, the last value that can win (see zl_plan.h)
    u64 C = range;
    {
        const u64 x = min_last > thr ? min_last : thr;
        u64 mine = 0;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int p = tid + r * NT;
            row[r].R = (u32)R;
            if (p < P) {
                row[r].f -= base;
                last[r] -= base;
                if constexpr (PRED) {
                    row[r].rcp = row[r].step ? 1.0 / (double)row[r].step : 0.0;
                    mine += direct_remainder(x - row[r].f, row[r].step, row[r].rcp, (u32)R - 1);
                } else {
                    row[r].base = base;
                    row[r].l = last[r];
                    const u32 i = row[r].below(x + 1);
                    mine += x - row[r].at(i ? i - 1 : 0u);
                }
            }
        }
        const u64 ub = block_reduce<u64, NT>(mine, sm.red, OpAdd());
        for (int it = 0; it < CUT_STEPS; ++it) {
            u64 lb = 0, n = 0;
#pragma unroll
            for (int r = 0; r < RPT; ++r)
                if (tid + r * NT < P && last[r] < C) { lb += C - last[r]; ++n; }
            block_reduce_to<NT>(sm.red, 0, lb, OpAdd());
            block_reduce_to<NT>(sm.red, 1, n, OpAdd());
            __syncthreads();
            lb = block_reduced<NT>(sm.red, 0, OpAdd());
            n = block_reduced<NT>(sm.red, 1, OpAdd());
            __syncthreads();
            const u64 was = C;
            if (!cut_step(C, lb, n, ub) || was - C < C >> 9) break;       // (the same in every thread)
        }
        // One interval for all workers: every candidate x from thr + interval on has one an interval before it, and there no
        // worker waits longer (one that is not through by x waits as long, one that is waits longer at x).
        if constexpr (PRED)
            if (!differ && interval && C - thr >= interval) C = thr + interval - 1;
        C = uniform(C);
    }

    // keys, cells and the slice
    const u64 steps = R > 1 ? spans / (u64)(R - 1) : 1ull;                // sum of the rows' mean iteration times
    int m = bit_length(C) - 31;
    m = m > bit_length(steps) - 31 ? m : bit_length(steps) - 31;          // (a round of all rows in one cell: below 2^32)
    const u32 ms = m > 0 ? (u32)m : 0u;
    const u32 Ck = (u32)(C >> ms), thrk = (u32)(thr >> ms), width = (Ck - thrk) / slices + 1;
    u32 shk;
    {
        const float rows = (float)P, wide = (PRED || slices == 1 ? SLICE_BLUR : SLICE_BLUR_MANY) * (float)steps / (rows * sqrtf(12.0f * rows));
        const int sh = wide > 1.0f ? (int)log2f(wide) : 0;
        shk = sh > (int)ms ? (u32)sh - ms : 0u;
        while (shk < 31u - LOG && ((width - 1) >> (shk + LOG)) >= (u32)SLICE_PARTS) ++shk;
        if (shk > 31u - LOG) shk = 31u - LOG;
        shk = uniform(shk);
    }
    out.shift = shk + ms;
    out.exact = ms == 0;
    const u64 Aw = (u64)thrk + (u64)width * k;
    const bool empty = Aw > Ck;
    u32 A = empty ? Ck : (u32)Aw;
    const u32 last_key = Ck - A < width ? Ck : A + width - 1;
    out.from = (u64)A << ms;
    out.to = empty ? 0ull : ((u64)(last_key + 1) << ms) - 1;
    if (empty) out.from = 1;
    int bad = 0;
    if (!PRED && slices > 1) {
        // the order of what lies behind C: the rows' stretches there are shared out among the slices
        const u32 pieces = (slices + (u32)P - 1u) / (u32)P;
        const u64 units = (u64)P * pieces;
        const u64 u0 = units * k / slices, u1 = units * (k + 1) / slices;
        for (u64 u = u0 + wave; u < u1; u += NW) {
            const i64* r = inst + (size_t)(u / pieces) * R;
            const u32 q = (u32)(u % pieces), t = row_first_at_least(r, (u32)R, base, (u64)(Ck + 1) << ms);
            const u32 t0 = t ? t - 1 : 0u;                 // pairs up to (t0 - 1, t0) are the slices'
            if (t0 + 1 >= (u32)R) continue;
            const u64 len = (u64)R - 1 - t0;
            const u32 from = t0 + (u32)(len * q / pieces), to = t0 + (u32)(len * (q + 1) / pieces);
            row_pairs(r, from, to, 6, [&](i64 p, i64 y) { bad |= y < p; });
        }
    }
    i64 top = INT64_MAX;                                   // in keys
    const i64 slack = ms ? (i64)P : 0, most = INT64_MAX >> ms;
    u64 before = 0;                                        // S before A, in keys
    for (bool begin = true; !empty; begin = false) {
        const u32 E = (u64)last_key - A < ((u64)NB << shk) ? last_key : A + ((u32)NB << shk) - 1;
        u64 sa = 0, se = 0;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int p = tid + r * NT;
            if (p < P) {
                u32 i0, i1;
                if (begin) {
                    if constexpr (PRED) {
                        i0 = row[r].below((u64)A << ms);
                        i1 = row[r].below((u64)(E + 1) << ms);
                    } else {
                        const RowProbe pa(row[r].row, (u32)R, base, row[r].f, row[r].l, (u64)A << ms);
                        const RowProbe pe(row[r].row, (u32)R, base, row[r].f, row[r].l, (u64)(E + 1) << ms);
                        i0 = pa.index();
                        i1 = pe.index();
                    }
                    if (i0) sa += row[r].at(i0 - 1) >> ms;
                    if constexpr (!PRED) space.ranges[(size_t)blockIdx.x * P + p].x = i0;
                } else {
                    i0 = sm.hi[p];
                    i1 = row[r].below((u64)(E + 1) << ms);
                }
                bad |= i1 < i0;
                i1 = i1 < i0 ? i0 : i1;
                if (i1) se += row[r].at(i1 - 1) >> ms;
                sm.lo[p] = i0;
                sm.hi[p] = i1;
                if (!PRED && E == last_key) space.ranges[(size_t)blockIdx.x * P + p].y = i1;
                if (i0 == 0 && i1 > 0) {                   // the row's first entry adds itself
                    const u32 fk = (u32)(row[r].f >> ms);
                    if (fk - A <= E - A) atomicAdd(&sm.cells[(fk - A) >> shk], fk);
                }
            }
        }
        if (begin) block_reduce_to<NT>(sm.red, 0, sa, OpAdd());
        block_reduce_to<NT>(sm.red, 1, se, OpAdd());
        __syncthreads();
        if (begin) before = uniform(block_reduced<NT>(sm.red, 0, OpAdd()));
        const u64 after = uniform(block_reduced<NT>(sm.red, 1, OpAdd()));
        // whole waves walk a row's stretch where it is long enough
        int lanes_log = 6;
        {
            const float len = 1.25f * (float)(E - A) * (float)P / ((float)(steps >> ms) + 1.0f);
            while (lanes_log > 0 && (float)(1 << lanes_log) > len) --lanes_log;
            lanes_log = (int)uniform((u32)lanes_log);
        }
        if (ms) slice_entries<NT, NB, PRED, true>(sm, inst, le, iv, P, R, base, A, E, shk, ms, lanes_log, begin && k == 0, bad);
        else slice_entries<NT, NB, PRED, false>(sm, inst, le, iv, P, R, base, A, E, shk, 0u, lanes_log, begin && k == 0, bad);
        bad = __syncthreads_or(bad);
        if (bad) break;
        // The waves' cells: every wave owns NB / NW neighbouring ones and walks them 256 at a time, four to a lane.
        const u32 mine = wave * (NB / NW) + 4 * lane;
        u64 sum[STEPS];                                    // of the cells before the lane's in its wave
        {
            u64 run = 0;
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const uint4 q = *(const uint4*)(sm.cells + mine + i * 256);
                const u64 own = (u64)q.x + q.y + ((u64)q.z + q.w);
                const u64 inc = wave_scan(own, OpAdd());
                sum[i] = run + inc - own;
                run += last_lane(inc);
            }
            if (lane == 0) sm.red[2 * NW + wave] = run;
        }
        __syncthreads();
        u64 all = 0, ahead = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const u64 s = sm.red[2 * NW + w];
            if (w < wave) ahead += s;
            all += s;
        }
        if (uniform(all) != after - before) { out.left = 1; break; }      // a cell's sum has passed 2^32
        // least(c): P * (its first key) - S at its end
        const i64 at_A = (i64)((u64)P * A - before - ahead), PL = (i64)((u64)P << shk);
        i64 low = INT64_MAX;
        auto cells_of = [&](int i, const auto& f) {
            const u32 c = mine + i * 256;
            const uint4 q = *(const uint4*)(sm.cells + c);
            i64 w = at_A + (i64)c * PL - (i64)sum[i];
            w -= q.x; f(c, w); w += PL;
            w -= q.y; f(c + 1, w); w += PL;
            w -= q.z; f(c + 2, w); w += PL;
            w -= q.w; f(c + 3, w);
        };
#pragma unroll
        for (int i = 0; i < STEPS; ++i) cells_of(i, [&](u32, i64 w) { low = w < low ? w : low; });
        const i64 least = (i64)block_reduce<i64, NT>(low, (i64*)sm.red, OpMin());
        const i64 found = least + PL - P;
        top = found < top ? found : top;
        if (low <= top + 2 * slack) {
#pragma unroll 1
            for (int i = 0; i < STEPS; ++i)
                cells_of(i, [&](u32 c, i64 w) {
                    if (w <= top + 2 * slack) {
                        const u32 at = atomicAdd(&sm.listed, 1u);
                        if (at < room) list[at] = SliceCell{(u64)(A + (c << shk)) << ms, (w - slack < most ? w - slack : most) * ((i64)1 << ms)};
                    }
                });
        }
        if (E == last_key) break;
        __syncthreads();
        for (int c = tid; c < NB / 4; c += NT) ((uint4*)sm.cells)[c] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        A = E + 1;
        before = after;
    }
    if (!PRED && !bad && (slices == 1 || out.left)) {
        // the order of what has not been walked: the rest of a slice that was left, and behind C where nobody else reads that
        for (int p = wave; p < P; p += NW) {
            const i64* r = inst + (size_t)p * R;
            const u32 hi = sm.hi[p], from = hi ? hi - 1 : 0u;
            const u32 end = slices == 1 ? (u32)R : row_first_at_least(r, (u32)R, base, (u64)(last_key + 1) << ms);
            bad |= end < hi;
            if (from + 1 < end) row_pairs(r, from, end - 1, 6, [&](i64 a, i64 y) { bad |= y < a; });
        }
    }
    if (!PRED) bad = __syncthreads_or(bad);
    else __syncthreads();
    if (tid == 0) {
        out.top = out.left || top > (INT64_MAX >> ms) - slack ? INT64_MAX : (top + slack) * ((i64)1 << ms);
        out.cells = sm.listed < room ? sm.listed : room;
        out.left |= sm.listed > room ? 1u : 0u;
        if (bad) out.flags = EBSP_STATUS_UNSORTED;
        space.part[blockIdx.x] = out;
    }
}

// What the slices listed: zl_slices_queue_kernel queues the cells that an instance's best upper bound does not rule out, of all
// instances in one queue behind their lowest ones, zl_slices_cells_kernel looks at them.  (Some instances have a few cells left
// and some a hundred: dealt out by instance or slice, the last workgroup took ten times the mean.)
// A cell's entries are found by a probe per row: eight neighbouring entries from where the slice's share of the row would
// put them, one round trip.  They are listed, and where keys are not shifted, with `least` the bound of the cell,
//     W(x) = least + P * (x - first) + what the cell's entries behind x add to S;
// else S before the cell is added up from the rows.
// The last of an instance's cells stores its results (an atomic count; nothing waits).
// zl_slices_rest_kernel: cells of more entries than a wave's list holds (workers in step), one LDS word per value, or, wider than
// that or of shifted keys, in a longer list or FINE cells of their own, of which those that may win are listed; what is still
// too full, and the slices that were left, by the general search of their values.
constexpr int SLICE_FINE = 4096, SLICE_FINE_LOG = 12, SLICE_LIST = 512, SLICE_SIDE = 4;
struct LiveCell {
    u64 first, last;
    i64 least;
    u32 slice;
    float at, end_at;    // where in the slice it begins and ends, 0 to 1
};
__device__ __forceinline__ LiveCell live_cell(const SlicePart& s, const SliceCell& c, u32 slice)
{
    const u64 end = c.first + ((1ull << s.shift) - 1);
    const u64 last = end < s.to ? end : s.to;
    const float all = 1.0f / (float)(s.to - s.from + 1);
    return LiveCell{c.first, last, c.least, slice, (float)(c.first - s.from) * all, (float)(last - s.from) * all};
}

// Row p of an instance for the cells of one slice.
template <bool PRED>
struct CellRows {
    const i64* inst;
    const i64* le;
    const i64* iv;
    int R;
    u64 base;
    static constexpr u32 W = 8;
    struct Window {      // what a row is asked for a cell
        u64 w[PRED ? 1 : W];
        u32 s;
        uint2 range;
    };
    // where W entries begin that are likely to hold the one at `at` of the slice's
    __device__ __forceinline__ u32 start(uint2 range, float at) const
    {
        u32 s = range.x + (u32)((float)(range.y - range.x) * at);
        s = s > W / 2 ? s - W / 2 : 0u;
        return (u32)R > W ? (s < (u32)R - W ? s : (u32)R - W) : 0u;
    }
    __device__ __forceinline__ Window window(int p, uint2 range, float at) const
    {
        Window o;
        o.range = range;
        o.s = 0;
        if constexpr (!PRED) {
            const i64* row = inst + (size_t)p * R;
            const u32 s = start(range, at);
            o.s = s;
#pragma unroll
            for (u32 k = 0; k < W; ++k) o.w[k] = (u64)row[s + k < (u32)R ? s + k : (u32)R - 1];
        }
        return o;
    }
    // The entries in [first, to]: f(entry, the entry before it or 0).  Returns the last entry before `first` (0: none).
    template <class F>
    __device__ __forceinline__ u64 entries(int p, const Window& o, u64 first, u64 to, const F& f) const
    {
        if constexpr (PRED) {
            const u64 s = (u64)iv[p], a = (u64)le[p] + s - base;
            const double rcp = s ? 1.0 / (double)s : 0.0;
            const u32 i0 = predicted_below(a, s, rcp, (u32)R, first);
            u64 x = i0 ? a + (u64)(i0 - 1) * s : 0ull;
            const u64 prev = x;
            for (u32 i = i0; i < (u32)R; ++i) {
                const u64 y = a + (u64)i * s;
                if (y > to || (s == 0 && i > i0)) break;
                f(y, x);
                x = y;
            }
            return prev;
        } else {
            u32 b0 = 0, b1 = 0;
            u64 prev = 0;
#pragma unroll
            for (u32 k = 0; k < W; ++k) {
                const u64 v = o.w[k] - base;
                if (v < first) { ++b0; prev = v; }
                b1 += v <= to ? 1u : 0u;
            }
            const bool seen = (b0 > 0 || o.s == 0) && (b1 < W || o.s + W >= (u32)R);
            if (seen && b0 == b1) return prev;             // (one row in a hundred has an entry in the cell)
            if (seen) return walk(p, o.s + b0, to, f);
            return search(p, o.range, o.s, b0, first, to, f);
        }
    }
    // the entries from index i on; returns the one before
    template <class F>
    __device__ __forceinline__ u64 walk(int p, u32 i, u64 to, const F& f) const
    {
        const i64* row = inst + (size_t)p * R;
        const u64 prev = i ? (u64)row[i - 1] - base : 0ull;
        u64 x = prev;
#pragma unroll 1
        for (; i < (u32)R; ++i) {
            const u64 y = (u64)row[i] - base;
            if (y > to) break;
            f(y, x);
            x = y;
        }
        return prev;
    }
    // the same where the first W entries from s on do not show where they are; b0: how many of those are below `first`
    template <class F>
    __device__ __forceinline__ u64 search(int p, uint2 range, u32 s, u32 b0, u64 first, u64 to, const F& f) const
    {
        const i64* row = inst + (size_t)p * R;
        u32 lo = range.x, hi = range.y, step = W;          // the first entry from `first` on is one of these, or behind them
        if (b0 > 0) {                                      // (galloping from the window)
            lo = s + b0 > lo ? s + b0 : lo;
            while (lo + step < hi && (u64)row[lo + step] - base < first) { lo += step + 1; step *= 2; }
            hi = lo + step < hi ? lo + step : hi;
        } else {
            hi = s < hi ? s : hi;
            while (lo + step < hi && (u64)row[hi - step] - base >= first) { hi -= step; step *= 2; }
            lo = lo + step < hi ? hi - step : lo;
        }
        while (lo < hi) {
            const u32 m = (lo + hi) >> 1;
            if ((u64)row[m] - base < first) lo = m + 1; else hi = m;
        }
        return walk(p, lo, to, f);
    }
    // how many entries of the row are up to x
    __device__ __forceinline__ u32 upto(int p, const Window& o, u64 x) const
    {
        if constexpr (PRED) {
            const u64 s = (u64)iv[p];
            return predicted_below((u64)le[p] + s - base, s, s ? 1.0 / (double)s : 0.0, (u32)R, x + 1);
        } else {
            const i64* row = inst + (size_t)p * R;
            u32 n = 0;
#pragma unroll
            for (u32 k = 0; k < W; ++k) n += o.w[k] - base <= x ? 1u : 0u;
            if ((u32)R <= W) return n < (u32)R ? n : (u32)R;
            if ((n > 0 || o.s == 0) && (n < W || o.s + W == (u32)R)) return o.s + n;
            u32 lo = o.range.x, hi = o.range.y;
            while (lo < hi) {
                const u32 m = (lo + hi) >> 1;
                if ((u64)row[m] - base <= x) lo = m + 1; else hi = m;
            }
            return lo;
        }
    }
};

template <bool PRED>
struct SliceRows {       // the rows of all instances
    const i64* ts;
    const i64* le;
    const i64* iv;
    int P, R;
    __device__ __forceinline__ CellRows<PRED> of(u32 b, u64 base) const
    {
        return CellRows<PRED>{PRED ? nullptr : ts + (size_t)b * P * R, PRED ? le + (size_t)b * P : nullptr, PRED ? iv + (size_t)b * P : nullptr, R, base};
    }
    __device__ __forceinline__ uint2 range(const SliceSpace& space, u32 slices, u32 b, u32 slice, int p) const
    {
        return PRED ? make_uint2(0u, 0u) : space.ranges[((size_t)b * slices + slice) * P + p];
    }
};
// By lane 0 of a wave: what was found in a cell of instance b.  True: it was the instance's last.
__device__ __forceinline__ bool cell_done(const SliceSpace& space, u32 b, u32 number, u64 w, u64 x)
{
    u64* const to = (u64*)(space.cell + number);
    publish(to, x);
    publish(to + 1, w);
    if (w != U64_MAX) atomicMin(&space.queued[b].best, w);
    return count_published(&space.queued[b].ended) + 1 == space.queued[b].cells;
}
// By a wave, when all of an instance's cells have been looked at.
template <bool PRED>
__device__ __forceinline__ void instance_done(const SliceSpace& space, const SliceRows<PRED>& all, u32 b, u32 slices, u32 room,
                                              i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    asm volatile("" ::: "memory");
    const int lane = threadIdx.x & (WAVE - 1);
    const SliceQueued q = space.queued[b];
    u64 w = U64_MAX, x = U64_MAX;
    u32 slice = 0;
    for (u32 j = lane; j <= q.cells; j += WAVE) {
        const u32 n = j < q.cells ? space.order[q.at + j] : q.lowest;
        if (n == NO_CELL) continue;
        u64* const from = (u64*)(space.cell + n);
        const u64 ox = published(from), ow = published(from + 1);
        if (ow < w || (ow == w && ox < x)) { w = ow; x = ox; slice = n / room - b * slices; }
    }
    const u64 mw = w, mx = x;
    wave_argmin(w, x);
    w = last_lane(w);
    x = last_lane(x);
    const u64 who = __ballot(mw == w && mx == x);
    slice = (u32)__builtin_amdgcn_readlane((int)slice, who ? __builtin_ctzll(who) : 0);
    const SlicePart& s = space.part[(size_t)b * slices + slice];
    const float where = (float)(x - s.from) / (float)(s.to - s.from + 1);
    const CellRows<PRED> rows = all.of(b, (u64)s.base);
    if (lane == 0) {
        barrier[b] = (i64)((u64)s.base + x);
        wait[b] = (i64)w;
        if (status) status[b] = 0;
    }
    for (int p0 = lane; p0 < all.P; p0 += 2 * WAVE) {      // two rows of a lane in flight
        const int p1 = p0 + WAVE < all.P ? p0 + WAVE : p0;
        const auto a = rows.window(p0, all.range(space, slices, b, slice, p0), where), z = rows.window(p1, all.range(space, slices, b, slice, p1), where);
        iters[(size_t)b * all.P + p0] = (int)rows.upto(p0, a, x);
        iters[(size_t)b * all.P + p1] = (int)rows.upto(p1, z, x);
    }
}

// A cell's entries, list(entry, the one before it in its row or 0), by `waves` waves of which this is the `wave`th; sums: the
// lanes' shares of S before the cell are added to `before`.  Ends early where *listed has passed `most`.
template <bool PRED, class F>
__device__ __forceinline__ void cell_entries(const SliceSpace& space, const SliceRows<PRED>& all, const CellRows<PRED>& rows, u32 slices, u32 b,
                                             const LiveCell& c, bool sums, int wave, int waves, u64& before, const F& list, const u32* listed = nullptr, u32 most = 0)
{
    constexpr int U = 2;
    const int lane = threadIdx.x & (WAVE - 1), P = all.P, R = all.R;
    if constexpr (PRED) {
        for (int p = wave * WAVE + lane; p - lane < P; p += waves * WAVE) {
            if (listed && uniform(*(volatile const u32*)listed) > most) return;
            if (p < P) before += rows.entries(p, typename CellRows<PRED>::Window{}, c.first, c.last, list);
        }
    } else {
        // Eight lanes to a row, an entry each, 64 U rows in flight: a lane's loads of eight entries of a row of its own would
        // ask the cache for 64 lines eight times over.
        constexpr u32 W = CellRows<PRED>::W;
        const u32 k = (u32)lane & (W - 1);
        for (int p0 = wave * WAVE * U; p0 < P; p0 += waves * WAVE * U) {
            if (listed && uniform(*(volatile const u32*)listed) > most) return;
            u32 from[U], pending = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = p0 + u * WAVE + lane;
                from[u] = rows.start(all.range(space, slices, b, c.slice, p < P ? p : P - 1), c.at);
            }
            i64 v[U][W];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (u32 j = 0; j < W; ++j) {
                    const int r = (int)(j * W) + (lane >> 3), p = p0 + u * WAVE + r;
                    const u32 i = (u32)__shfl((int)from[u], r) + k;
                    v[u][j] = rows.inst[(size_t)(p < P ? p : P - 1) * R + (i < (u32)R ? i : (u32)R - 1)];
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (u32 j = 0; j < W; ++j) {
                    const u64 y = (u64)v[u][j] - rows.base;
                    const bool in = y >= c.first && y <= c.last;
                    const bool open = k == 0 ? y >= c.first : k == W - 1 && y <= c.last;      // the row goes on to that side
                    const u64 seen = __ballot(in || open);
                    if (seen == 0 && !sums) continue;      // (half of the times)
                    const int r = (int)(j * W) + (lane >> 3), p = p0 + u * WAVE + r;
                    const u32 s = (u32)__shfl((int)from[u], r);
                    const u64 ahead = dpp_take<DPP_WAVE_SHR1, 0xf>(0ull, y);
                    const u64 opens = __ballot(open && (k == 0 ? s > 0 : s + W < (u32)R)) >> (lane & ~7) & 0xff;
                    if (p < P && opens == 0 && in && s + k < (u32)R) list(y, k == 0 ? 0ull : ahead);
                    if (sums) {                            // the last entry before the cell
                        const u64 below = __ballot(y < c.first) >> (lane & ~7) & 0xff;
                        if (p < P && opens == 0 && below && k == (u32)__popcll(below) - 1) before += y;
                    }
                    if (p < P && opens != 0 && k == 0) pending |= 1u << (u * W + j);
                }
            while (pending) {                      // rows whose entries lie elsewhere
                const u32 q = (u32)__builtin_ctz(pending);
                pending &= pending - 1;
                const int p = p0 + (int)(q * W) + (lane >> 3);
                const uint2 range = all.range(space, slices, b, c.slice, p);
                before += rows.entries(p, rows.window(p, range, c.at), c.first, c.last, list);
            }
        }
    }
}

// A workgroup per instance: looks at its lowest cell, which rules out most of the others, and queues the rest.
template <int NT, bool PRED>
__global__ __launch_bounds__(NT, 4) void zl_slices_queue_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, int P, int R, u32 slices,
    void* __restrict__ workspace, u32 room,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    constexpr int NW = NT / WAVE;
    __shared__ u64 red[2 * NW];
    __shared__ u64 lx[NT], ld[NT];
    __shared__ u32 ranks[NW], at, listed, crowded_at;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x;
    const SliceSpace space = slice_space(workspace, B, slices, PRED ? 0 : P, room);
    const SlicePart* const parts = space.part + b * slices;
    i64 top = INT64_MAX;
    int flags = 0, left = 0;
    u32 cells = 0;
    for (u32 j = tid; j < slices; j += NT) {
        const SlicePart s = parts[j];
        top = s.top < top ? s.top : top;
        flags |= (int)s.flags;
        cells = s.cells > cells ? s.cells : cells;
        left |= s.left != 0;
    }
    const int unsorted = __syncthreads_or(flags & (int)EBSP_STATUS_UNSORTED), over = __syncthreads_or(flags & (int)EBSP_STATUS_OVERFLOW);
    left = __syncthreads_or(left);
    if (unsorted || over) {                                // (no results then)
        if (tid == 0) {
            barrier[b] = parts[0].base;
            wait[b] = 0;
            if (status) status[b] = (unsorted ? (int)EBSP_STATUS_UNSORTED : 0) | (over ? (int)EBSP_STATUS_OVERFLOW : 0);
            space.queued[b] = SliceQueued{0, 0, 0, 0, NO_CELL, 0, 0};
        }
        for (int p = tid; p < P; p += NT) iters[b * (i64)P + p] = 0;
        return;
    }
    top = (i64)uniform((u64)block_reduce<i64, NT>(top, (i64*)red, OpMin()));
    auto by_windows = [&] {
        if (tid == 0) {
            space.queued[b] = SliceQueued{(u64)top, 0, 0, 0, NO_CELL, 0, 0};
            space.rest[atomicAdd(&space.queue->rest, 1u)] = (u32)b;
        }
    };
    if (left) { by_windows(); return; }
    cells = uniform(block_reduce<u32, NT>(cells, (u32*)red, OpMax()));               // the most of a slice
    // the cells of all slices: a thread per cell, as many slices at once as that makes
    const u32 chunk = cells < (u32)NT ? cells : (u32)NT, at_once = (u32)NT / (chunk ? chunk : 1u);
    auto each = [&](const auto& f) {                       // f(the thread has a cell, its number, its bound): all threads together
        for (u32 j0 = 0; j0 < slices && cells; j0 += at_once)
            for (u32 c0 = 0; c0 < cells; c0 += chunk) {
                const u32 j = j0 + tid / chunk, c = c0 + tid % chunk;
                const bool is = tid < (int)(at_once * chunk) && j < slices && c < parts[j].cells;
                const u32 number = is ? (u32)(b * slices + j) * room + c : 0u;
                f(is, number, is ? space.cell[number].least : INT64_MAX);
            }
    };
    u64 low = U64_MAX, where = U64_MAX;
    each([&](bool is, u32 number, i64 least) {
        if (!is || least > top) return;
        const u64 l = (u64)least ^ (1ull << 63);
        if (l < low || (l == low && number < where)) { low = l; where = number; }
    });
    if (tid == 0) listed = 0;
    const u32 lowest = (u32)block_first_min<NT>(Best{low, where}, red).x;
    if (lowest == NO_CELL) { by_windows(); return; }       // (never: a slice's smallest upper bound is above some cell's lower one)
    const u32 slice = lowest / room;
    const SlicePart& s = space.part[slice];
    const LiveCell c = live_cell(s, space.cell[lowest], slice - (u32)(b * slices));
    const SliceRows<PRED> all{ts, le, iv, P, R};
    const bool exact = s.exact != 0;
    u64 before = 0;
    cell_entries<PRED>(space, all, all.of((u32)b, (u64)s.base), slices, (u32)b, c, !exact, wave, NW, before, [&](u64 y, u64 prev) {
        const u32 n = atomicAdd(&listed, 1u);
        if (n < (u32)NT) { lx[n] = y; ld[n] = y - prev; }
    });
    before = block_reduce<u64, NT>(before, red, OpAdd());  // (also: the list is there)
    const u32 n = listed;
    const bool seen = n <= (u32)NT;
    Best best{U64_MAX, U64_MAX};
    if (seen) {
        if (tid < (int)n) {
            const u64 x = lx[tid];
            u64 behind = 0, upto = before;
            for (u32 o = 0; o < n; ++o) {
                const u64 d = ld[o];
                if (lx[o] > x) behind += d; else upto += d;
            }
            if (x >= s.thr) best = Best{exact ? (u64)c.least + (u64)P * (x - c.first) + behind : (u64)P * x - upto, x};
        }
        best = block_first_min<NT>(best, red);
        top = best.d < (u64)top ? (i64)best.d : top;
    }
    u32 count = 0;
    each([&](bool is, u32 number, i64 least) { count += is && least <= top && !(seen && number == lowest) ? 1u : 0u; });
    count = block_reduce<u32, NT>(count, (u32*)red, OpAdd());
    // Many cells: workers whose waits repeat, searched by windows.  Those in step fill cells with more entries than a window's bucket may
    // hold, and take the general search there, or are searched by cells, but not by a wave's list: cell by cell they are read
    // eight entries to a row, and keys that are shifted three times.  us, by windows / by cells, within 20 us: stored 256 of 256 x
    // 1024 3237 / 4658, 1024 of 256 x 1024 11795 / 18377, 200 of 300 x 1024 4224 / 4225, 60 of 1021 x 1031 5018 / 2246; in
    // nanoseconds 256 of 256 x 1024 3578 / 16433, 60 of 1021 x 1031 5010 / 7113; predicted 1024 of 256 x 1024 11340 / 8102.
    const bool many = count > (u32)R / 4 + WAVE;
    const bool crowd = many && n > (PRED ? 1u : 2u) * BUCKET_LIMIT && exact && s.shift <= (u32)SLICE_FINE_LOG;
    if (many && !crowd) { by_windows(); return; }
    if (tid == 0) {
        at = atomicAdd(&space.queue->cells, count);
        if (crowd) crowded_at = atomicAdd(&space.queue->crowded, count);
        space.queued[b] = SliceQueued{(u64)top, count, at, 0, seen ? lowest : NO_CELL, crowd ? 1u : 0u, 0};
        if (seen) {
            u64* const to = (u64*)(space.cell + lowest);
            publish(to, best.x);
            publish(to + 1, best.d);
        }
    }
    __syncthreads();
    if (count == 0) {                                      // (what this workgroup has stored is read past the caches)
        if (wave == 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            instance_done<PRED>(space, all, (u32)b, slices, room, barrier, iters, wait, status);
        }
        return;
    }
    u32 to = at;
    each([&](bool is, u32 number, i64 least) {
        const bool live = is && least <= top && !(seen && number == lowest);
        const u64 votes = __ballot(live);
        __syncthreads();
        if (lane == 0) ranks[wave] = (u32)__popcll(votes);
        __syncthreads();
        u32 rank = (u32)__popcll(votes & ((1ull << lane) - 1)), all = 0;
        for (int w = 0; w < NW; ++w) { const u32 n = ranks[w]; if (w < wave) rank += n; all += n; }
        if (live) {
            space.order[to + rank] = number;
            if (crowd) space.crowded[crowded_at + (to - at) + rank] = number;
        }
        to += all;
    });
}

// A wave per cell, from the queue until it is empty, or, where the queue leaves most waves without one, a workgroup's four
// waves together (64 of 1024 x 4096, predicted, 1400 cells: 28 us by waves, 23 together; stored, with more cells, 122 and 163).  Up to 64 entries, a lane each.
template <bool PRED>
__global__ __launch_bounds__(256, 4) void zl_slices_cells_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, int P, int R, u32 slices,
    void* __restrict__ workspace, u32 room, i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    constexpr int NW = 4;
    __shared__ u64 lx[NW][WAVE], ld[NW][WAVE];
    __shared__ u32 listed[NW];
    __shared__ u64 shares[NW];
    const int lane = threadIdx.x & (WAVE - 1);
    const u32 wave = uniform((u32)threadIdx.x >> 6);
    const SliceSpace space = slice_space(workspace, B, slices, PRED ? 0 : P, room);
    const SliceRows<PRED> all{ts, le, iv, P, R};
    const u32 total = space.queue->cells;
    const bool together = total <= gridDim.x * NW / 2;      // (the same in every workgroup)
    const u32 list_of = together ? 0u : wave;
    for (u32 i = together ? blockIdx.x : blockIdx.x * NW + wave; i < total; i += together ? gridDim.x : gridDim.x * NW) {
        const u32 number = uniform(space.order[i]);
        const u32 slice = number / room, b = slice / slices;
        if (space.queued[b].many) continue;
        const SlicePart& s = space.part[slice];
        const LiveCell c = live_cell(s, space.cell[number], slice - b * slices);
        u64 w = U64_MAX, x = U64_MAX;
        bool look = c.least <= (i64)published(&space.queued[b].best);
        if (together) look = __syncthreads_or(look);       // (the answer may change; also: the list is free)
        if (look) {
            const CellRows<PRED> rows = all.of(b, (u64)s.base);
            if (lane == 0 && (!together || wave == 0)) listed[list_of] = 0;
            if (together) __syncthreads();
            __builtin_amdgcn_wave_barrier();
            auto list = [&](u64 y, u64 prev) {
                const u32 at = atomicAdd(&listed[list_of], 1u);
                if (at < (u32)WAVE) { lx[list_of][at] = y; ld[list_of][at] = y - prev; }
            };
            u64 before = 0;
            const bool exact = s.exact != 0;
            cell_entries<PRED>(space, all, rows, slices, b, c, !exact, together ? (int)wave : 0, together ? NW : 1, before, list, &listed[list_of], WAVE);
            if (!exact) before = last_lane(wave_incl_scan(before));
            if (together) {
                if (lane == 0) shares[wave] = before;
                __syncthreads();
                before = 0;
                for (int q = 0; q < NW; ++q) before += shares[q];
                if (wave != 0) continue;                   // (the first wave goes on alone)
            }
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const u32 n = uniform(listed[list_of]);
            if (n > (u32)WAVE) {                           // left to zl_slices_rest_kernel
                if (lane == 0) {
                    if (exact && s.shift <= (u32)SLICE_FINE_LOG) space.crowded[atomicAdd(&space.queue->crowded, 1u)] = number;
                    else space.crowded[space.cells - 1 - atomicAdd(&space.queue->wide, 1u)] = number;
                }
                continue;
            }
            if (lane < (int)n) {
                x = lx[list_of][lane];
                u64 behind = 0, upto = before;
                for (u32 o = 0; o < n; ++o) {
                    const u64 d = ld[list_of][o];
                    if (lx[list_of][o] > x) behind += d; else upto += d;
                }
                w = exact ? (u64)c.least + (u64)P * (x - c.first) + behind : (u64)P * x - upto;
                if (x < s.thr) w = x = U64_MAX;
            }
            wave_argmin(w, x);
            w = last_lane(w);
            x = last_lane(x);
        }
        if (together && wave != 0) continue;
        int last = 0;
        if (lane == 0) last = cell_done(space, b, number, w, x);
        if (__builtin_amdgcn_readfirstlane(last)) instance_done<PRED>(space, all, b, slices, room, barrier, iters, wait, status);
    }
}

template <int NT>
struct SliceCrowdedSmem {
    u64 fine[SLICE_FINE];
    u32 is[SLICE_FINE / 32];
    LiveCell cell[SLICE_SIDE];
    u64 thr[SLICE_SIDE], base[SLICE_SIDE], w[SLICE_SIDE], x[SLICE_SIDE];
    u32 number[SLICE_SIDE], inst[SLICE_SIDE], shift[SLICE_SIDE], last[SLICE_SIDE];
};

// Cells of more entries, by a workgroup, SIDE of them at a time (a round with one of more than FINE / SIDE values takes its cells one
// by one): one word per value.
template <int NT, bool PRED>
__device__ __forceinline__ void slices_crowded(unsigned char* smem, const SliceSpace& space, const SliceRows<PRED>& all, u32 i0, u32 total,
                                               u32 slices, u32 room, i64* __restrict__ barrier, int* __restrict__ iters,
                                               i64* __restrict__ wait, int* __restrict__ status)
{
    constexpr int NW = NT / WAVE, SIDE = SLICE_SIDE;
    SliceCrowdedSmem<NT>& sm = *(SliceCrowdedSmem<NT>*)smem;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6, P = all.P;
    if (tid < SIDE) {
        u32 number = 0xffffffffu, b = 0, shift = 0;
        LiveCell c{};
        u64 best = 0;
        if (i0 + tid < total) {
            number = space.crowded[i0 + tid];
            const u32 slice = number / room;
            b = slice / slices;
            const SlicePart s = space.part[slice];
            best = published(&space.queued[b].best);
            c = live_cell(s, space.cell[number], slice - b * slices);
            shift = s.shift;
            sm.thr[tid] = s.thr;
            sm.base[tid] = (u64)s.base;
        }
        sm.cell[tid] = c;
        sm.number[tid] = number;
        sm.inst[tid] = b;
        sm.shift[tid] = number == 0xffffffffu || c.least > (i64)best ? 255u : shift;        // 255: nothing to look at
        sm.w[tid] = sm.x[tid] = U64_MAX;
        sm.last[tid] = 0;
    }
    __syncthreads();
    bool wide = false;
#pragma unroll
    for (int c = 0; c < SIDE; ++c) wide |= sm.shift[c] != 255u && (1u << sm.shift[c]) > (u32)(SLICE_FINE / SIDE);
    for (int c0 = 0; c0 < SIDE; c0 += wide ? 1 : SIDE) {
        const u32 K = wide ? 1u : (u32)SIDE, slot = wide ? (u32)SLICE_FINE : (u32)(SLICE_FINE / SIDE);
        bool any = false;
        for (u32 c = 0; c < K; ++c) any |= sm.shift[c0 + c] != 255u;
        if (!any) continue;
        for (u32 c = 0; c < K; ++c)
            if (sm.shift[c0 + c] != 255u) {
                const u32 words = 1u << sm.shift[c0 + c];
                for (u32 q = tid; q < words; q += NT) sm.fine[c * slot + q] = 0;
                for (u32 q = tid; q < (words + 31) / 32; q += NT) sm.is[c * (slot / 32) + q] = 0;
            }
        __syncthreads();
        {
            const u32 ci = uniform((u32)wave % K);         // NW / K waves to a cell
            if (sm.shift[c0 + ci] != 255u) {
                const LiveCell c = sm.cell[c0 + ci];
                const u32 b = uniform(sm.inst[c0 + ci]), from = ci * slot;
                u64 before = 0;
                cell_entries<PRED>(space, all, all.of(b, uniform(sm.base[c0 + ci])), slices, b, c, false, (int)(wave / K), (int)(NW / K), before, [&](u64 x, u64 prev) {
                    const u32 at = from + (u32)(x - c.first);
                    atomicAdd(&sm.fine[at], x - prev);
                    atomicOr(&sm.is[at >> 5], 1u << (at & 31u));
                });
            }
        }
        __syncthreads();
        // the waits: a wave per cell, 64 words at a time from the last
        for (u32 c = wave; c < K; c += NW) {
            if (sm.shift[c0 + c] == 255u) continue;
            const LiveCell cell = sm.cell[c0 + c];
            const u64 thr = sm.thr[c0 + c];
            u64 behind = 0;                                // of the words behind
            Best got{U64_MAX, U64_MAX};
            for (int q = (1 << sm.shift[c0 + c]) - 1 - lane; q + lane >= 0; q -= WAVE) {
                const u64 d = q >= 0 ? sm.fine[c * slot + q] : 0ull;
                const u64 inc = wave_scan(d, OpAdd());
                if (q >= 0 && ((sm.is[c * (slot / 32) + (q >> 5)] >> (q & 31)) & 1u)) {
                    const Best one{(u64)cell.least + (u64)P * (u32)q + behind + inc - d, cell.first + (u32)q};
                    if (one.x >= thr && one.before(got)) got = one;
                }
                behind += last_lane(inc);
            }
            wave_argmin(got.d, got.x);
            if (lane == WAVE - 1) { sm.w[c0 + c] = got.d; sm.x[c0 + c] = got.x; }
        }
        __syncthreads();
    }
    if (tid < SIDE && sm.number[tid] != 0xffffffffu) sm.last[tid] = cell_done(space, sm.inst[tid], sm.number[tid], sm.w[tid], sm.x[tid]);
    __syncthreads();
    if (wave < SIDE && sm.last[wave]) instance_done<PRED>(space, all, uniform(sm.inst[wave]), slices, room, barrier, iters, wait, status);
    __syncthreads();
}

template <int NT>
struct RowsBetween : Rows {                      // of whole rows a part, which the thread that asks for a row knows: row tid + c * NT
    u32 lo[ROWS_PER_THREAD<NT>], hi[ROWS_PER_THREAD<NT>];
    __device__ __forceinline__ void range(int p, u32& first, u32& end) const
    {
        first = lo[0];
        end = hi[0];
#pragma unroll
        for (int c = 1; c < ROWS_PER_THREAD<NT>; ++c)
            if (p >= c * NT) { first = lo[c]; end = hi[c]; }
    }
};
template <int NT>
struct SlicesRestSmem {
    union {
        struct { u64 fine[SLICE_FINE]; u32 is[SLICE_FINE / 32]; };
        struct { u64 x[SLICE_LIST], d[SLICE_LIST]; };      // entries and additions
    };
    u64 sub[64];
    u64 red[3 * (NT / WAVE) + 2];
    u64 acc;                                     // S before a cell
    u32 listed;
};

// One workgroup's search of cells and slices of an instance, S before a cell from the rows.
template <int NT, int ITEMS, bool PRED>
struct RestSearch {
    unsigned char* smem;
    const SliceSpace& space;
    const SliceRows<PRED>& all;
    u32 b, slices;
    u64 base, thr;
    i64 top;             // no more than this, or it is not worth looking at
    Best best;
    __device__ __forceinline__ SlicesRestSmem<NT>& sm() const { return *(SlicesRestSmem<NT>*)smem; }
    __device__ __forceinline__ void take(const Best& got)
    {
        if (got.before(best)) best = got;
        if (best.d < (u64)top) top = (i64)best.d;
    }
    // the general search of the entries lo[p] up to hi[p] (not itself) of every row, all those in [first, last] (takes the whole of LDS)
    __device__ __forceinline__ void general(u64 first, u64 last, const u32 (&lo)[ROWS_PER_THREAD<NT>], const u32 (&hi)[ROWS_PER_THREAD<NT>])
    {
        __syncthreads();
        const Smem gm = carve<NT, ITEMS>(smem);
        RowsBetween<NT> rw = rows_of();
#pragma unroll
        for (int c = 0; c < ROWS_PER_THREAD<NT>; ++c) { rw.lo[c] = lo[c]; rw.hi[c] = hi[c]; }
        int none = 0;
        u64 w = U64_MAX, x = 0;
        zl_window<NT, ITEMS, true, false, RowsBetween<NT>>(gm, rw, thr, first, last, w, x, none);
        __syncthreads();
        if (w != U64_MAX) take(Best{w, x});
    }
    __device__ __forceinline__ void general(u64 first, u64 last)
    {
        const Rows rw = rows_of();
        u32 lo[ROWS_PER_THREAD<NT>], hi[ROWS_PER_THREAD<NT>];
#pragma unroll
        for (int c = 0; c < ROWS_PER_THREAD<NT>; ++c) {
            const int p = (int)threadIdx.x + c * NT;
            lo[c] = p < all.P ? row_lower_bound(rw, p, 0u, (u32)all.R, first) : 0u;
            hi[c] = p < all.P ? row_lower_bound(rw, p, lo[c], (u32)all.R, last + 1) : 0u;
        }
        general(first, last, lo, hi);
    }
    __device__ __forceinline__ RowsBetween<NT> rows_of() const
    {
        const CellRows<PRED> rows = all.of(b, base);
        RowsBetween<NT> rw;
        rw.inst = rows.inst; rw.le = rows.le; rw.iv = rows.iv;
        rw.par = nullptr; rw.cr = nullptr; rw.narrow = false; rw.wide = false; rw.stride = 0; rw.k0 = rw.k1 = 0;
        rw.P = all.P; rw.R = all.R; rw.base = base;
        return rw;
    }
    // a cell's entries from a list; false: it does not hold them
    __device__ __forceinline__ bool listed(const LiveCell& c)
    {
        __syncthreads();
        if (threadIdx.x == 0) { sm().acc = 0; sm().listed = 0; }
        __syncthreads();
        u64 s = 0;
        cell_entries<PRED>(space, all, all.of(b, base), slices, b, c, true, (int)threadIdx.x >> 6, NT / WAVE, s, [&](u64 x, u64 prev) {
            const u32 at = atomicAdd(&sm().listed, 1u);
            if (at < (u32)SLICE_LIST) { sm().x[at] = x; sm().d[at] = x - prev; }
        });
        s = wave_scan(s, OpAdd());
        if ((threadIdx.x & (WAVE - 1)) == WAVE - 1) atomicAdd(&sm().acc, s);
        __syncthreads();
        const u32 total = sm().listed;
        Best got{U64_MAX, U64_MAX};
        if (total <= (u32)SLICE_LIST)
            for (u32 e = threadIdx.x; e < total; e += NT) {
                const u64 x = sm().x[e];
                u64 S = sm().acc;
#pragma unroll 4
                for (u32 o = 0; o < total; ++o) {
                    const u64 d = sm().d[o];
                    S += sm().x[o] <= x ? d : 0ull;
                }
                const Best one{(u64)all.P * x - S, x};
                if (x >= thr && one.before(got)) got = one;
            }
        take(block_first_min<NT>(got, sm().red));          // (ends with a barrier)
        return total <= (u32)SLICE_LIST;
    }
    // a cell of any number of entries
    __device__ __forceinline__ void cell(const LiveCell& c)
    {
        if (listed(c)) return;
        const u64 span = c.last - c.first;
        const int tid = threadIdx.x, lane = tid & (WAVE - 1);
        const int bits = bit_length(span) - SLICE_FINE_LOG;
        const u32 fs = bits > 0 ? (u32)bits : 0u;          // fine cells are 2^fs values wide
        for (int q = tid; q < SLICE_FINE; q += NT) sm().fine[q] = 0;
        for (int q = tid; q < SLICE_FINE / 32; q += NT) sm().is[q] = 0;
        if (tid == 0) { sm().acc = 0; sm().listed = 0; }
        __syncthreads();
        u64 s = 0;
        cell_entries<PRED>(space, all, all.of(b, base), slices, b, c, true, tid >> 6, NT / WAVE, s, [&](u64 x, u64 prev) {
            const u32 q = (u32)((x - c.first) >> fs);
            atomicAdd(&sm().fine[q], x - prev);
            atomicOr(&sm().is[q >> 5], 1u << (q & 31u));
        });
        s = wave_scan(s, OpAdd());
        if (lane == WAVE - 1) atomicAdd(&sm().acc, s);
        __syncthreads();
        constexpr int CPT = SLICE_FINE / NT;
        u64 part = 0, sum;
        for (int j = 0; j < CPT; ++j) part += sm().fine[tid * CPT + j];
        const u64 S0 = sm().acc + block_excl_scan<u64, NT>(part, sm().red, sum);
        auto each = [&](const auto& f) {
            u64 S = S0;
            for (int j = 0; j < CPT; ++j) {
                const u32 q = (u32)(tid * CPT + j);
                S += sm().fine[q];
                if ((sm().is[q >> 5] >> (q & 31u)) & 1u) f(c.first + ((u64)q << fs), S);
            }
        };
        const u64 wide = (1ull << fs) - 1, P = (u64)all.P;
        if (fs == 0) {                                     // single values
            Best got{U64_MAX, U64_MAX};
            each([&](u64 x, u64 S) {
                const Best one{P * x - S, x};
                if (x >= thr && one.before(got)) got = one;
            });
            take(block_first_min<NT>(got, sm().red));
            return;
        }
        i64 up = INT64_MAX;
        each([&](u64 lo, u64 S) {
            const i64 w = (i64)(P * (lo + wide) - S);
            if (lo + wide >= thr && w < up) up = w;
        });
        up = block_reduce<i64, NT>(up, (i64*)sm().red, OpMin());
        top = up < top ? up : top;
        each([&](u64 lo, u64 S) {
            if ((i64)(P * lo - S) <= top) {
                const u32 at = atomicAdd(&sm().listed, 1u);
                if (at < 64u) sm().sub[at] = lo;
            }
        });
        __syncthreads();
        const u32 total = sm().listed;
        if (total > 64u) { general(c.first, c.last); return; }
        const u64 mine = sm().sub[lane];                   // (the searches take their place)
        const float part_of = 1.0f / (float)(span + 1);
        for (u32 q = 0; q < total; ++q) {
            const u64 lo = (u64)__shfl((i64)mine, (int)q);
            LiveCell one = c;
            one.first = lo;
            one.last = lo + wide < c.last ? lo + wide : c.last;
            one.at = c.at + (c.end_at - c.at) * (float)(lo - c.first) * part_of;
            if (!listed(one)) general(one.first, one.last);
        }
    }
};

// A slice by windows (see zl_window.h) without a crossing table: the rows are searched for each window's end, and windows are
// as wide as the ones before have shown to fit.  Behind one of few entries the next begins where an entry is, so that there are no
// more windows than entries, however far apart those are.  Windows that the fast search gives up are left to the general one.
// In step, they are then as narrow as that takes at once: cut by bisection, stored rows in step within 20 us, in nanoseconds, 60 of
// 1021 x 1031 took 224 ms, 5.0 so.
// What a window costs is a search of every row ahead of it (64 of 1024 x 4096, predicted, two intervals: 26 us a window, by windows
// with a table 14).  Measured and not kept: a kernel of its own, which no longer keeps 168 registers of a thread in memory beside
// the general search (2224 -> 1764 us, stored 48 of 1021 x 1031 1260 -> 1071, but a launch more in every call); the rows' ends in
// registers (3474); all cells added up again and the entries of those that may win listed by a second walk (1860, stored 1303),
// the same right behind the first walk (the kernel of all other inputs 1.3 times slower).
template <int NT, bool PRED>
struct SliceWindowsSmem {
    __align__(16) unsigned char hot[WinHot<NT, 16, PRED>::BYTES];
    uint2 par[PRED ? SLICE_PMAX : 1];            // predicted rows: low words of first value and interval
    Partial found;
};
template <int NT, int ITEMS, bool PRED>
__device__ __forceinline__ void slice_windows(unsigned char* smem, RestSearch<NT, ITEMS, PRED>& search, const SlicePart& s)
{
    using H = HotCfg<NT, 16>;
    constexpr int RPT = ROWS_PER_THREAD<NT>;
    static_assert(RPT * NT >= SLICE_PMAX, "all rows in one round");
    SliceWindowsSmem<NT, PRED>& sm = *(SliceWindowsSmem<NT, PRED>*)smem;
    const Smem hot = WinHot<NT, 16, PRED>::carve(sm.hot);
    const int tid = threadIdx.x, P = search.all.P, R = search.all.R;
    const u64 base = search.base;
    const CellRows<PRED> rows = search.all.of(search.b, base);
    auto row_of = [&](int p) -> SliceRow<PRED> {
        SliceRow<PRED> r;
        r.R = (u32)R;
        if constexpr (PRED) {
            r.step = (u64)rows.iv[p];
            r.f = (u64)rows.le[p] + r.step - base;
            r.rcp = r.step ? 1.0 / (double)r.step : 0.0;
        } else {
            r.row = rows.inst + (size_t)p * R;
            r.base = base;
            r.f = (u64)r.row[0] - base;
            r.l = (u64)r.row[R - 1] - base;
        }
        return r;
    };
    Rows rw;
    rw.inst = rows.inst; rw.le = nullptr; rw.iv = nullptr;
    rw.P = P; rw.R = R; rw.base = base;
    rw.cr = nullptr; rw.narrow = true; rw.wide = s.far != 0; rw.stride = 0; rw.k0 = rw.k1 = 0;
    InstInfo ii{};
    ii.base = s.base;
    ii.thr = s.thr;
    const bool fits = (u64)P * (u64)R < HOT_MAX_ENTRIES;
    u64 a = s.from, width = (s.to - s.from) / 16 + 1;
    constexpr u32 GENERAL = WinCfg<NT, ITEMS>::CAP_WIDE;
    u32 limit = H::CAP;                                    // entries of a window
    u32 lo[RPT], hi[RPT];
#pragma unroll
    for (int c = 0; c < RPT; ++c) {
        const int p = tid + c * NT;
        lo[c] = hi[c] = 0;
        if (p < P) lo[c] = row_of(p).below(a);
    }
    while (a <= s.to) {
        if (width > 0xffffffffull) width = 0xffffffffull;
        const u64 el = s.to - a < width ? s.to : a + width - 1;
        u32 mine = 0;
        int far = 0;                                       // distances that do not fit 32 bits
        if constexpr (PRED) rw.par = sm.par;
#pragma unroll
        for (int c = 0; c < RPT; ++c) {
            const int p = tid + c * NT;
            if (p < P) {
                const SliceRow<PRED> r = row_of(p);
                hi[c] = r.below(el + 1);
                hi[c] = hi[c] < lo[c] ? lo[c] : hi[c];
                mine += hi[c] - lo[c];
                if (s.far && (PRED || hi[c] > lo[c]))      // (of stored rows without an entry zl_place_rows takes the whole values)
                    far |= (((hi[c] > lo[c] ? r.at(lo[c]) : a) - (lo[c] ? r.at(lo[c] - 1) : a)) >> 32) != 0;
                if constexpr (PRED) sm.par[p] = make_uint2((u32)((u64)r.f + base), (u32)r.step);
            }
        }
        const u32 count = block_reduce<u32, NT>(mine, (u32*)hot.red, OpAdd());
        far = __syncthreads_or(far);
        auto narrower = [&] {
            width = (u64)((double)(el - a + 1) * (0.75 * limit) / (double)count);
            width = width ? width : 1;
        };
        if (count > limit && el > a) { narrower(); continue; }
        if (count > 0) {
            WinVal wv;
            wv.A = a;
            wv.Elast = el;
            wv.scale = far ? 0u : linear_scale(el - a, (u32)H::NB);
            wv.inv52 = wv.scale ? (1ull << 52) / wv.scale : 0;
            wv.pad_ = 0;
            window_search<NT, 16, unsigned short, PRED>(hot, rw, wv, ii, fits && !far, lo, hi, &search.space.queued[search.b].best, &sm.found);
            __syncthreads();
            const Partial f = sm.found;
            __syncthreads();
            if (f.wait == U64_MAX && f.brel == DEFERRED_WINDOW) {
                // (workers in step: as many entries as the general search takes at once, which otherwise looks for where to cut)
                if (count > GENERAL && el > a) { limit = GENERAL; narrower(); continue; }
                search.general(a, el, lo, hi);
            } else {
                if (f.wait != U64_MAX) search.take(Best{f.wait, f.brel});
                limit = limit < (u32)H::CAP / 2 ? 2 * limit : (u32)H::CAP;
            }
        }
        u64 next = el + 1;
        if (count < (u32)H::CAP / 4) {
            next = U64_MAX;
#pragma unroll
            for (int c = 0; c < RPT; ++c) {
                const int p = tid + c * NT;
                if (p < P && hi[c] < (u32)R) {
                    const u64 x = row_of(p).at(hi[c]);
                    next = x < next ? x : next;
                }
            }
            next = block_reduce<u64, NT>(next, hot.red, OpMin());
        }
#pragma unroll
        for (int c = 0; c < RPT; ++c) lo[c] = hi[c];
        if (el == s.to) break;
        a = next;
        if (count < limit / 2) width *= 2;
    }
}

template <int NT, int ITEMS, bool PRED>
__global__ __launch_bounds__(NT, (PRED ? 2 : 4)) void zl_slices_rest_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, int P, int R, u32 slices,
    void* __restrict__ workspace, u32 room, i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    using G = WinCfg<NT, ITEMS>;
    constexpr size_t BYTES0 = sizeof(SlicesRestSmem<NT>) > G::BYTES ? sizeof(SlicesRestSmem<NT>) : G::BYTES;
    constexpr size_t BYTES = sizeof(SliceWindowsSmem<NT, PRED>) > BYTES0 ? sizeof(SliceWindowsSmem<NT, PRED>) : BYTES0;
    static_assert(sizeof(SliceCrowdedSmem<NT>) <= BYTES && NT / WAVE >= SLICE_SIDE, "the cells of more entries use the same memory, a wave each in the end");
    __shared__ __align__(16) unsigned char smem[BYTES];
    __shared__ u32 last;
    const int tid = threadIdx.x;
    const SliceSpace space = slice_space(workspace, B, slices, PRED ? 0 : P, room);
    const SliceRows<PRED> all{ts, le, iv, P, R};
    const u32 crowded = space.queue->crowded;
    for (u32 i = blockIdx.x * SLICE_SIDE; i < crowded; i += gridDim.x * SLICE_SIDE)
        slices_crowded<NT, PRED>(smem, space, all, i, crowded, slices, room, barrier, iters, wait, status);
    // wide cells, and the slices of the instances that are searched by windows: one after the other
    const u32 wide = space.queue->wide;
    const u64 units = (u64)wide + (u64)space.queue->rest * slices;
    for (u64 u = blockIdx.x; u < units; u += gridDim.x) {
        const bool is_cell = u < wide;
        const u32 number = is_cell ? space.crowded[space.cells - 1 - u] : 0u;
        const u32 slice = is_cell ? number / room : space.rest[(u - wide) / slices] * slices + (u32)((u - wide) % slices);
        const SlicePart& s = space.part[slice];
        const u32 b = slice / slices;
        RestSearch<NT, ITEMS, PRED> search{smem, space, all, b, slices, (u64)s.base, s.thr, 0, Best{U64_MAX, U64_MAX}};
        // (one thread asks: the answer may change)
        __syncthreads();
        if (tid == 0) *(u64*)smem = published(&space.queued[b].best);
        __syncthreads();
        search.top = (i64)*(u64*)smem;
        __syncthreads();
        if (is_cell) search.cell(live_cell(s, space.cell[number], slice - b * slices));
        else if (s.from <= s.to) slice_windows<NT, ITEMS, PRED>(smem, search, s);
        __syncthreads();
        if (tid == 0) {
            if (is_cell) last = cell_done(space, b, number, search.best.d, search.best.x) ? 1u : 0u;
            else {
                u64* const to = (u64*)(space.result + slice);
                publish(to, search.best.d);
                publish(to + 1, search.best.x);
                if (search.best.d != U64_MAX) atomicMin(&space.queued[b].best, search.best.d);
                last = count_published(&space.queued[b].ended) + 1 == slices ? 1u : 0u;
            }
        }
        __syncthreads();
        if (!last) continue;                               // (a barrier before it is written again)
        if (is_cell) {
            if (tid < WAVE) instance_done<PRED>(space, all, b, slices, room, barrier, iters, wait, status);
            continue;
        }
        asm volatile("" ::: "memory");
        Best best{U64_MAX, U64_MAX};
        for (u32 j = tid; j < slices; j += NT) {
            u64* const from = (u64*)(space.result + (size_t)b * slices + j);
            const Best got{published(from), published(from + 1)};
            if (got.before(best)) best = got;
        }
        best = block_first_min<NT>(best, (u64*)smem);
        const CellRows<PRED> rows = all.of(b, (u64)s.base);
        const i64 bar = (i64)((u64)s.base + best.x);
        if (tid == 0) {
            barrier[b] = bar;
            wait[b] = (i64)best.d;
            if (status) status[b] = 0;
        }
        for (int p = tid; p < P; p += NT) iters[(size_t)b * P + p] = zl_iters_of(rows.inst, rows.le, rows.iv, p, R, bar);
    }
}

}  // namespace
