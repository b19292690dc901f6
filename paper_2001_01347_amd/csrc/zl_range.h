// The search under the objective max(Z) - min(Z).
// Part of the ZipLine library (see zipline.hip); device code for gfx950.
#pragma once
#include "zl_window.h"

namespace {

// The paper's formal objective (Section III): d_Z = max(Z) - min(Z).  For a barrier
// c the tightest Z holds every worker's latest timestamp <= c, so
// d(c) = c - min_p last_p(c); the search returns the first minimum over the
// timestamps c >= max_p t[p][0] (Algorithm 2 evaluates exactly these states of Z).
//
// The general search (zl_range_window), for what the search by successors below gives up: one value
// interval [a, el] of whole rows is handled by one workgroup: the entries are gathered as
// (key = value - a, next = the same worker's next value - a, or NEVER) plus, for the
// first entry of a row inside the interval, gone = a - the worker's last value
// before the interval (NEVER if the worker has none: it has not finished an
// iteration yet), and sorted by key (zl_sort).  At sorted position k:
//   * a worker whose first entry in the interval lies at a position > k (or that has
//     no entry in it) still stands at its value before the interval: the largest
//     `gone` over those workers, G(k), is a suffix maximum, and d = key_k + G(k);
//   * if there is no such worker, min(Z) is the first entry j whose successor has
//     not arrived yet (next_j > key_k): with M(j) the prefix maximum of next,
//     j = #{ j' : M(j') <= key_k } (M is monotone: a binary search), d = key_k - key_j.
// Entries equal to key_k at later positions are treated as not yet arrived; that can
// only raise d at position k, and the last position of the run of equal keys sees
// them all, so the minimum over all positions is the minimum over the timestamps.
// An interval is at most 2^32 - 2 wide (keys and the NEVER mark share 32 bits); a `next`
// beyond the interval is as good as NEVER inside it.  `gone` reaches back before the
// interval: it fits 32 bits when the instance's value spread does (below 2^32 - 1);
// otherwise (FAR) it is kept in 64 bits, its upper half in a third plane.
constexpr u32 NEVER = 0xffffffffu;
constexpr u64 RANGE_PIECE_MAX = 0xfffffffeull;          // widest interval searched in one go

template <bool FAR> struct Gone { using type = u32; static constexpr u32 never = NEVER; };
template <> struct Gone<true> { using type = u64; static constexpr u64 never = U64_MAX; };

template <class T, int NT, class Op>
__device__ __forceinline__ T block_excl_scan_op(T v, T* red, Op op)      // `red` holds NT/64 T's
{
    constexpr int NW = NT / WAVE;
    constexpr T id = Op::template identity<T>();
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x >> 6;
    const T inc = wave_scan(v, op);
    if (lane == WAVE - 1) red[wave] = inc;
    T before = dpp_take<DPP_WAVE_SHR1, 0xf>(id, inc);       // exclusive inside the wave
    if (lane == 0) before = id;
    __syncthreads();
    T base = id;
#pragma unroll 4
    for (int w = 0; w < NW; ++w)
        if (w < wave) base = op(base, red[w]);
    __syncthreads();
    return op(base, before);
}

// Gather for the range objective; returns the number of entries (nothing useful is
// stored if it exceeds `cap`).  absent = the largest `gone` over the workers without
// an entry in the interval (this thread's share).
template <int NT, bool FAR>
__device__ __forceinline__ int zl_range_gather(const Smem& sm, const Rows& rw, u64 a, u64 el, bool lx, bool rx,
                                               int cap, typename Gone<FAR>::type& absent, int& bad)
{
    using G = typename Gone<FAR>::type;
    const u64 width = el - a;
    const int tid = threadIdx.x;
    u32* rowoff = sm.cnt;
    u32* rowlo = sm.cnt + NT;
    int total = 0;
    for (int p0 = 0; p0 < rw.P; p0 += NT) {
        const int p = p0 + tid;
        u32 lo = 0, hi = 0;
        if (p < rw.P) {
            sub_range(rw, p, a, el, lx, rx, lo, hi);
            if (lo == hi) {
                const G gone = lo > 0 ? (G)(a - rw.rel(p, lo - 1)) : Gone<FAR>::never;
                absent = gone > absent ? gone : absent;
            }
        }
        u32 chunk;
        const u32 off = block_excl_scan<u32, NT>(hi - lo, (u32*)sm.red, chunk);
        rowoff[tid] = off;
        rowlo[tid] = lo;
        __syncthreads();
        const int room = cap - total;
        const int take = (int)chunk < room ? (int)chunk : room;
        const int nrows = (rw.P - p0) < NT ? (rw.P - p0) : NT;
        for (int e = tid; e < take; e += NT) {
            int l = 0, h = nrows;                 // the last row r with rowoff[r] <= e
            while (h - l > 1) {
                const int m = (l + h) >> 1;
                if (rowoff[m] <= (u32)e) l = m; else h = m;
            }
            const u32 i = rowlo[l] + ((u32)e - rowoff[l]);
            const i64* src = rw.inst + (size_t)(p0 + l) * rw.R + i;
            const i64 cur = src[0];
            const u64 rel = (u64)cur - rw.base;
            u32 next = NEVER;
            G gone = 0;
            if (i + 1 < (u32)rw.R) {
                const i64 nxt = src[1];
                bad |= (nxt < cur);
                const u64 nrel = (u64)nxt - rw.base - a;
                next = FAR && nrel > width ? NEVER : (u32)nrel;
            }
            if (i == rowlo[l]) {                  // the row's first entry inside the interval
                gone = Gone<FAR>::never;
                if (i > 0) {
                    const i64 prv = src[-1];
                    bad |= (cur < prv);
                    gone = (G)(a - ((u64)prv - rw.base));
                }
            }
            const int slot = phys(total + e);
            sm.recs[slot] = (u64)(u32)(rel - a) | ((u64)next << 32);
            sm.dhi[slot] = (u32)gone;
            if (FAR) sm.ext[slot] = (u32)((u64)gone >> 32);
        }
        total += (int)chunk;
        __syncthreads();
    }
    return total;
}

// The search over the sorted entries [0, total); thread t owns positions
// [t*items, (t+1)*items).  Returns the first minimum (d, key); d == U64_MAX: none.
template <int NT, bool FAR>
__device__ __forceinline__ void zl_range_scan_argmin(const Smem& sm, int items, int total, u64 a, u64 thr,
                                                     typename Gone<FAR>::type absent_all, u64& best_d, u32& best_key)
{
    using GT = typename Gone<FAR>::type;
    u64* recs = sm.recs;
    auto gone = [&](int slot) -> GT { return FAR ? (GT)(((u64)sm.ext[slot] << 32) | sm.dhi[slot]) : (GT)sm.dhi[slot]; };
    GT* mirror = (GT*)sm.cnt;                    // NT of them (the counter plane holds 2*NT words at least)
    const int tid = threadIdx.x;
    const int q0 = tid * items < total ? tid * items : total;
    const int qe = q0 + items < total ? q0 + items : total;
    // M: prefix maximum of `next`, written over `next`
    u32 mine = 0;
    for (int q = q0; q < qe; ++q) { const u32 nx = (u32)(recs[phys(q)] >> 32); mine = nx > mine ? nx : mine; }
    u32 run = block_excl_scan_op<u32, NT>(mine, (u32*)sm.red, OpMax());
    for (int q = q0; q < qe; ++q) {
        const u64 r = recs[phys(q)];
        const u32 nx = (u32)(r >> 32);
        run = nx > run ? nx : run;
        recs[phys(q)] = (u64)(u32)r | ((u64)run << 32);
    }
    // G: largest `gone` over the positions behind the thread's own (threads in mirrored order)
    GT far = 0;
    for (int q = q0; q < qe; ++q) { const GT g = gone(phys(q)); far = g > far ? g : far; }
    mirror[NT - 1 - tid] = far;
    __syncthreads();
    const GT mv = mirror[tid];
    __syncthreads();
    const GT behind_m = block_excl_scan_op<GT, NT>(mv, (GT*)sm.red, OpMax());   // for thread NT-1-tid
    mirror[NT - 1 - tid] = behind_m;
    __syncthreads();                              // also: every M is in place
    GT G = mirror[tid];
    G = absent_all > G ? absent_all : G;

    u64 bd = U64_MAX;
    u32 bq = 0xffffffffu, bk = 0;
    for (int q = qe - 1; q >= q0; --q) {          // right to left: G covers the positions behind q
        const u32 key = (u32)recs[phys(q)];
        if (a + key >= thr && G != Gone<FAR>::never) {
            u64 d;
            bool ok = true;
            if (G > 0) {
                d = (u64)key + G;
            } else {
                int l = 0, h = total;             // number of positions j with M(j) <= key
                while (l < h) {
                    const int m = (l + h) >> 1;
                    if ((u32)(recs[phys(m)] >> 32) <= key) l = m + 1; else h = m;
                }
                ok = l < total;
                d = ok ? (u64)(key - (u32)recs[phys(l)]) : 0;
            }
            if (ok && (d < bd || (d == bd && (u32)q < bq))) { bd = d; bq = (u32)q; bk = key; }
        }
        const GT g = gone(phys(q));
        G = g > G ? g : G;
    }
    // block arg-min over (d, position): smaller d, then earlier position
    u64 pk = ((u64)bq << 32) | bk;
    wave_argmin(bd, pk);
    constexpr int NW = NT / WAVE;
    const int lane = tid & (WAVE - 1), wave = tid >> 6;
    u64* red = sm.red;
    __syncthreads();
    if (lane == WAVE - 1) { red[wave] = bd; red[NW + wave] = pk; }
    __syncthreads();
    bd = red[0]; pk = red[NW];
#pragma unroll 4
    for (int w = 1; w < NW; ++w) {
        const u64 od = red[w], ok = red[NW + w];
        if (od < bd || (od == bd && ok < pk)) { bd = od; pk = ok; }
    }
    __syncthreads();
    best_d = bd;
    best_key = (u32)pk;
}

// One interval [A, Elast]: gather, sort, search.  An interval wider than RANGE_PIECE_MAX
// (FAR only) or with more than CAP_WIDE entries is walked in pieces that do fit, the latter
// cut by bisection on the value (every piece is searched on its own: what a piece needs from outside it
// are the neighbouring entries of its rows, which the gather reads); a single value
// that alone occurs more than CAP_WIDE times is one candidate and is evaluated
// directly from the rows.  (bd, bb) is updated with the first minimum found.
template <int NT, int ITEMS, bool FAR>
__device__ __forceinline__ void zl_range_window(const Smem& sm, const Rows& rw, u64 thr, u64 A, u64 Elast,
                                                u64& bd, u64& bb, int& bad)
{
    using C = WinCfg<NT, ITEMS>;
    using GT = typename Gone<FAR>::type;
    constexpr int CAPW = C::CAP_WIDE;
    u64 a = A;
    bool lx = true;
    for (;;) {
        u64 el = Elast;
        bool rx = true;
        if (FAR && el - a > RANGE_PIECE_MAX) { el = a + RANGE_PIECE_MAX; rx = false; }
        GT absent = 0;
        int total = zl_range_gather<NT, FAR>(sm, rw, a, el, lx, rx, CAPW, absent, bad);
        bool single = false;
        if (total > CAPW) {
            if (count_interval<NT>(sm, rw, a, a, lx) > (u32)CAPW) {
                single = true;                     // the value `a` alone overflows a piece
                el = a;
            } else {
                u64 l = a, h = el;                 // count(a, l) <= CAPW < count(a, h)
                while (h - l > 1) {
                    const u64 m = l + ((h - l) >> 1);
                    if (count_interval<NT>(sm, rw, a, m, lx) <= (u32)CAPW) l = m; else h = m;
                }
                el = l;
                absent = 0;
                total = zl_range_gather<NT, FAR>(sm, rw, a, el, lx, false, CAPW, absent, bad);
            }
            rx = false;
        }
        if (single) {
            // candidate c = a: every row stops at its last entry <= a
            u64 far = 0;
            int missing = 0;
            for (int p = threadIdx.x; p < rw.P; p += NT) {
                u32 lo, hi;
                sub_range(rw, p, a, a, lx, false, lo, hi);
                if (hi > 0) { const u64 g = a - rw.rel(p, hi - 1); far = g > far ? g : far; } else missing = 1;
            }
            const u64 d = block_reduce<u64, NT>(far, sm.red, OpMax());
            missing = __syncthreads_or(missing);
            if (!missing && a >= thr && (d < bd || (d == bd && a < bb))) { bd = d; bb = a; }
        } else {
            const GT absent_all = block_reduce<GT, NT>(absent, (GT*)sm.red, OpMax());   // also orders the record writes
            if (total > 0) {
                const int items = (total + NT - 1) / NT;
                fill_sentinels<NT>(sm.recs, total, items);
                __syncthreads();
                zl_sort<NT, ITEMS, true, FAR>(sm, items, bit_length(el - a));
                u64 d;
                u32 key;
                zl_range_scan_argmin<NT, FAR>(sm, items, total, a, thr, absent_all, d, key);
                if (d != U64_MAX && (d < bd || (d == bd && a + key < bb))) { bd = d; bb = a + key; }
            }
        }
        if (rx) break;
        // continue at the smallest entry above el, if any
        u64 nxt = U64_MAX;
        int have = 0;
        for (int p = threadIdx.x; p < rw.P; p += NT) {
            u32 lo, hi;
            rw.range(p, lo, hi);
            const u32 i = row_lower_bound(rw, p, lo, hi, el + 1);
            if (i < hi) { const u64 v = rw.rel(p, i); nxt = v < nxt ? v : nxt; have = 1; }
        }
        nxt = block_reduce<u64, NT>(nxt, sm.red, OpMin());
        have = __syncthreads_or(have);
        if (!have || nxt > Elast || nxt <= el) break;
        a = nxt;
        lx = false;
    }
}

// ---------------------------------------------------------------------------
// The search by successors.  For an entry x let g(x) be the latest of all workers' first entries at or after x, the
// smallest barrier whose set Z holds nothing before x.  min over c of c - min(Z at c) is the minimum of g(x) - x over
// the entries x up to `lim`, the earliest of the rows' ends (behind it some worker has no successor): at the best c
// x = min(Z) gives g(x) <= c, and every g(x) is a candidate whose Z begins at x or later.  g never decreases, so of
// equal minima the first x has the first barrier.
//
// With prev(y) the entry before y in its row (a row's first entry: before everything, so g >= thr), g(x) is the
// largest y with prev(y) < x.  So no order, count or sum is needed: one LDS word per value cell keeps the largest y
// whose predecessor falls in the cell, a prefix maximum over the cells gives G, and for x in cell c
//     G(c - 1) <= g(x) <= G(c)        (exactly G(c - 1) if no predecessor in the cell is below x).
// A cell is 2^sh values wide; the cells span the values up to lim alone, where all rows are still running and their
// entries lie evenly.
//
// Each thread owns NB / NT neighbouring cells: their prefix maximum in place, `seed` before the first of them.
template <int NT, int NB>
__device__ __forceinline__ void cells_prefix_max(u32* cells, u32 seed, u32* red)
{
    constexpr int CPT = NB / NT;
    static_assert(CPT >= 4 && CPT % 4 == 0 && NB % NT == 0, "whole 16-byte words per thread");
    uint4* mine = (uint4*)cells + threadIdx.x * (CPT / 4);
    u32 top = 0;
#pragma unroll
    for (int i = 0; i < CPT / 4; ++i) {
        const uint4 q = mine[i];
        const u32 a = q.x > q.y ? q.x : q.y, b = q.z > q.w ? q.z : q.w, m = a > b ? a : b;
        top = m > top ? m : top;
    }
    u32 run = block_excl_scan_op<u32, NT>(top, red, OpMax());
    run = seed > run ? seed : run;
#pragma unroll
    for (int i = 0; i < CPT / 4; ++i) {
        uint4 q = mine[i];
        run = q.x > run ? q.x : run; q.x = run;
        run = q.y > run ? q.y : run; q.y = run;
        run = q.z > run ? q.z : run; q.z = run;
        run = q.w > run ? q.w : run; q.w = run;
        mine[i] = q;
    }
}

// First of equal minima (d, x) over the workgroup, for every thread: two words, or (NARROW: both below 2^32) packed in one.
struct Best {
    u64 d, x;
    __device__ __forceinline__ bool before(const Best& o) const { return d < o.d || (d == o.d && x < o.x); }
};
template <class T, int NT, class Op>
__device__ __forceinline__ T block_reduce_any(T v, u64* red, Op op)
{
    if constexpr (NT == WAVE) return last_lane(wave_scan(v, op));
    else return block_reduce<T, NT>(v, (T*)red, op);
}
template <int NT>
__device__ __forceinline__ Best block_first_min(Best v, u64* red)
{
    constexpr int NW = NT / WAVE;
    wave_argmin(v.d, v.x);
    if constexpr (NW == 1) return Best{last_lane(v.d), last_lane(v.x)};
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x >> 6;
    if (lane == WAVE - 1) { red[wave] = v.d; red[NW + wave] = v.x; }
    __syncthreads();
    v = Best{red[0], red[NW]};
#pragma unroll 4
    for (int w = 1; w < NW; ++w) {
        const Best o{red[w], red[NW + w]};
        if (o.before(v)) v = o;
    }
    __syncthreads();
    return v;
}

// An instance's facts from the ends of its rows.
struct RowEnds {
    i64 base;            // smallest first entry; the rest relative to it
    u64 thr, lim, range; // largest first, smallest last and largest last entry
};
template <int NT>                                          // own_first, own_last: of row threadIdx.x
__device__ __forceinline__ RowEnds row_ends(const i64* __restrict__ inst, int P, int R, u64* red, u64& own_first, u64& own_last)
{
    i64 mn = INT64_MAX, mxf = INT64_MIN, mxl = INT64_MIN, nml = INT64_MIN;       // the last one: of ~last
    own_first = own_last = 0;
    for (int p = threadIdx.x; p < P; p += NT) {
        const i64 f = inst[(size_t)p * R], l = inst[(size_t)p * R + R - 1];
        if (p < NT) { own_first = (u64)f; own_last = (u64)l; }
        mn = f < mn ? f : mn;
        mxf = f > mxf ? f : mxf;
        mxl = l > mxl ? l : mxl;
        nml = ~l > nml ? ~l : nml;
    }
    mn = block_reduce_any<i64, NT>(mn, red, OpMin());
    mxf = block_reduce_any<i64, NT>(mxf, red, OpMax());
    mxl = block_reduce_any<i64, NT>(mxl, red, OpMax());
    nml = block_reduce_any<i64, NT>(nml, red, OpMax());
    RowEnds e;
    e.base = (i64)uniform((u64)mn);
    own_first -= (u64)e.base;
    own_last -= (u64)e.base;
    e.thr = uniform((u64)mxf - (u64)mn);
    e.range = uniform((u64)mxl - (u64)mn);
    e.lim = ~nml < mn ? 0ull : uniform((u64)~nml - (u64)mn);      // (below base only in unsorted rows)
    return e;
}
__device__ __forceinline__ u32 cell_shift(u64 span, int log2_cells)     // smallest sh with span >> sh below 2^log2_cells
{
    const int bl = bit_length(span);
    return bl > log2_cells ? (u32)(bl - log2_cells) : 0u;
}

// First index in [0, R) of a sorted row whose value relative to base is at least v (R: none), given the row's ends f and
// l (relative): eight neighbouring entries at once from where evenly spaced ones would put it (one round trip; where
// iteration times vary by a fifth they hold it as a rule), galloping from there.  (Any row: the search ends and stays
// inside.)
struct RowProbe {
    static constexpr u32 W = 8;
    const i64* row;
    u32 R, s;
    u64 base, v, f, l;
    i64 w[W];
    __device__ __forceinline__ RowProbe(const i64* row_, u32 R_, u64 base_, u64 f_, u64 l_, u64 v_)
        : row(row_), R(R_), base(base_), v(v_), f(f_), l(l_)
    {
        s = 0;
        if (R > W && f < v && v <= l) {
            s = (u32)((float)(v - f) / (float)(l - f) * (float)(R - 1));
            s = s > W / 2 - 1 ? s - (W / 2 - 1) : 0u;
            s = s < R - W ? s : R - W;
        }
#pragma unroll
        for (u32 k = 0; k < W; ++k) w[k] = row[s + k < R ? s + k : R - 1];
    }
    __device__ __forceinline__ u32 index() const
    {
        if (f >= v) return 0;
        if (l < v) return R;
        u32 below = 0;
#pragma unroll
        for (u32 k = 0; k < W; ++k) below += (u64)w[k] - base < v ? 1u : 0u;
        if (R <= W) return below < R ? below : R;          // (the last entry stands for those that are not there: not below)
        if (below > 0 && below < W) return s + below;
        u32 lo = 0, hi = R - 1, step = W;                  // the entry at lo is below v, the one at hi not
        if (below) {
            lo = s + W - 1;
            while (lo + step < hi) {
                if ((u64)row[lo + step] - base < v) { lo += step; step *= 2; } else { hi = lo + step; break; }
            }
        } else {
            hi = s;                                        // (s > 0, or the row is not sorted)
            while (hi > lo + step) {
                if ((u64)row[hi - step] - base >= v) { hi -= step; step *= 2; } else { lo = hi - step; break; }
            }
        }
        while (hi > lo + 1) {
            const u32 m = lo + ((hi - lo) >> 1);
            if ((u64)row[m] - base < v) lo = m; else hi = m;
        }
        return hi;
    }
};
__device__ __forceinline__ u32 row_first_at_least(const i64* __restrict__ row, u32 R, u64 base, u64 v)
{
    return RowProbe(row, R, base, (u64)row[0] - base, (u64)row[R - 1] - base, v).index();
}

// The same (R - 1: none) for a row that has been found as far as index `from`: galloping from there, or from where evenly
// spaced entries would put it.
__device__ __forceinline__ u32 row_seek(const i64* __restrict__ row, u32 R, u64 base, u32 from, u64 v)
{
    auto below = [&](u32 i) { return (u64)row[i] - base < v; };
    if (!below(from)) return from;
    u32 lo = from, step = 1;                               // the entry at lo is below v
    const u64 f = (u64)row[0] - base, l = (u64)row[R - 1] - base;
    u32 g = f < v && v < l ? (u32)((float)(v - f) / (float)(l - f) * (float)(R - 1)) : 0u;
    g = g < R ? g : R - 1;
    if (g > lo + 8 && below(g - 4)) lo = g - 4;
    while (lo + step < R - 1 && below(lo + step)) { lo += step; step *= 2; }
    u32 hi = lo + step < R - 1 ? lo + step : R - 1;
    while (hi > lo + 1) {
        const u32 m = lo + ((hi - lo) >> 1);
        if (below(m)) lo = m; else hi = m;
    }
    return hi;
}

// Every row's entries up to the barrier (relative to base); thread p knows the ends of row p.
template <int NT>
__device__ __forceinline__ void store_iters(const i64* __restrict__ inst, int P, int R, u64 base, u64 barrier, u64 own_first, u64 own_last,
                                            int* __restrict__ iters)
{
    for (int p = threadIdx.x; p < P; p += NT) {
        const i64* row = inst + (size_t)p * R;
        const u64 f = p < NT ? own_first : (u64)row[0] - base, l = p < NT ? own_last : (u64)row[R - 1] - base;
        iters[p] = (int)RowProbe(row, (u32)R, base, f, l, barrier + 1).index();
    }
}

// Instances of at most 4096 entries: one workgroup each, the entries held in registers (wave w holds elements
// [w * 64 * items, (w + 1) * 64 * items), 64 neighbouring ones per item: prev(y) sits in the neighbouring lane).
// Every entry reads the two words of its own cell, so its bounds are tight: G(c - 1) - x and G(c) - x.  The entry with
// the smallest upper bound is the answer unless some entry's lower bound is smaller; those are evaluated one by one, the
// smallest first, each by one pass over the registers, until none is left below the best.  How many that takes depends
// on the values alone (about one where iteration times vary); RANGE_TRIES of them leave the instance to
// zl_range_window_kernel where SORT_REST says that it follows.
// Bound by the chain of one workgroup's steps and by the vector ALU.  4096 of 16 x 64: 77.8 us by a radix sort of
// every instance, 25 so; 16384 of 64 x 30: 607, 160.
constexpr int RANGE_TRIES = 96;

// Values spread over 2^32 and more (`wide`): keys, cells and bounds from the values shifted down to 32 bits, which widens
// the bounds; the candidates are then entries, evaluated from the values in memory.
template <int NT, int ITEMS, int NB, bool SORT_REST>
__device__ __forceinline__ bool zl_range_registers(u32* cells, u64* red, const i64* __restrict__ inst, int wbase, const i64 (&v)[ITEMS],
                                                   i64 ahead, u32 have, u32 heads, const RowEnds& ends, Best& best, int& bad)
{
    constexpr int LOG = __builtin_ctz((unsigned)NB);
    const bool wide = (ends.range >> 32) != 0;
    const u32 ms = wide ? (u32)bit_length(ends.range) - 32u : 0u;
    const u32 lim = (u32)(ends.lim >> ms), thr = (u32)(ends.thr >> ms);
    const u32 sh = cell_shift(lim, LOG);
    const int lane = threadIdx.x & (WAVE - 1);
    u32 inner = have & ~heads;                             // items with an entry before them in their row
    u32 key[ITEMS];
    u32 over = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const u64 rel = ((u64)v[j] - (u64)ends.base) >> ms;
        over |= (have >> j) & 1u ? (u32)(rel >> 32) : 0u;  // beyond the range only in unsorted rows
        key[j] = (u32)rel;
    }
    bad |= over != 0;
    asm volatile("" : "+v"(have), "+v"(inner));            // (the items' tests as lane masks would fill the scalar registers)
    const u32 first_prev = (u32)(((u64)ahead - (u64)ends.base) >> ms);
    auto prev_of = [&](int j) -> u32 {
        const u32 p = dpp_take<DPP_WAVE_SHR1, 0xf>(0u, key[j]);
        const u32 edge = j > 0 ? last_lane(key[j > 0 ? j - 1 : 0]) : first_prev;
        return lane == 0 ? edge : p;
    };
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const u32 p = prev_of(j);
        if ((inner >> j) & 1u) {
            bad |= p > key[j];
            if (p <= lim) atomicMax(&cells[p >> sh], key[j]);
        }
    }
    asm volatile("" : "+v"(have), "+v"(inner));
    if (wide) {                                            // the order of values whose keys are equal
#pragma unroll 1
        for (int j = 0; j < ITEMS; ++j)
            if ((inner >> j) & 1u) {
                const i64* e = inst + (wbase + j * WAVE + lane);
                bad |= e[0] < e[-1];
            }
    }
    __syncthreads();
    cells_prefix_max<NT, NB>(cells, thr, (u32*)red);
    if (threadIdx.x == 0) cells[-1] = thr;
    __syncthreads();
    // A bound (in keys) and what its candidate is called, in one word: its key, or (wide) its index.
    auto lower = [&](int j) -> u64 {
        const u32 g0 = cells[(int)(key[j] >> sh) - 1];
        return ((u64)(g0 > key[j] ? g0 - key[j] : 0u) << 32) | (wide ? (u32)(wbase + j * WAVE + lane) : key[j]);
    };
    u64 ub = U64_MAX, next = U64_MAX;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (((have >> j) & 1u) && key[j] <= lim) {
            const u32 g1 = cells[key[j] >> sh];
            const u64 u = ((u64)(g1 > key[j] ? g1 - key[j] : 0u) << 32) | key[j], l = lower(j);
            ub = u < ub ? u : ub;
            next = l < next ? l : next;
        }
    ub = block_reduce_any<u64, NT>(ub, red, OpMin());
    next = block_reduce_any<u64, NT>(next, red, OpMin());
    // (wide: the bound is no candidate, and an entry as good as it may be the first)
    Best top{ub >> 32, ub & 0xffffffffull};
    if (wide) top = Best{((ub >> 32) << ms) | ((1ull << ms) - 1), U64_MAX};
    for (int tries = 0;; ++tries) {
        const u64 d0 = next >> 32;
        if (next == U64_MAX) break;
        if (wide ? (d0 ? ((d0 - 1) << ms) + 1 : 0ull) > top.d : next >= ((top.d << 32) | top.x)) break;
        if (SORT_REST && tries == RANGE_TRIES) return false;
        // nothing below is worth keeping in registers from one try to the next
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) asm volatile("" : "+v"(key[j]));
        asm volatile("" : "+v"(have), "+v"(inner));
        Best got;
        if (wide) {
            const u64 x = (u64)inst[(u32)next] - (u64)ends.base;
            u64 g = ends.thr;
#pragma unroll 1
            for (int j = 0; j < ITEMS; ++j)
                if ((inner >> j) & 1u) {
                    const i64* e = inst + (wbase + j * WAVE + lane);
                    const u64 p = (u64)e[-1] - (u64)ends.base, y = (u64)e[0] - (u64)ends.base;
                    if (p < x) g = y > g ? y : g;
                }
            g = block_reduce_any<u64, NT>(g, red, OpMax());
            got = x <= ends.lim ? Best{g > x ? g - x : 0ull, x} : Best{U64_MAX, U64_MAX};
        } else {
            const u32 x = (u32)next;
            u32 g = thr;
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const u32 p = prev_of(j);
                if (((inner >> j) & 1u) && p < x) g = key[j] > g ? key[j] : g;
            }
            g = block_reduce_any<u32, NT>(g, red, OpMax());
            got = Best{(u64)(g > x ? g - x : 0u), (u64)x};
        }
        if (got.before(top)) top = got;
        u64 after = U64_MAX;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (((have >> j) & 1u) && key[j] <= lim) {
                const u64 l = lower(j);
                if (l > next) after = l < after ? l : after;
            }
        next = block_reduce_any<u64, NT>(after, red, OpMin());
    }
    best = top;
    return true;
}

template <int NT, int ITEMS, int NB, bool SORT_REST>
__global__ __launch_bounds__(NT, (NT == 64 ? 5 : 6)) void zl_range_instance_kernel(
    const i64* __restrict__ ts, int P, int R, int rshift,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ dmin, int* __restrict__ status)
{
    static_assert(ITEMS <= 32, "item masks are one word");
    __shared__ __align__(16) u32 cellmem[4 + NB];
    __shared__ u64 red[2 * (NT / WAVE) + 2];
    u32* const cells = cellmem + 4;                        // cells[-1]: the largest value before the first cell
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x;
    const int n = P * R;
    const i64* __restrict__ inst = ts + b * (i64)n;
    const int items = (n + NT - 1) / NT;
    const int wbase = wave * WAVE * items;
    i64 v[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int e = wbase + j * WAVE + lane;
        v[j] = (j < items && e < n) ? inst[e] : 0;
    }
    const i64 ahead = (wbase > 0 && wbase < n) ? inst[wbase - 1] : 0;     // element before the wave's first
    for (int c = tid; c < NB / 4; c += NT) ((uint4*)cells)[c] = make_uint4(0u, 0u, 0u, 0u);
    u64 own_first, own_last;                               // the ends of row `tid`
    const RowEnds ends = row_ends<NT>(inst, P, R, red, own_first, own_last);
    if constexpr (NT == WAVE) __syncthreads();             // (row_ends passed barriers otherwise)
    // which items exist, and which are a row's first entry (e / R for e < 2^16 by the rounded-up reciprocal)
    u32 have = 0, heads = 0;
    {
        const int e0 = wbase + lane;
        const int p0 = rshift >= 0 ? (e0 >> rshift) : (int)__umulhi((u32)e0, 0xffffffffu / (u32)R + 1u);
        int i = e0 - p0 * R;
        const int step = WAVE % R;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (j < items && e0 + j * WAVE < n) {
                have |= 1u << j;
                if (i == 0) heads |= 1u << j;
            }
            i += step;
            i = i >= R ? i - R : i;
        }
    }
    Best best{0ull, 0ull};
    int bad = 0;
    const bool found = zl_range_registers<NT, ITEMS, NB, SORT_REST>(cells, red, inst, wbase, v, ahead, have, heads, ends, best, bad);
    bad = __syncthreads_or(bad);
    if (!found && !bad) {                                  // (the order of the rows has been seen here)
        if (tid == 0) dmin[b] = DEFERRED;
        return;
    }
    const i64 bar = (i64)((u64)ends.base + best.x + best.d);
    if (tid == 0) {
        barrier[b] = bar;
        dmin[b] = (i64)best.d;
        if (status) status[b] = bad ? (int)EBSP_STATUS_UNSORTED : 0;
    }
    store_iters<NT>(inst, P, R, (u64)ends.base, best.x + best.d, own_first, own_last, iters + b * (i64)P);
}

// ---------------------------------------------------------------------------
// Larger instances: one workgroup per slice of the values up to lim (all of them, where the batch fills the chip by
// itself).  The entries are read once, from HBM, and not kept: what bounds it is that one reading (1024 of 256 x 1024:
// 390 us, 5.5 TB/s, without what follows it) and, behind it, two or three dependent round trips to HBM per cell looked
// at.  1024 of 256 x 1024: 1822 us by windows of an instance's sorted-out segments (a counting pass, then each entry
// again with both neighbours), 513 so; 64 of 1024 x 4096 1071, 605; 4096 of 64 x 256 859, 172; one of 1000 x 150 76, 37.

// What a slice found.
struct RangePart {
    u64 d, g;            // smallest max(Z) - min(Z) and its barrier, relative to base (d == U64_MAX: no entry)
    u32 flags;
    u32 left;            // the slice gave up: it is zl_range_window_kernel's
};
// What the workspace holds behind the slices' results: those of the slices that were left, and how many of an instance's have ended.
struct RangeRest {
    RangePart* part;
    u32* ended;
};
__device__ __forceinline__ RangeRest range_rest(RangePart* part, i64 all) { return RangeRest{part + all, (u32*)(part + 2 * all)}; }
ZL_FN size_t range_rest_bytes(i64 B, i64 slices) { return (size_t)B * ((size_t)slices * 2 * sizeof(RangePart) + sizeof(u32)); }

// The pairs of neighbouring entries (i - 1, i), from < i <= to, of a row: f(before, entry).  A whole wave, 128 entries a step, two
// neighbouring ones to a lane, U steps asked for ahead, the entry before a lane's from the neighbouring lane.
template <int U, class F>
__device__ __forceinline__ void row_pairs_ahead(const i64* __restrict__ row, u32 from, u32 to, const F& f)
{
    const u32 lane = threadIdx.x & (WAVE - 1);
    i64 carry = 0;
    for (u64 s = from; s <= to; s += U * 2 * WAVE) {       // (64 bits: to may be near 2^31)
        i64 v[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const u64 i = s + (u64)(u * 2 * WAVE) + 2 * lane;
            const i64* e = row + (i < to ? i : (u64)to - 1);
            v[u][0] = e[0];
            v[u][1] = e[1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const u64 i = s + (u64)(u * 2 * WAVE) + 2 * lane;
            i64 p = dpp_take<DPP_WAVE_SHR1, 0xf>((i64)0, v[u][1]);
            if (lane == 0) p = carry;
            carry = (i64)last_lane((u64)v[u][1]);
            if (i > from && i <= to) f(p, i < to ? v[u][0] : v[u][1]);
            if (i < to) f(v[u][0], v[u][1]);
        }
    }
}
// The same by LANES = 2^lanes_log lanes: fewer than a wave (short stretches) load both.  Whole waves ask for as much ahead as the
// stretch has.  us, an entry a lane and 256 ahead / two, 256 ahead / 512 / 1024 / by the stretch: 1024 of 256 x 1024 531 / 529 / 507 /
// 477 / 479, 64 of 1024 x 4096 595 / 583 / 581 / 620 / 569, 8192 of 64 x 128 236 / 224 / 239 / 320 / 230.
// MOST: the most steps; workgroups of small slices have no long stretches.  0: an entry a lane, 256 ahead, where registers are
// short (zl_range_window_kernel, which has nothing to do as a rule, 9.5 us for one of 1000 x 150 and 10.6 with two a lane).
template <int MOST = 8, class F>
__device__ __forceinline__ void row_pairs(const i64* __restrict__ row, u32 from, u32 to, int lanes_log, const F& f)
{
    const u32 lane = threadIdx.x & (WAVE - 1);
    if (MOST == 0 && lanes_log == 6) {
        constexpr int U = 4;
        i64 carry = 0;
        for (u64 s = from; s <= to; s += U * WAVE) {
            i64 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const u64 i = s + u * WAVE + lane;
                v[u] = row[i <= to ? i : (u64)to];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const u64 i = s + u * WAVE + lane;
                i64 p = dpp_take<DPP_WAVE_SHR1, 0xf>((i64)0, v[u]);
                if (lane == 0) p = carry;
                carry = (i64)last_lane((u64)v[u]);
                if (i > from && i <= to) f(p, v[u]);
            }
        }
    } else if (lanes_log == 6) {
        from = uniform(from);
        to = uniform(to);
        if (from >= to) return;
        if (MOST == 2 || to - from < 4 * WAVE) row_pairs_ahead<2>(row, from, to, f);
        else if (to - from < 8 * WAVE) row_pairs_ahead<4>(row, from, to, f);
        else row_pairs_ahead<8>(row, from, to, f);
    } else {
        const u32 lanes = 1u << lanes_log;
        for (u64 i = (u64)from + 1 + (lane & (lanes - 1)); i <= to; i += lanes) f(row[i - 1], row[i]);
    }
}

// One slice.  Each cell's bounds follow from G at its two ends; cells whose lower bound exceeds the smallest upper bound
// are dropped.  The cell with the smallest lower bound is looked at first, which as a rule leaves none.  A cell's entries
// and their successors are found by one search per row, listed, and evaluated exactly (inside a cell only successors of
// earlier entries of the cell can lie behind G of its first value).  Workers in step put a whole round of iterations
// into a cell, more entries than the list holds: there the cell's first entry x is evaluated (g(x) is that of the cell's
// first value) and settles the cell as a rule, because g of all entries behind it is the successor of x or later, an
// iteration away.  What of such a cell may still win is cut into cells of its own later: such intervals wait on a stack,
// and where a cell is one value, no list is needed.  Where an interval leaves more than RANGE_LEVEL of them (iterations
// as short as a cell is wide), it is cut into RANGE_LEVEL pieces instead.
// `cells` words hold (y >> ms) + 1, 0 where no predecessor falls in the cell.
// Workers in step, a round within 20 us of 100 ms, us, with every such cell on the stack and whole instances left to one
// workgroup's sort / so: 64 of 1024 x 4096 800 000 / 7800 (13 400 with 16 cells a walk), 300 of 600 x 100 13 900 / 490,
// 1100 of 300 x 300 41 800 / 2340, 2000 of 300 x 60 9870 / 830, 64 of 520 x 150 1320 / 277 (within 1000 us 2080 / 437), one
// of 1000 x 150 235 / 95.
constexpr int RANGE_ROUND_CELLS = 64;                     // cells looked at together
constexpr int RANGE_LEVEL = 16;                           // intervals that one interval leaves at most
constexpr int RANGE_WALK = 8;                             // cells that a thread walks along
constexpr int RANGE_STACK = 96;                           // intervals that wait
template <int NT, int NB, bool DEEP>
struct SliceSmem {
    static constexpr int LIST = NT < 512 ? NT : 512;      // entries of the cells looked at together
    static constexpr int LIVE = NT;                       // cells gathered at a time
    static_assert(NB <= 65536, "cells are kept as 16-bit numbers");
    u32 pad[4];
    u32 cells[NB];                                        // cells[-1] is pad[3]
    union {
        struct { u32 lo[NT], hi[NT]; };                   // index ranges of NT rows, while the entries are read
        struct {
            u64 lx[LIST], ln[LIST];                       // an entry and its successor
            u16 lc[LIST], cell[LIVE];                     // its cell's number among those looked at; the cells gathered
        };
    };
    u64 at_start[RANGE_ROUND_CELLS];                      // g of the cell's first value
    u64 first[DEEP ? RANGE_ROUND_CELLS : 1];              // the cell's first entry
    u64 red[2 * (NT / WAVE) + 2];
    static constexpr int STACK = DEEP ? RANGE_STACK : 1;
    u64 from[STACK], to[STACK], least[STACK];             // intervals and their lower bounds
    u32 listed, waiting;
};
template <bool WIDE> struct SliceWord { using type = u32; };          // values relative to base: below 2^31, or any
template <> struct SliceWord<true> { using type = u64; };

// DEEP: cells that are too full are gone into.  Otherwise the slice ends where it meets them, with false, for
// zl_range_window_kernel to begin anew: that code beside the rest costs every other slice 2 to 8 %, in registers.
template <int NT, int NB, bool WIDE, bool DEEP>
__device__ __forceinline__ bool zl_range_slice(SliceSmem<NT, NB, DEEP>& sm, const i64* __restrict__ inst, int P, int R, u32 slices, u32 k,
                                               int lanes_log, const RowEnds& ends, u64 own_first, u64 own_last, RangePart& out)
{
    using V = typename SliceWord<WIDE>::type;
    constexpr int LOG = __builtin_ctz((unsigned)NB), NW = NT / WAVE, STEPS = NB / NT / 4, MOST = DEEP ? 0 : NB >= 16384 ? 8 : 2;
    static_assert(NB % (4 * NT) == 0 && 4 * STEPS <= 32, "whole steps; a thread's cells are bits of a word");
    const int tid = threadIdx.x;
    const u64 base = (u64)ends.base;
    const u64 width = ends.lim / slices + 1;
    u64 A = width * k;
    out = RangePart{U64_MAX, 0ull, 0u, 0u};
    const bool empty = A > ends.lim;
    u64 E = ends.lim - A < width ? ends.lim : A + width - 1;              // (if not empty)
    u32 sh = empty ? 0u : cell_shift(E - A, LOG);
    const u32 ms = WIDE ? (u32)bit_length(ends.range) - 31u : 0u;
    const V rest = WIDE ? (V)((1ull << ms) - 1) : (V)0;
    int bad = 0;
    u64 start = ends.thr;                                  // g(A)
    auto pair = [&](i64 p, i64 y) {
        if (WIDE) {
            const u64 pr = (u64)p - base, yr = (u64)y - base;
            bad |= yr < pr;
            if (pr - A <= E - A) atomicMax(&sm.cells[(u32)((pr - A) >> sh)], (u32)(yr >> ms) + 1u);
        } else {
            const u64 yr = (u64)y - base;
            const u32 p32 = (u32)((u64)p - base), y32 = (u32)yr;
            bad |= (int)(y32 < p32) | (int)(yr >> 32);     // (in sorted rows all values are below 2^31)
            if (p32 - (u32)A <= (u32)(E - A)) atomicMax(&sm.cells[(p32 - (u32)A) >> sh], y32 + 1u);
        }
    };
    // the ends of row p, which thread p kept since the first pass over them
    auto first_in = [&](int p) -> u64 { return p == tid ? own_first : (u64)inst[(size_t)p * R] - base; };
    auto last_in = [&](int p) -> u64 { return p == tid ? own_last : (u64)inst[(size_t)p * R + R - 1] - base; };
    const int groups = NT >> lanes_log, group = tid >> lanes_log;
    if (slices > 1) {
        // the order of what lies behind lim: the rows' stretches there are shared out among the slices
        const u32 pieces = (slices + (u32)P - 1u) / (u32)P;
        const u64 units = (u64)P * pieces;
        const u64 u0 = units * k / slices, u1 = units * (k + 1) / slices;
        for (u64 u = u0 + group; u < u1; u += groups) {
            const i64* row = inst + (size_t)(u / pieces) * R;
            const u32 q = (u32)(u % pieces);
            const u32 t0 = row_first_at_least(row, (u32)R, base, ends.lim + 1);     // pairs up to (t0 - 1, t0) are the slices'
            if (t0 + 1 >= (u32)R) continue;
            const u64 len = (u64)R - 1 - t0;
            const u32 from = t0 + (u32)(len * q / pieces), to = t0 + (u32)(len * (q + 1) / pieces);
            row_pairs<MOST>(row, from, to, lanes_log, [&](i64 p, i64 y) { bad |= y < p; });
        }
    }
    if (tid == 0) { sm.listed = 0; sm.waiting = 0; }
    Best best{U64_MAX, U64_MAX};
    u64 top = U64_MAX;                                     // the best is no larger
    for (bool whole = slices == 1;; whole = false) {
        // the entries of all rows in [A, E]; `start` becomes g(A)
        if (!empty) {
            u64 far = whole ? start : 0ull;
            for (int p0 = 0; p0 < P; p0 += NT) {
                if (p0 > 0) __syncthreads();
                if (p0 + tid < P && !whole) {
                    const i64* row = inst + (size_t)(p0 + tid) * R;
                    const u64 f = first_in(p0 + tid), l = last_in(p0 + tid);
                    const RowProbe pa(row, (u32)R, base, f, l, A), pe(row, (u32)R, base, f, l, E + 1);
                    const u32 i0 = pa.index(), i1 = pe.index();
                    bad |= i1 < i0 || i0 >= (u32)R;
                    if (i0 < (u32)R) { const u64 s = (u64)row[i0] - base; far = s > far ? s : far; }
                    sm.lo[tid] = i0;
                    sm.hi[tid] = i1 < i0 ? i0 : i1;
                }
                __syncthreads();
                const int rows = P - p0 < NT ? P - p0 : NT;
                for (int r = group; r < rows; r += groups) {
                    const u32 i0 = whole ? 0u : sm.lo[r], i1 = whole ? (u32)R : sm.hi[r];
                    const u32 to = i1 < (u32)R ? i1 : (u32)R - 1u;
                    if (i0 < to) row_pairs<MOST>(inst + (size_t)(p0 + r) * R, i0, to, lanes_log, pair);
                }
            }
            start = block_reduce_any<u64, NT>(far, sm.red, OpMax());
        }
        bad = __syncthreads_or(bad);
        if (bad) out.flags = EBSP_STATUS_UNSORTED;
        if (empty || bad) return true;
        // lim is an entry (without a successor)
        if (E == ends.lim && tid == 0) atomicMax(&sm.cells[(u32)((E - A) >> sh)], 1u);
        __syncthreads();
        // G in place.  Every wave owns NB / NW neighbouring cells and walks them 256 at a time, four to a lane.
        const V A_ = (V)A, E_ = (V)E, wide_cell = (V)((1ull << sh) - 1);
        auto first_of = [&](u32 c) -> V { return A_ + ((V)c << sh); };
        auto last_of = [&](u32 c) -> V { const V h = A_ + ((V)c << sh) + wide_cell; return h < E_ ? h : E_; };
        auto low_bound = [&](u32 g0, u32 c) -> V {        // of cell c, g0 the word before it
            const V g = (V)(g0 - 1u) << ms, h = last_of(c);
            return g > h ? g - h : (V)0;
        };
        // (the best itself is the first of its kind: of equal ones behind it none can win.  Where `top` is only some cell's upper
        // bound, the entry that is as good is still to be found, anywhere)
        auto may_be = [&](u64 lb, u64 from) -> bool { return lb < top || (lb == top && (best.d > top || from <= best.x)); };
        auto wins = [&](V lb, u32 c) -> bool { return may_be((u64)lb, (u64)first_of(c)); };
        auto may_win = [&](u32 c) -> bool { return wins(low_bound(sm.cells[(int)c - 1], c), c); };
        const u32 lane = tid & (WAVE - 1), wave = tid >> 6;
        const u32 mine = wave * (NB / NW) + 4 * lane;      // the thread's k-th cell:
        auto cell_of = [&](int i) -> u32 { return mine + (u32)(i >> 2) * 256u + (u32)(i & 3); };
        const u32 seed = (u32)(start >> ms) + 1u;
        u32 todo = 0;                                      // cells that hold entries and have not been looked at
        Best low{U64_MAX, U64_MAX};                        // the smallest lower bound and its cell,
        u64 second = U64_MAX;                              // the thread's next one,
        Best first_low;                                    // and its own smallest
        {
            u32 m = 0;
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const uint4 q = *(const uint4*)(sm.cells + mine + i * 256);
                const u32 x = q.x > q.y ? q.x : q.y, y = q.z > q.w ? q.z : q.w, z = x > y ? x : y;
                m = z > m ? z : m;
            }
            m = last_lane(wave_scan(m, OpMax()));
            if (lane == 0) ((u32*)sm.red)[wave] = m;
            if (tid == 0) sm.pad[3] = seed;                // cells[-1]
            __syncthreads();
            u32 run = seed;
            for (u32 w = 0; w < wave; ++w) { const u32 x = ((u32*)sm.red)[w]; run = x > run ? x : run; }
            run = uniform(run);
            __syncthreads();
            V ub = std::numeric_limits<V>::max(), lb1 = ub, lb2 = ub;
            u32 lc1 = 0;
#pragma unroll 2
            for (int i = 0; i < STEPS; ++i) {
                const u32 c = mine + i * 256;
                uint4 q = *(const uint4*)(sm.cells + c);
                todo |= ((q.x ? 1u : 0u) | (q.y ? 2u : 0u) | (q.z ? 4u : 0u) | (q.w ? 8u : 0u)) << (4 * i);
                const u32 x = q.x > q.y ? q.x : q.y, y = q.z > q.w ? q.z : q.w;
                const u32 inc = wave_scan(x > y ? x : y, OpMax());
                u32 before = dpp_take<DPP_WAVE_SHR1, 0xf>(0u, inc);
                before = lane == 0 ? 0u : before;
                before = before > run ? before : run;
                const u32 end = last_lane(inc);
                run = end > run ? end : run;
                u32 g = before;
                auto cell = [&](u32& word, u32 at) {
                    const u32 g1 = word > g ? word : g;
                    if (word) {
                        const V lo = first_of(c + at), v = ((V)(g1 - 1u) << ms) | rest, u = v > lo ? v - lo : (V)0;
                        ub = u < ub ? u : ub;
                        const V l = low_bound(g, c + at);
                        if (l < lb1) { lb2 = lb1; lb1 = l; lc1 = c + at; }
                        else if (l < lb2) lb2 = l;
                    }
                    word = g = g1;
                };
                cell(q.x, 0u); cell(q.y, 1u); cell(q.z, 2u); cell(q.w, 3u);
                *(uint4*)(sm.cells + c) = q;
            }
            if (todo) { first_low = Best{(u64)lb1, (u64)lc1}; second = lb2 == std::numeric_limits<V>::max() ? U64_MAX : (u64)lb2; }
            else first_low = low;
            const u64 all_ub = block_reduce_any<V, NT>(ub, sm.red, OpMin());
            top = all_ub < top ? all_ub : top;
            low = block_first_min<NT>(first_low, sm.red);
        }
        // the gathered cells r .. r + K - 1, those that may still win; false: more entries than the list holds.  (Cell r + ci
        // has the place slot + ci of at_start.)
        auto look_at = [&](u32 r, u32 K, u32 slot) -> bool {
            auto cell_at = [&](u32 ci) -> u32 { return sm.cell[r + ci]; };
            u64* const at_start = sm.at_start + slot;
            for (u32 c = tid; c < K; c += NT) at_start[c] = 0;
            __syncthreads();
            for (u64 q = tid; q < (u64)K * (u32)P; q += NT) {
                const u32 ci = (u32)(q / (u32)P);
                const int p = (int)(q - (u64)ci * (u32)P);
                const u32 c = cell_at(ci);
                if (!may_win(c)) continue;
                const i64* row = inst + (size_t)p * R;
                u32 i = RowProbe(row, (u32)R, base, first_in(p), last_in(p), first_of(c)).index();
                if (i >= (u32)R) continue;                 // (never: the cell begins at lim or before)
                u64 x = (u64)row[i] - base, nx = (u64)row[i + 1 < (u32)R ? i + 1 : i] - base;
                atomicMax(&at_start[ci], x);
                if (sh == 0) continue;
                const u64 hi = last_of(c);
                while (x <= hi) {
                    const u32 at = atomicAdd(&sm.listed, 1u);
                    if (at >= (u32)sm.LIST) break;
                    sm.lx[at] = x; sm.ln[at] = nx; sm.lc[at] = (u16)ci;
                    if (++i >= (u32)R) break;
                    x = nx;
                    nx = (u64)row[i + 1 < (u32)R ? i + 1 : i] - base;
                }
            }
            __syncthreads();
            const u32 total = sm.listed;
            __syncthreads();
            if (tid == 0) sm.listed = 0;
            if (total > (u32)sm.LIST) return false;
            Best got{U64_MAX, U64_MAX};
            if (sh == 0) {                                 // the cell is its only value
                for (u32 ci = tid; ci < K; ci += NT)
                    if (may_win(cell_at(ci))) {
                        const u64 x = first_of(cell_at(ci));
                        const Best one{at_start[ci] - x, x};
                        if (one.before(got)) got = one;
                    }
            } else
                for (u32 e = tid; e < total; e += NT) {
                    const u64 x = sm.lx[e];
                    const u32 ci = sm.lc[e];
                    u64 g = at_start[ci];
                    for (u32 o = 0; o < total; ++o)
                        if (sm.lc[o] == ci && sm.lx[o] < x && sm.ln[o] > g) g = sm.ln[o];
                    const Best one{g > x ? g - x : 0ull, x};
                    if (one.before(got)) got = one;
                }
            got = block_first_min<NT>(got, sm.red);        // (ends with a barrier: the list may be written again)
            if (got.before(best)) best = got;
            top = best.d < top ? best.d : top;
            __syncthreads();
            return true;
        };
        // the first entries of the gathered cells r .. r + K - 1, where look_at finds them too full; at_start becomes g of what
        // lies behind them.  The cells are in order: a thread walks along a few of them in a row, from line to line.
        auto look_at_first = [&](u32 r, u32 K) {
            const u32 parts = (K + RANGE_WALK - 1) / RANGE_WALK;
            for (u32 c = tid; c < K; c += NT) { sm.at_start[c] = may_win(sm.cell[r + c]) ? 0 : U64_MAX; sm.first[c] = U64_MAX; }
            __syncthreads();
#pragma unroll 1
            for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
                for (u64 q = tid; q < (u64)P * parts; q += NT) {
                    const int p = (int)(q / parts);
                    const u32 part = (u32)(q % parts), from = part * K / parts, to = (part + 1) * K / parts;
                    const i64* row = inst + (size_t)p * R;
                    u32 i = 0;
                    u64 x = first_in(p), nx = (u64)row[R > 1 ? 1 : 0] - base;      // the row's entry at i and the next (the last one: again)
                    for (u32 ci = from; ci < to; ++ci) {
                        const u64 lo = first_of(sm.cell[r + ci]), g = sm.at_start[ci], f = sm.first[ci];
                        if (g == U64_MAX) continue;        // (cannot win)
                        if (x < lo) {
                            if (nx >= lo) { ++i; x = nx; }
                            else { i = row_seek(row, (u32)R, base, i, lo); x = (u64)row[i] - base; }
                            nx = (u64)row[i + 1 < (u32)R ? i + 1 : i] - base;
                        }
                        if (pass == 0) {
                            if (x > g) atomicMax(&sm.at_start[ci], x);
                            if (x < f && x >= lo && x <= last_of(sm.cell[r + ci])) atomicMin(&sm.first[ci], x);
                        } else if (x == f && nx > g)
                            atomicMax(&sm.at_start[ci], nx);
                    }
                }
                __syncthreads();
                if (pass == 0) {
                    Best got{U64_MAX, U64_MAX};
                    for (u32 ci = tid; ci < K; ci += NT)
                        if (sm.first[ci] != U64_MAX) {
                            const Best one{sm.at_start[ci] - sm.first[ci], sm.first[ci]};
                            if (one.before(got)) got = one;
                        }
                    got = block_first_min<NT>(got, sm.red);
                    if (got.before(best)) best = got;
                    top = best.d < top ? best.d : top;
                }
            }
        };
        const u32 level0 = sm.waiting;
        bool in_pieces = false;                            // the interval leaves too much
        u32 K = (u32)(4 * NT) / (u32)P;
        K = K < 1u ? 1u : (K > (u32)RANGE_ROUND_CELLS ? (u32)RANGE_ROUND_CELLS : K);
        for (int round = 0; !in_pieces; ++round) {
            // gathered: first the cell with the smallest lower bound, then what may still win, in most slices nothing (no
            // thread's smallest bound that was not looked at is among it)
            u32 have;
            if (round == 0) {
                if (low.d == U64_MAX) break;               // (no entries)
                const u32 c = (u32)low.x - wave * (NB / NW);                  // inside the wave's cells
                if (c < NB / NW && (c & 255u) >> 2 == lane) {
                    todo &= ~(1u << ((c >> 8) * 4 + (c & 3u)));
                    first_low.d = second;
                }
                if (tid == 0) sm.cell[0] = (u16)low.x;
                have = 1;
                __syncthreads();
            } else {
                u32 now_mask = 0;
                if (round == 1 && !__syncthreads_or(first_low.d <= top)) break;
#pragma unroll 2
                for (int i = 0; i < STEPS; ++i) {
                    const u32 c = mine + i * 256;
                    const uint4 q = *(const uint4*)(sm.cells + c);
                    const u32 g0 = sm.cells[(int)c - 1];
                    if (wins(low_bound(g0, c), c)) now_mask |= 1u << (4 * i);
                    if (wins(low_bound(q.x, c + 1), c + 1)) now_mask |= 2u << (4 * i);
                    if (wins(low_bound(q.y, c + 2), c + 2)) now_mask |= 4u << (4 * i);
                    if (wins(low_bound(q.z, c + 3), c + 3)) now_mask |= 8u << (4 * i);
                }
                now_mask &= todo;
                todo = now_mask;
                // in order, by way of a bit per cell
                static_assert(NB / 32 <= NT && NB / 32 <= 2 * SliceSmem<NT, NB, DEEP>::LIST, "a thread per word, in place of the list");
                u32* const bits = (u32*)sm.lx;
                if (tid < NB / 32) bits[tid] = 0;
                __syncthreads();
                for (u32 m = now_mask; m; m &= m - 1) {
                    const u32 c = cell_of(__ffs(m) - 1);
                    atomicOr(&bits[c >> 5], 1u << (c & 31u));
                }
                __syncthreads();
                u32 word = tid < NB / 32 ? bits[tid] : 0u, all;
                u32 at = block_excl_scan<u32, NT>((u32)__popc(word), (u32*)sm.red, all);
                for (; word && at < (u32)sm.LIVE; word &= word - 1, ++at) sm.cell[at] = (u16)(tid * 32 + __ffs(word) - 1);
                __syncthreads();
                if (all == 0) break;
                have = all < (u32)sm.LIVE ? all : (u32)sm.LIVE;
                const u32 last = sm.cell[have - 1];
                for (; now_mask; now_mask &= now_mask - 1) {
                    const int i = __ffs(now_mask) - 1;
                    if (cell_of(i) <= last) todo &= ~(1u << i);
                }
            }
            if constexpr (!DEEP) {
                for (u32 r = 0; r < have; r += K)
                    if (!look_at(r, have - r < K ? have - r : K, 0)) return false;
                __syncthreads();
                continue;
            }
            // the cells' first entries, then those not settled one by one
            u32 r = 0, group = 0, ci = 0;
            while (r < have && !in_pieces) {
                if (group == 0) {
                    group = have - r < (u32)RANGE_ROUND_CELLS ? have - r : (u32)RANGE_ROUND_CELLS;
                    look_at_first(r, group);
                    ci = 0;
                }
                u64 x = 0, h = 0, lb = 0;
                for (; ci < group; ++ci) {
                    const u32 c = sm.cell[r + ci];
                    const u64 g = sm.at_start[ci];
                    x = sm.first[ci];
                    h = (u64)last_of(c);
                    lb = g > h ? g - h : 0ull;
                    if (x < h && may_win(c) && may_be(lb, x + 1)) break;
                }
                __syncthreads();                           // (the cells' places may be written again)
                if (ci == group) { r += group; group = 0; continue; }
                const bool seen = look_at(r + ci, 1, ci);
                if (!seen) {                               // cut into cells of its own later
                    const u32 to = sm.waiting;
                    __syncthreads();
                    in_pieces = to - level0 >= (u32)RANGE_LEVEL;
                    if (tid == 0 && !in_pieces) {
                        if (to < (u32)RANGE_STACK) { sm.from[to] = x + 1; sm.to[to] = h; sm.least[to] = lb; }
                        sm.waiting = to + 1;
                    }
                }
                ++ci;
            }
            __syncthreads();
        }
        if constexpr (!DEEP) break;
        if (in_pieces) {
            const u32 n_cells = (u32)((E - A) >> sh) + 1u, per = (n_cells + RANGE_LEVEL - 1) / RANGE_LEVEL;
            const u32 at = level0 + (u32)tid, c = per * (u32)(RANGE_LEVEL - 1 - tid);        // (the first piece on top)
            if (tid < RANGE_LEVEL && at < (u32)RANGE_STACK) {
                const u32 z = c + per - 1 < n_cells ? c + per - 1 : n_cells - 1u;
                // (behind the interval's end: one that cannot win)
                sm.from[at] = c < n_cells ? (u64)first_of(c) : U64_MAX;
                sm.to[at] = c < n_cells ? (u64)last_of(z) : U64_MAX;
                const u64 g = c < n_cells ? (u64)((V)(sm.cells[(int)c - 1] - 1u) << ms) : 0ull;
                sm.least[at] = c >= n_cells ? U64_MAX : g > sm.to[at] ? g - sm.to[at] : 0ull;
            }
            if (tid == 0) sm.waiting = level0 + RANGE_LEVEL;
        }
        __syncthreads();
        u32 waiting = sm.waiting;
        if (waiting > (u32)RANGE_STACK) { out.left = 1; return true; }
        while (waiting > 0 && !may_be(sm.least[waiting - 1], sm.from[waiting - 1])) --waiting;
        if (waiting == 0) break;
        A = sm.from[waiting - 1];
        E = sm.to[waiting - 1];
        sh = cell_shift(E - A, LOG);
        for (int c = tid; c < NB / 4; c += NT) ((uint4*)sm.cells)[c] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        if (tid == 0) sm.waiting = waiting - 1;
    }
    out.d = best.d;
    out.g = best.x + best.d;
    return true;
}

// With one slice per instance the results go straight to the caller's arrays (dmin: DEFERRED where the slice gave up).
template <int NT, int NB>
__global__ __launch_bounds__(NT, (NB == 8192 ? 3 : 4)) void zl_range_fast_kernel(
    const i64* __restrict__ ts, int P, int R, u32 slices, int lanes_log, RangePart* __restrict__ part,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ dmin, int* __restrict__ status)
{
    __shared__ __align__(16) SliceSmem<NT, NB, false> sm;
    const int tid = threadIdx.x;
    const i64 b = blockIdx.x / slices;
    const u32 k = blockIdx.x % slices;
    const i64* __restrict__ inst = ts + (size_t)b * P * R;
    for (int c = tid; c < NB / 4; c += NT) ((uint4*)sm.cells)[c] = make_uint4(0u, 0u, 0u, 0u);
    u64 own_first, own_last;                               // the ends of row `tid`
    const RowEnds ends = row_ends<NT>(inst, P, R, sm.red, own_first, own_last);
    const u64 base = (u64)ends.base;
    RangePart r;
    const bool done = ends.range >> 31
        ? zl_range_slice<NT, NB, true, false>(sm, inst, P, R, slices, k, lanes_log, ends, own_first, own_last, r)
        : zl_range_slice<NT, NB, false, false>(sm, inst, P, R, slices, k, lanes_log, ends, own_first, own_last, r);
    r.left = !done;
    if (slices > 1) {
        if (tid == 0) {
            part[blockIdx.x] = r;
            if (k == 0) range_rest(part, gridDim.x).ended[b] = 0;
        }
        return;
    }
    if (r.d == U64_MAX) r.d = r.g = 0;                     // (unsorted rows only, or nothing found out)
    if (tid == 0) {
        barrier[b] = (i64)(base + r.g);
        dmin[b] = r.left ? DEFERRED : (i64)r.d;
        if (status) status[b] = (int)r.flags;
    }
    store_iters<NT>(inst, P, R, base, r.g, own_first, own_last, iters + b * (i64)P);
}

// What the kernels above gave up, and, for instances in slices, the best of the slices and the iteration counts.  DEEP: the
// slices are searched again, too full cells gone into, a workgroup each (without slices: a fixed grid, every workgroup looks
// through its share of the instances).  The last of an instance's to end takes the best of them.  What that gives up as well,
// and small instances (not DEEP), go to the sort-based search over whole rows.
template <int NT, int ITEMS, int NB, bool DEEP>
__global__ __launch_bounds__(NT, DEEP ? 4 : 1) void zl_range_window_kernel(
    const i64* __restrict__ ts, i64 B, int P, int R, u32 slices, int lanes_log, RangePart* part,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ dmin, int* __restrict__ status)
{
    using C = WinCfg<NT, ITEMS>;
    using Slice = SliceSmem<NT, NB, true>;
    constexpr size_t BYTES = DEEP && sizeof(Slice) > C::BYTES ? sizeof(Slice) : C::BYTES;
    __shared__ __align__(16) unsigned char smem[BYTES];
    const Smem sm = carve<NT, ITEMS>(smem);
    const int tid = threadIdx.x;
    auto store = [&](i64 b, i64 base, Best best, int flags) {            // best.x: the barrier, relative to base
        if (best.d == U64_MAX) best = Best{0ull, 0ull};                  // (unsorted rows only)
        if (tid == 0) {
            barrier[b] = (i64)((u64)base + best.x);
            dmin[b] = (i64)best.d;
            if (status) status[b] = flags ? (int)EBSP_STATUS_UNSORTED : 0;
        }
        for (int p = tid; p < P; p += NT)
            iters[b * (i64)P + p] = (int)row_first_at_least(ts + ((size_t)b * P + p) * R, (u32)R, (u64)base, best.x + 1);
    };
    auto search = [&](i64 b) {
        const i64* __restrict__ inst = ts + (size_t)b * P * R;
        u64 first, last;
        const RowEnds ends = row_ends<NT>(inst, P, R, sm.red, first, last);
        Rows rw;
        rw.inst = inst; rw.le = nullptr; rw.iv = nullptr; rw.par = nullptr; rw.P = P; rw.R = R; rw.base = (u64)ends.base;
        rw.cr = nullptr; rw.narrow = false; rw.wide = false; rw.stride = 0; rw.k0 = rw.k1 = 0;
        u64 d = U64_MAX, g = 0;
        int bad = 0;
        if (ends.range > RANGE_PIECE_MAX) zl_range_window<NT, ITEMS, true>(sm, rw, ends.thr, 0ull, ends.range, d, g, bad);
        else zl_range_window<NT, ITEMS, false>(sm, rw, ends.thr, 0ull, ends.range, d, g, bad);
        store(b, ends.base, Best{d, g}, __syncthreads_or(bad));
    };
    auto go_into = [&](i64 b, u32 k, i64& base) -> RangePart {
        Slice& sl = *(Slice*)smem;
        const i64* __restrict__ inst = ts + (size_t)b * P * R;
        __syncthreads();
        for (int c = tid; c < NB / 4; c += NT) ((uint4*)sl.cells)[c] = make_uint4(0u, 0u, 0u, 0u);
        u64 own_first, own_last;
        const RowEnds ends = row_ends<NT>(inst, P, R, sl.red, own_first, own_last);
        base = ends.base;
        RangePart r;
        if (ends.range >> 31) zl_range_slice<NT, NB, true, true>(sl, inst, P, R, slices, k, lanes_log, ends, own_first, own_last, r);
        else zl_range_slice<NT, NB, false, true>(sl, inst, P, R, slices, k, lanes_log, ends, own_first, own_last, r);
        __syncthreads();
        return r;
    };
    if (DEEP && slices > 1) {
        // (the instances are shared out by the first workgroups, so that all dies of the chip have some)
        const RangeRest rest = range_rest(part, gridDim.x);
        Best best;
        int flags;
        u32 left;
        auto look_through = [&](i64 b) {
            best = Best{U64_MAX, U64_MAX};
            flags = 0;
            left = 0;
            for (u32 j = tid; j < slices; j += NT) {
                const RangePart r = part[b * slices + j];
                const Best got{r.d, r.g};
                if (!r.left && got.before(best)) best = got;
                flags |= (int)r.flags;
                left += r.left;
            }
            flags = __syncthreads_or(flags);               // (the slices have seen all neighbours in all rows)
            left = block_reduce<u32, NT>(left, (u32*)sm.red, OpAdd());
        };
        auto finish = [&](i64 b) {
            i64 base = INT64_MAX;
            for (int p = tid; p < P; p += NT) { const i64 f = ts[((size_t)b * P + p) * R]; base = f < base ? f : base; }
            base = block_reduce<i64, NT>(base, (i64*)sm.red, OpMin());
            best = block_first_min<NT>(best, sm.red);
            store(b, base, best, flags);
        };
        i64 whose = -1;                                    // the instance to finish
        if (blockIdx.x < B) {
            look_through(blockIdx.x);
            if (left == 0 || flags) whose = blockIdx.x;
        }
        if (part[blockIdx.x].left) {
            const i64 b = blockIdx.x / slices;
            if (whose >= 0) { finish(whose); whose = -1; }
            look_through(b);
            if (flags) return;                             // (finished by another workgroup)
            i64 base;
            const RangePart r = go_into(b, blockIdx.x % slices, base);
            if (tid == 0) {
                u64* const to = (u64*)(rest.part + blockIdx.x);
                __hip_atomic_store(to, r.d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(to + 1, r.g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(to + 2, (u64)r.left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sm.red[0] = __hip_atomic_fetch_add(&rest.ended[b], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            const bool last = sm.red[0] + 1 == left;
            __syncthreads();
            if (!last) return;
            __threadfence();
            int again = 0;
            for (u32 j = tid; j < slices; j += NT)
                if (part[b * slices + j].left) {
                    u64* const from = (u64*)(rest.part + b * slices + j);
                    const Best got{__hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                                   __hip_atomic_load(from + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
                    if (got.before(best)) best = got;
                    again |= __hip_atomic_load(from + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
                }
            if (__syncthreads_or(again)) { search(b); return; }
            whose = b;
        }
        if (whose >= 0) finish(whose);
        return;
    }
    const u32 total = (u32)B;
    const u32 share = (total + gridDim.x - 1) / gridDim.x;
    const u32 first = blockIdx.x * share;
    const u32 end = first + share < total ? first + share : total;
    int any = 0;                                          // mostly nothing is marked: out before anything is set up
    for (u32 idx = first + tid; idx < end; idx += NT) any |= dmin[idx] == DEFERRED;
    if (!__syncthreads_or(any)) return;
    for (u32 base0 = first; base0 < end; base0 += NT) {
        const u32 idx = base0 + tid;
        bool mine = idx < end && dmin[idx] == DEFERRED;
        for (;;) {
            const u32 b = block_reduce<u32, NT>(mine ? idx : 0xffffffffu, (u32*)sm.red, OpMin());
            if (b == 0xffffffffu) break;
            if (b == idx) mine = false;
            bool again = true;
            if constexpr (DEEP) {
                i64 base;
                const RangePart r = go_into((i64)b, 0, base);
                again = r.left != 0;
                if (!again) store((i64)b, base, Best{r.d, r.g}, (int)r.flags);
            }
            if (again) search((i64)b);
            __syncthreads();
        }
    }
}

}  // namespace
