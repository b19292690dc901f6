// GridScan and FullGridScan: the paper's heuristic and exhaustive-ish comparators of the search.
// Part of the ZipLine library (see zipline.hip); device code for gfx950.
#pragma once
#include "zl_sweep.h"

namespace {

// Section IV, Algorithm 1 ("GridScan") and the paragraph "FullGridScan".  For a designated point e
// (an entry of a designated row) the set Z holds e and every other row's point nearest to e;
// d_Z = max(Z) - min(Z).  GridScan designates the row with the smallest first timestamp and keeps
// the smallest d_Z over its R points; FullGridScan designates every row in turn (n*R sets).  The
// paper scans a whole row for the nearest point; rows are sorted, so here it is a bisection: the
// last point below e and the first at or above it are the only candidates (the earlier one when
// both are equally near).
//   zl_gridscan_kernel         one workgroup per piece of an instance's designated points (rows of up to
//                              GRID_RMAX entries; the pieces follow (row, point) order): the rows are staged
//                              in LDS as many at a time as fit and searched there by all threads, each of
//                              which keeps max(Z) and min(Z) of a few consecutive points; first minimum over
//                              the points.
//   zl_gridscan_long_kernel    longer rows: one workgroup per (instance, designated row), searched where they are.
//   zl_gridscan_finish_kernel  first minimum over the workgroups, then Z* itself: every row's
//                              nearest point to the winning e (of equal timestamps the first),
//                              barrier = max(Z*), iters[p] = 1 + index of the point.
// Of equal d_Z the set met first in (row, point) order is kept, as a loop with a strict "<" would.

constexpr int GRID_NT = 256;
constexpr int GRID_JPT = 16;                 // designated points a thread of zl_gridscan_long_kernel handles at a time
constexpr int GRID_RMAX = 4096;              // longest row that is staged in LDS
constexpr int GRID_STAGE_PER_THREAD = 64;    // bytes of rows in LDS at a time: as many workgroups per CU as their threads allow

// How many threads of zl_gridscan_kernel share out a piece's points (a multiple of 64); the workgroup's other
// waves take the same points against other rows.  A piece has at least R points, so that there are no more
// pieces than designated rows, and `least` or more where the instance has them: the rows are staged once per piece.
inline int grid_point_threads(i64 points, int R, int least, int per_thread)
{
    i64 t = points < least ? points : (R > least ? (i64)R : least);
    t = (t + per_thread - 1) / per_thread;
    return (int)((t + WAVE - 1) / WAVE * WAVE);
}

struct GridBest {      // best designated point of one designated row
    u64 d;             // max(Z) - min(Z)
    u32 row, point;
};

// Value of the point of a sorted row (R entries, in LDS or global memory) nearest to e.
__device__ __forceinline__ i64 grid_nearest(const i64* row, u32 R, i64 e)
{
    u32 lo = 0, hi = R;                      // first index with row[i] >= e
    while (lo < hi) {
        const u32 m = lo + ((hi - lo) >> 1);
        if (row[m] < e) lo = m + 1; else hi = m;
    }
    if (lo == 0) return row[0];
    const i64 below = row[lo - 1];
    if (lo == R) return below;
    const i64 above = row[lo];
    return (u64)e - (u64)below <= (u64)above - (u64)e ? below : above;
}

// Index of that point: of equal timestamps the first.
__device__ __forceinline__ u32 grid_nearest_index(const i64* __restrict__ row, u32 R, i64 e)
{
    auto first_at_or_above = [&](i64 v) {
        u32 lo = 0, hi = R;
        while (lo < hi) {
            const u32 m = lo + ((hi - lo) >> 1);
            if (row[m] < v) lo = m + 1; else hi = m;
        }
        return lo;
    };
    const u32 up = first_at_or_above(e);
    if (up == 0) return 0;
    const u32 down = first_at_or_above(row[up - 1]);
    if (up == R) return down;
    return (u64)e - (u64)row[down] <= (u64)row[up] - (u64)e ? down : up;
}

__global__ __launch_bounds__(GRID_NT) void zl_gridscan_long_kernel(
    const i64* __restrict__ ts, int P, int R, int full, GridBest* __restrict__ best, int* __restrict__ status)
{
    __shared__ u64 red[3 * (GRID_NT / WAVE)];
    constexpr int NW = GRID_NT / WAVE;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const int designated = full ? P : 1;
    const i64 b = blockIdx.x / (u32)designated;
    const i64* __restrict__ inst = ts + b * (i64)P * R;
    int pb = (int)(blockIdx.x % (u32)designated);
    if (!full) {
        // the row with the smallest first timestamp (of several the first)
        i64 f = INT64_MAX;
        u32 who = 0xffffffffu;
        for (int p = tid; p < P; p += GRID_NT) {
            const i64 v = inst[(size_t)p * R];
            if (v < f) { f = v; who = (u32)p; }                // (p grows: the first of equal values stays)
        }
        u64 w = (u64)f ^ (1ull << 63);                          // order-preserving map to unsigned
        wave_argmin(w, who);
        if (lane == WAVE - 1) { red[wave] = w; red[NW + wave] = who; }
        __syncthreads();
        w = red[0]; who = (u32)red[NW];
        for (int k = 1; k < NW; ++k) {
            const u64 ow = red[k];
            const u32 ok = (u32)red[NW + k];
            if (ow < w || (ow == w && ok < who)) { w = ow; who = ok; }
        }
        pb = (int)who;
        __syncthreads();
    }
    const bool checker = status != nullptr && blockIdx.x % (u32)designated == 0;   // one workgroup per instance checks the rows' order
    int bad = 0;
    u64 bd = U64_MAX;
    u32 bj = 0xffffffffu;
    const i64* __restrict__ drow = inst + (size_t)pb * R;
    for (u32 j0 = 0; j0 < (u32)R; j0 += GRID_NT * GRID_JPT) {
        i64 e[GRID_JPT], mx[GRID_JPT], mn[GRID_JPT];
#pragma unroll
        for (int k = 0; k < GRID_JPT; ++k) {
            const u32 j = j0 + (u32)k * GRID_NT + tid;
            e[k] = j < (u32)R ? drow[j] : 0;
            mx[k] = mn[k] = e[k];
        }
        for (int p = 0; p < P; ++p) {
            const i64* __restrict__ row = inst + (size_t)p * R;
            if (checker && j0 == 0)
                for (int i = tid + 1; i < R; i += GRID_NT) bad |= row[i] < row[i - 1];
            if (p == pb) continue;
#pragma unroll
            for (int k = 0; k < GRID_JPT; ++k) {
                const u32 j = j0 + (u32)k * GRID_NT + tid;
                if (j < (u32)R) {
                    const i64 v = grid_nearest(row, (u32)R, e[k]);
                    mx[k] = v > mx[k] ? v : mx[k];
                    mn[k] = v < mn[k] ? v : mn[k];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < GRID_JPT; ++k) {
            const u32 j = j0 + (u32)k * GRID_NT + tid;
            if (j < (u32)R) {
                const u64 d = (u64)mx[k] - (u64)mn[k];
                if (d < bd || (d == bd && j < bj)) { bd = d; bj = j; }
            }
        }
    }
    // first minimum over the designated points: smaller d_Z, then the earlier point
    wave_argmin(bd, bj);
    __syncthreads();
    if (lane == WAVE - 1) { red[wave] = bd; red[NW + wave] = bj; }
    bad = __syncthreads_or(bad);
    if (tid == 0) {
        u64 w = red[0];
        u32 j = (u32)red[NW];
        for (int k = 1; k < NW; ++k) {
            const u64 ow = red[k];
            const u32 oj = (u32)red[NW + k];
            if (ow < w || (ow == w && oj < j)) { w = ow; j = oj; }
        }
        GridBest r;
        r.d = w;
        r.row = (u32)pb;
        r.point = j;
        best[blockIdx.x] = r;
        if (checker) status[b] = bad ? (int)EBSP_STATUS_UNSORTED : 0;
    }
}

// First index of a sorted row with row[i] >= e, galloping from `hint` (0..R): a step or two where e is near the
// last one asked for, never more than twice a bisection's.
template <class VT>
__device__ __forceinline__ u32 grid_seek(const VT* row, u32 R, VT e, u32 hint)
{
    u32 lo = 0, hi = R, step = 1;
    if (hint < R && row[hint] < e) {
        lo = hint + 1;
        while (lo + step <= R) {
            const u32 m = lo + step - 1;
            if (row[m] < e) { lo = m + 1; step *= 2; } else { hi = m; break; }
        }
    } else {
        hi = hint;
        while (step <= hi) {
            const u32 m = hi - step;
            if (row[m] < e) { lo = m + 1; break; }
            hi = m; step *= 2;
        }
    }
    while (lo < hi) {
        const u32 m = lo + ((hi - lo) >> 1);
        if (row[m] < e) lo = m + 1; else hi = m;
    }
    return lo;
}

// The points [first, first + PER) of the flattened designated rows `drow` against every row of the
// instance, values relative to base in VT.  Threads of the first slice end with the thread's best (d, point).
template <int NT, int PER, class VT>
__device__ __forceinline__ void grid_scan_points(const i64* __restrict__ inst, const i64* __restrict__ drow, u64 base, int P, int R,
                                                 u32 first, u32 points, int slice, int slices, int pthreads, int pt,
                                                 unsigned char* stage, bool check, int& bad, u64& bd, u32& bj)
{
    VT* const staged = (VT*)stage;
    const int tid = threadIdx.x;
    VT e[PER], mx[PER], mn[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const u32 j = first + (u32)k < points ? first + (u32)k : points - 1;      // (beyond the end: the last point again)
        e[k] = mx[k] = mn[k] = (VT)((u64)drow[j] - base);
    }
    const int batch = (int)(NT * GRID_STAGE_PER_THREAD / sizeof(VT)) / R;   // rows in LDS at a time: one or more (R <= 4 NT)
    for (int p0 = 0; p0 < P; p0 += batch) {
        const int rows = P - p0 < batch ? P - p0 : batch;
        const i64* __restrict__ src = inst + (size_t)p0 * R;
        __syncthreads();                                                // the rows staged before have been searched
        for (int i = tid; i < rows * R; i += NT) {
            const i64 v = src[i];
            staged[i] = (VT)((u64)v - base);
            if (check && i % R != 0) bad |= v < src[i - 1];
        }
        __syncthreads();
        if (slice < slices)
            for (int p = slice; p < rows; p += slices) {
                const VT* row = staged + p * R;
                u32 pos = 0, lo = 0, hi = (u32)R;
                while (lo < hi) {                                       // the first point: bisection
                    const u32 m = (lo + hi) >> 1;
                    if (row[m] < e[0]) lo = m + 1; else hi = m;
                }
                pos = lo;
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    if (k > 0) pos = grid_seek<VT>(row, (u32)R, e[k], pos);
                    // at a row's end both are the entry there (the designated row itself gives e)
                    const VT below = row[pos > 0 ? pos - 1 : 0], above = row[pos < (u32)R ? pos : (u32)R - 1];
                    const VT v = (VT)(e[k] - below) <= (VT)(above - e[k]) ? below : above;
                    mx[k] = v > mx[k] ? v : mx[k];
                    mn[k] = v < mn[k] ? v : mn[k];
                }
            }
    }
    if (slices > 1) {                                                   // the slices' max(Z) and min(Z) per point
        VT* const top = staged;                                         // at most 2 NT points each where there are slices
        VT* const bot = staged + pthreads * PER;
        __syncthreads();
        if (slice == 0)
            for (int k = 0; k < PER; ++k) { top[k * pthreads + pt] = mx[k]; bot[k * pthreads + pt] = mn[k]; }
        __syncthreads();
        if (slice > 0 && slice < slices)
            for (int k = 0; k < PER; ++k) { atomicMax(&top[k * pthreads + pt], mx[k]); atomicMin(&bot[k * pthreads + pt], mn[k]); }
        __syncthreads();
        if (slice == 0)
            for (int k = 0; k < PER; ++k) { mx[k] = top[k * pthreads + pt]; mn[k] = bot[k * pthreads + pt]; }
    }
    if (slice == 0)
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const u64 d = (u64)(VT)(mx[k] - mn[k]);
            if (first + (u32)k < points && d < bd) { bd = d; bj = first + (u32)k; }
        }
}

// Bound by LDS latency and the vector ALU: P searches per designated point.  Four consecutive points per thread
// (the next point's place in a row is a step or two further), values in 32 bits where the instance's spread allows
// (half the LDS, half the instructions), all threads at work whatever R is, one staging per 64 bytes of rows and thread.
// FullGridScan of 64 instances of 100 x 150: 1.04 ms with a workgroup of 256 threads per designated row, a row staged
// at a time and every search a bisection of 64-bit values, 0.30 ms so (1024 threads; the other sizes: ebsp_gridscan_batch).
template <int NT, int PER>
__global__ __launch_bounds__(NT, 8) void zl_gridscan_kernel(
    const i64* __restrict__ ts, int P, int R, int full, int pieces, int pthreads, GridBest* __restrict__ best, int* __restrict__ status)
{
    __shared__ __align__(16) unsigned char stage[NT * GRID_STAGE_PER_THREAD];
    constexpr int NW = NT / WAVE;
    __shared__ u64 red[3 * NW];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x / (u32)pieces;
    const int piece = (int)(blockIdx.x % (u32)pieces);
    const i64* __restrict__ inst = ts + b * (i64)P * R;
    i64 mn = INT64_MAX, mxf = INT64_MIN, mxl = INT64_MIN;
    u32 who = 0xffffffffu;                                      // the thread's row with the smallest first timestamp
    for (int p = tid; p < P; p += NT) {
        const i64 f = inst[(size_t)p * R], l = inst[(size_t)p * R + (R - 1)];
        if (f < mn || who == 0xffffffffu) { mn = f; who = (u32)p; }   // (p grows: the first of equal values stays)
        mxl = l > mxl ? l : mxl;
    }
    const i64 my_min = mn;
    i64 base, top;
    block_bounds<NT>(mn, mxf, mxl, (i64*)red, base, mxf, top);
    u32 pb = 0;
    if (!full) pb = block_reduce<u32, NT>(who != 0xffffffffu && my_min == base ? who : 0xffffffffu, (u32*)red, OpMin());
    const u32 points = full ? (u32)(P * R) : (u32)R;
    const i64* __restrict__ drow = inst + (size_t)pb * R;
    const int slices = NT / pthreads;
    const int slice = tid / pthreads, pt = tid - slice * pthreads;
    const u32 first = (u32)piece * (u32)(pthreads * PER) + (u32)(pt * PER);
    const bool checker = status != nullptr && piece == 0;       // one workgroup per instance checks the rows' order
    int bad = 0;
    u64 bd = U64_MAX;
    u32 bj = 0xffffffffu;
    if ((((u64)top - (u64)base) >> 32) == 0)
        grid_scan_points<NT, PER, u32>(inst, drow, (u64)base, P, R, first, points, slice, slices, pthreads, pt, stage, checker, bad, bd, bj);
    else
        grid_scan_points<NT, PER, u64>(inst, drow, (u64)base, P, R, first, points, slice, slices, pthreads, pt, stage, checker, bad, bd, bj);
    // first minimum over the designated points: smaller d_Z, then the earlier point
    wave_argmin(bd, bj);
    __syncthreads();
    if (lane == WAVE - 1) { red[wave] = bd; red[NW + wave] = bj; }
    bad = __syncthreads_or(bad);
    if (tid == 0) {
        u64 w = red[0];
        u32 j = (u32)red[NW];
        for (int k = 1; k < NW; ++k) {
            const u64 ow = red[k];
            const u32 oj = (u32)red[NW + k];
            if (ow < w || (ow == w && oj < j)) { w = ow; j = oj; }
        }
        GridBest r;
        r.d = w;
        r.row = full ? j / (u32)R : pb;
        r.point = full ? j % (u32)R : j;
        best[blockIdx.x] = r;
        if (checker) status[b] = bad ? (int)EBSP_STATUS_UNSORTED : 0;
    }
}

// FullGridScan of many rows: most points need few of them.  max(Z) - min(Z) only grows from row to row, so a point whose set has
// spread beyond the best found is out.  The rows that spread it are those with the longest iterations (a point's nearest
// entry is half an iteration away at most), and FIRST of them are searched for all points; the narrowest set of every 16
// threads is then evaluated over all rows, and so are the points whose sets are no wider than the best of those, a thread per row.
// Where that leaves more than LEFT points, or more than ROUNDS rounds of as many as the workgroup takes at once, every row is searched
// for every point as above, and so it is from the start where more than LONG rows are three quarters as long as the longest or more:
// then a few of them rule out little.
// us, all rows searched for all points / so, with configuration 2's workers | 5's | 4's, of three seeds: 64 of 100 x 150 300 / 145 to
// 155 | 203 to 214 | 188 to 211, 64 of 128 x 150 455 / 191 to 201 | 278 to 299 | 304 to 362, 64 of 200 x 100 500 / 305 to 345 | 515 to
// 534 | 623 to 631, 30 of 300 x 150 1205 / 730 to 770 | 1207 to 1211 | 1294 to 1325, 20 of 500 x 100 975 / 1109 to 1129 | 990 to 1005 |
// 1031 to 1038; with 3's 165 to 175, 216 to 227, 253 to 302, 430 to 614, 798 to 975; workers alike 1.01 to 1.04 of all rows.
// 256 points whatever the rows: 64 of 200 x 100 of 4's 792 to 836, 20 of 500 x 100 of 2's 1493 to 1727; 128: 64 of 100 x 150 of 5's 206 to
// 255, 20 of 500 x 100 of 2's 1380 to 1409; 40 rounds: 64 of 200 x 100 of 4's 673 to 691, 24 of 400 x 120 of 3's 635 to 774 instead of
// 645 to 807.  Without LONG 64 of 200 x 100 of 5's took 463 to 496, but of workers alike 644, 20 of 500 x 100 of 5's 2606.
// Beyond PMAX a round of evaluation takes one point: 10 of 1000 x 150 4017 / 4518, 64 of 1000 x 60 6471 / 8194; below PMIN there
// are too few rows to save: 64 of 50 x 240 105 / 126.  R up to RMAX: the first rows fit the stage, and longer ones are searched in
// pieces of a row or more by chips that are not full, 16 of 96 x 512 188 / 349 (256 points left).  Fewer than 128 rows in small
// batches (ebsp_gridscan_batch): 40 of 100 x 180 178 / 208 | 179 / 177, 32 of 100 x 240 189 / 228 | 188 / 203 (2's with one straggler in twenty | 5's).
constexpr int GRID_FIRST = 16, GRID_LEFT = 256, GRID_ROUNDS = 32, GRID_LONG = 52, GRID_FULL_RMAX = 256, GRID_FULL_PMIN = 96, GRID_FULL_PMAX = 512;
template <int NT, int PER, class VT>
__device__ __forceinline__ bool grid_scan_pruned(const i64* __restrict__ inst, u64 base, u64 longest, int P, int R, u32 first, u32 points, int slice,
                                                 int slices, int pthreads, int pt, unsigned char* stage, u64& bd, u32& bj)
{
    constexpr int BINS = 64;
    static_assert(NT >= 1024 && GRID_LEFT <= NT, "a thread per point of the list");
    __shared__ u32 bins[BINS], rows[GRID_FIRST], taken, left, list[GRID_LEFT];
    __shared__ u64 top[16], bot[16], ub, early, late;
    VT* const staged = (VT*)stage;
    const int tid = threadIdx.x;
    // the rows with the longest iterations, roughly
    for (int q = tid; q < BINS; q += NT) bins[q] = 0;
    if (tid == 0) { taken = 2; left = 0; ub = U64_MAX; early = U64_MAX; late = 0; rows[0] = rows[1] = 0; }
    __syncthreads();
    const float scale = (float)(BINS - 1) / ((float)longest + 1.0f);
    auto bin_of = [&](int p) -> u32 {
        const i64* row = inst + (size_t)p * R;
        const float q = (float)((u64)row[R - 1] - (u64)row[0]) * scale;
        return q < (float)(BINS - 1) ? (u32)q : (u32)BINS - 1;      // (beyond in unsorted rows only)
    };
    u64 mine_early = U64_MAX, mine_late = 0;
    for (int p = tid; p < P; p += NT) {
        atomicAdd(&bins[bin_of(p)], 1u);
        const u64 f = (u64)inst[(size_t)p * R] - base, l = (u64)inst[(size_t)p * R + R - 1] - base;
        mine_early = l < mine_early ? l : mine_early;
        mine_late = f > mine_late ? f : mine_late;
    }
    if (mine_early != U64_MAX) { atomicMin(&early, mine_early); atomicMax(&late, mine_late); }
    __syncthreads();
    // and the first to end and the last to begin, far from every point behind or ahead of them
    for (int p = tid; p < P; p += NT) {
        if ((u64)inst[(size_t)p * R + R - 1] - base == early) rows[0] = (u32)p;
        if ((u64)inst[(size_t)p * R] - base == late) rows[1] = (u32)p;
    }
    constexpr int want = GRID_FIRST;
    static_assert((size_t)GRID_FIRST * GRID_FULL_RMAX * sizeof(u64) <= (size_t)NT * GRID_STAGE_PER_THREAD, "the first rows are staged together");
    int cut = BINS - 1;                                    // its rows and those of the bins above are `want` or more
    for (u32 sum = bins[cut]; cut > 0 && sum < (u32)want;) sum += bins[--cut];
    for (int pass = 0; pass < 2; ++pass) {
        for (int p = tid; p < P; p += NT) {
            const int q = (int)bin_of(p);
            if (pass == 0 ? q > cut : q == cut) {
                const u32 at = atomicAdd(&taken, 1u);
                if (at < (u32)want) rows[at] = (u32)p;
            }
        }
        __syncthreads();
    }
    const int count = (int)taken < want ? (int)taken : want;
    for (int i = tid; i < count * R; i += NT) {
        const int r = i / R;
        staged[i] = (VT)((u64)inst[(size_t)rows[r] * R + (i - r * R)] - base);
    }
    __syncthreads();
    VT e[PER], mx[PER], mn[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const u32 j = first + (u32)k < points ? first + (u32)k : points - 1;      // (beyond the end: the last point again)
        e[k] = mx[k] = mn[k] = (VT)((u64)inst[j] - base);
    }
    if (slice < slices)
        for (int r = slice; r < count; r += slices) {
            const VT* row = staged + r * R;
            u32 pos = grid_seek<VT>(row, (u32)R, e[0], (u32)R / 2);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (k > 0) pos = grid_seek<VT>(row, (u32)R, e[k], pos);
                const VT below = row[pos > 0 ? pos - 1 : 0], above = row[pos < (u32)R ? pos : (u32)R - 1];
                const VT v = (VT)(e[k] - below) <= (VT)(above - e[k]) ? below : above;
                mx[k] = v > mx[k] ? v : mx[k];
                mn[k] = v < mn[k] ? v : mn[k];
            }
        }
    __syncthreads();
    if (slices > 1) {                                      // the slices' max(Z) and min(Z) per point
        VT* const hi = staged;
        VT* const lo = staged + pthreads * PER;
        if (slice == 0)
            for (int k = 0; k < PER; ++k) { hi[k * pthreads + pt] = mx[k]; lo[k * pthreads + pt] = mn[k]; }
        __syncthreads();
        if (slice > 0 && slice < slices)
            for (int k = 0; k < PER; ++k) { atomicMax(&hi[k * pthreads + pt], mx[k]); atomicMin(&lo[k * pthreads + pt], mn[k]); }
        __syncthreads();
        if (slice == 0)
            for (int k = 0; k < PER; ++k) { mx[k] = hi[k * pthreads + pt]; mn[k] = lo[k * pthreads + pt]; }
    }
    // the narrowest set of every 16 threads so far
    u64 d = U64_MAX;
    u32 j = 0xffffffffu;
    if (slice == 0)
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const u64 w = (u64)(VT)(mx[k] - mn[k]);
            if (first + (u32)k < points && w < d) { d = w; j = first + (u32)k; }
        }
    for (int m = 1; m < 16; m *= 2) {
        const u64 od = (u64)__shfl_xor((i64)d, m);
        const u32 oj = (u32)__shfl_xor((int)j, m);
        if (od < d || (od == d && oj < j)) { d = od; j = oj; }
    }
    if ((tid & 15) == 0 && j != 0xffffffffu) {
        const u32 at = atomicAdd(&left, 1u);
        if (at < (u32)GRID_LEFT) list[at] = j;
    }
    __syncthreads();
    // the listed points over all rows, G at a time: ub becomes the best; (bd, bj) the thread's own
    const int per = P < NT ? (P + WAVE - 1) / WAVE * WAVE : NT;
    const int G = NT / per < 16 ? NT / per : 16, g = tid / per;
    auto evaluate = [&](u32 n) {
        for (u32 q0 = 0; q0 < n; q0 += (u32)G) {
            if (tid < G) { top[tid] = 0; bot[tid] = U64_MAX; }
            __syncthreads();
            if (g < G && q0 + g < n) {
                const u32 point = list[q0 + g];
                const i64 at = inst[point];
                u64 hi = 0, lo = U64_MAX;
                for (int p = tid - g * per; p < P; p += per) {
                    const u64 v = (u64)((u32)p == point / (u32)R ? at : grid_nearest(inst + (size_t)p * R, (u32)R, at)) - base;
                    hi = v > hi ? v : hi;
                    lo = v < lo ? v : lo;
                }
                hi = wave_scan(hi, OpMax());
                lo = wave_scan(lo, OpMin());
                if ((tid & (WAVE - 1)) == WAVE - 1) { atomicMax(&top[g], hi); atomicMin(&bot[g], lo); }
            }
            __syncthreads();
            if (tid < G && q0 + tid < n) {
                const u64 w = top[tid] - bot[tid];
                const u32 point = list[q0 + tid];
                if (w < bd || (w == bd && point < bj)) { bd = w; bj = point; }
                atomicMin(&ub, w);
            }
            __syncthreads();
        }
    };
    evaluate(left);
    const u64 best = ub;
    __syncthreads();
    if (tid == 0) left = 0;
    __syncthreads();
    if (slice == 0)
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (first + (u32)k < points && (u64)(VT)(mx[k] - mn[k]) <= best) {
                const u32 at = atomicAdd(&left, 1u);
                if (at < (u32)GRID_LEFT) list[at] = first + (u32)k;
            }
    __syncthreads();
    const u32 n = left;
    if (n > (u32)GRID_LEFT || n > (u32)(GRID_ROUNDS * G)) return false;
    evaluate(n);
    return true;
}

template <int NT, int PER>
__global__ __launch_bounds__(NT, 8) void zl_fullgridscan_kernel(
    const i64* __restrict__ ts, int P, int R, int pieces, int pthreads, GridBest* __restrict__ best, int* __restrict__ status)
{
    __shared__ __align__(16) unsigned char stage[NT * GRID_STAGE_PER_THREAD];
    constexpr int NW = NT / WAVE;
    __shared__ u64 red[3 * NW];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x / (u32)pieces;
    const int piece = (int)(blockIdx.x % (u32)pieces);
    const i64* __restrict__ inst = ts + b * (i64)P * R;
    static_assert(GRID_FULL_PMAX <= NT, "a row to a thread");
    i64 mn = INT64_MAX, mxl = INT64_MIN, mine = 0, longest;
    if (tid < P) {
        mn = inst[(size_t)tid * R];
        mxl = inst[(size_t)tid * R + (R - 1)];
        mine = (i64)((u64)mxl - (u64)mn);
    }
    i64 base, top;
    block_bounds<NT>(mn, mxl, mine, (i64*)red, base, top, longest);
    const u64 long_rows = __ballot(tid < P && mine >= longest - longest / 4);
    if (lane == 0) red[wave] = (u64)__popcll(long_rows);
    __syncthreads();
    u32 longs = 0;
#pragma unroll
    for (int w = 0; w < GRID_FULL_PMAX / WAVE; ++w) longs += (u32)red[w];
    const bool few = uniform(longs) <= (u32)GRID_LONG;         // rows that may rule points out
    int bad = 0;
    if (status != nullptr && piece == 0) {                     // one workgroup per instance checks the rows' order
        const u32 all = (u32)P * (u32)R;
#pragma unroll 4
        for (u32 i = (u32)tid; i < all; i += NT) {             // (a row's first entry: against itself)
            const u32 before = i % (u32)R ? i - 1 : i;
            bad |= inst[i] < inst[before];
        }
    }
    const u32 points = (u32)(P * R);
    const int slices = NT / pthreads;
    const int slice = tid / pthreads, pt = tid - slice * pthreads;
    const u32 first = (u32)piece * (u32)(pthreads * PER) + (u32)(pt * PER);
    u64 bd = U64_MAX;
    u32 bj = 0xffffffffu;
    const bool narrow = (((u64)top - (u64)base) >> 32) == 0;
    bool found = false;
    if (few && narrow) found = grid_scan_pruned<NT, PER, u32>(inst, (u64)base, (u64)longest, P, R, first, points, slice, slices, pthreads, pt, stage, bd, bj);
    if (few && !narrow) found = grid_scan_pruned<NT, PER, u64>(inst, (u64)base, (u64)longest, P, R, first, points, slice, slices, pthreads, pt, stage, bd, bj);
    if (!found) {
        bd = U64_MAX;
        bj = 0xffffffffu;
        int seen = 0;
        if (narrow) grid_scan_points<NT, PER, u32>(inst, inst, (u64)base, P, R, first, points, slice, slices, pthreads, pt, stage, false, seen, bd, bj);
        else grid_scan_points<NT, PER, u64>(inst, inst, (u64)base, P, R, first, points, slice, slices, pthreads, pt, stage, false, seen, bd, bj);
    }
    wave_argmin(bd, bj);
    __syncthreads();
    if (lane == WAVE - 1) { red[wave] = bd; red[NW + wave] = bj; }
    bad = __syncthreads_or(bad);
    if (tid == 0) {
        u64 w = red[0];
        u32 j = (u32)red[NW];
        for (int k = 1; k < NW; ++k) {
            const u64 ow = red[k];
            const u32 oj = (u32)red[NW + k];
            if (ow < w || (ow == w && oj < j)) { w = ow; j = oj; }
        }
        best[blockIdx.x] = GridBest{w, j / (u32)R, j % (u32)R};
        if (status != nullptr && piece == 0) status[b] = bad ? (int)EBSP_STATUS_UNSORTED : 0;
    }
}

__global__ __launch_bounds__(GRID_NT) void zl_gridscan_finish_kernel(
    const i64* __restrict__ ts, int P, int R, int pieces, const GridBest* __restrict__ best,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ dz)
{
    __shared__ u64 red[3 * (GRID_NT / WAVE)];
    constexpr int NW = GRID_NT / WAVE;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x;
    const GridBest* mine = best + b * (i64)pieces;
    // first minimum over the pieces: smaller d_Z, then the earlier piece (its point is its own first minimum)
    u64 bd = U64_MAX;
    u32 bq = 0xffffffffu;
    for (int q = tid; q < pieces; q += GRID_NT) {
        const u64 d = mine[q].d;
        if (d < bd) { bd = d; bq = (u32)q; }
    }
    wave_argmin(bd, bq);
    if (lane == WAVE - 1) { red[wave] = bd; red[NW + wave] = bq; }
    __syncthreads();
    bd = red[0]; bq = (u32)red[NW];
    for (int k = 1; k < NW; ++k) {
        const u64 od = red[k];
        const u32 oq = (u32)red[NW + k];
        if (od < bd || (od == bd && oq < bq)) { bd = od; bq = oq; }
    }
    __syncthreads();
    const GridBest win = mine[bq];
    const i64* __restrict__ inst = ts + b * (i64)P * R;
    const i64 e = inst[(size_t)win.row * R + win.point];
    i64 mx = e;
    for (int p = tid; p < P; p += GRID_NT) {
        const i64* __restrict__ row = inst + (size_t)p * R;
        const u32 i = (u32)p == win.row ? win.point : grid_nearest_index(row, (u32)R, e);
        iters[b * (i64)P + p] = (int)i + 1;
        const i64 v = row[i];
        mx = v > mx ? v : mx;
    }
    const i64 top = block_reduce<i64, GRID_NT>(mx, (i64*)red, OpMax());
    if (tid == 0) { barrier[b] = top; dz[b] = (i64)win.d; }
}

}  // namespace
