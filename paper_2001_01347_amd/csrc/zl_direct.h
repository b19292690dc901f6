// The summed-wait search over predicted rows by evaluating every candidate.
// Part of the ZipLine library (see zipline.hip); device code for gfx950.
#pragma once
#include "zl_finish.h"

namespace {

// A predicted row first, first + step, ..., first + (R - 1) * step needs no search: at a barrier c >= first its latest
// entry is first + q * step with q = min((c - first) / step, R - 1), so
//     wait(c) = P * c - sum_p first_p - sum_p q_p * step_p
// comes from P divisions with no order, sums or memory between candidates.  They are done in double precision, whose
// vector rate is that of 32-bit integers here, and exactly (direct_quotient): four instructions per (candidate, worker), a
// fused multiply-add, the rounding to a whole number, the minimum with R - 1, and a fused multiply-add into the sum of
// q * step (whole numbers below 2^53).  Values that do not fit are held as 64-bit integers, their quotient estimated in
// double precision and put right by the remainder (one of 1000 x 150 45 us and 395, 1000 of 32 x 256 60 and 195).
// Bound by these instructions (54 us for 64 supersteps of 256 of 16 x 60, a quarter billion divisions: 28 us of them; 487
// us by the bucket search, a superstep after the other); for few candidates by the launches and one chain of steps.
constexpr int DIRECT_PMAX = 1024;            // workers whose constants LDS holds
struct DirectRow {
    double rcp, shift;                       // t = c * rcp + shift
};
template <int NT, int PM, bool SPLIT = false>
struct DirectSmem {
    DirectRow row[PM];
    double step[PM], first[PM];              // (of values that do not fit: the bits of whole numbers, first relative to ref)
    u64 red[2 * (NT / WAVE) + 2];
    double part[SPLIT ? NT / WAVE : 1][SPLIT ? NT : 1];
};
struct DirectFacts {
    i64 ref;             // candidates and first entries are relative to it
    double thr, sum;     // largest first entry, sum of the first entries (if they fit)
    u32 flags;
    bool fits;
};
struct DirectBest {
    u64 wait;
    i64 c;               // relative to ref
};

// The rows' constants and the instance's facts.  le == nullptr: all workers start at time 0.
template <int NT, int PM, bool SPLIT>
__device__ __forceinline__ DirectFacts direct_rows(DirectSmem<NT, PM, SPLIT>& sm, const i64* __restrict__ le, const i64* __restrict__ iv, int P, int R)
{
    DirectFacts f;
    f.ref = le ? le[0] : 0;
    // Quotients want values up to 2^DIRECT_BITS (a row ends at twice `most` at most), sums over the workers whole numbers
    // up to 2^53 (three times `most` each: a candidate and its distance to a first entry).
    const i64 sums = ((i64)1 << 51) / P, most = sums < (i64)1 << (DIRECT_BITS - 1) ? sums : (i64)1 << (DIRECT_BITS - 1), most_step = most / R;
    double thr = -1e300, sum = 0.0;
    int off = 0, back = 0;
    for (int p = threadIdx.x; p < P; p += NT) {
        // (start times may be anything: a difference that does not fit 64 bits would look small wrapped round)
        const i64 s = iv[p];
        const i64 l = le ? le[p] : f.ref, first = (i64)((u64)l - (u64)f.ref + (u64)s);
        const bool wraps = __builtin_fabs((double)l - (double)f.ref) > 0x1p61;
        back |= s < 0;
        off |= wraps || s < 0 || s > most_step || first > most || first < -most;
        const double fs = (double)s, ff = (double)first, rcp = direct_rcp(fs);
        sm.row[p] = DirectRow{rcp, direct_shift(ff, fs, rcp)};
        sm.step[p] = fs;
        sm.first[p] = ff;
        thr = ff > thr ? ff : thr;
        sum += ff;
    }
    off = __syncthreads_or(off);             // also: the constants are in place
    f.fits = off == 0;
    f.flags = 0;
    if (__builtin_expect(!f.fits, 0)) {      // spread and order in whole numbers
        back = __syncthreads_or(back);
        i64 mn = INT64_MAX, mxl = INT64_MIN, mxf = INT64_MIN;
        for (int p = threadIdx.x; p < P; p += NT) {
            const u64 l = le ? (u64)le[p] : 0ull, s = (u64)iv[p];
            const i64 a = (i64)(l + s), z = (i64)(l + (u64)R * s);
            mn = a < mn ? a : mn;
            mxf = a > mxf ? a : mxf;
            mxl = z > mxl ? z : mxl;
        }
        mn = block_reduce_any<i64, NT>(mn, sm.red, OpMin());
        mxf = block_reduce_any<i64, NT>(mxf, sm.red, OpMax());
        mxl = block_reduce_any<i64, NT>(mxl, sm.red, OpMax());
        if (R > 1 && back) f.flags |= EBSP_STATUS_UNSORTED;
        if ((u64)mxl - (u64)mn > (u64)INT64_MAX / (u64)P) f.flags |= EBSP_STATUS_OVERFLOW;
        f.ref = mn;                          // candidates relative to the smallest first entry
        for (int p = threadIdx.x; p < P; p += NT) {
            const u64 s = (u64)iv[p], a = (le ? (u64)le[p] : 0ull) + s - (u64)mn;
            sm.step[p] = __longlong_as_double((i64)s);
            sm.first[p] = __longlong_as_double((i64)a);
            sm.row[p].rcp = s ? 1.0 / (double)s : 0.0;
        }
        f.thr = 0.0;
        f.sum = 0.0;
        if (threadIdx.x == 0) sm.red[2 * (NT / WAVE)] = (u64)mxf - (u64)mn;
        __syncthreads();
        return f;
    }
    // (whole numbers below 2^53 in the order of their bit patterns, shifted into the positive)
    constexpr double UP = 4503599627370496.0;            // 2^52
    f.thr = (double)(i64)block_reduce_any<u64, NT>((u64)(thr + UP < 0.0 ? 0.0 : thr + UP), sm.red, OpMax()) - UP;
    f.sum = (double)(i64)block_reduce_any<u64, NT>((u64)(i64)sum, sm.red, OpAdd());
    return f;
}

template <int NT>
__device__ __forceinline__ DirectBest direct_first_min(u64 w, i64 c, u64* red)
{
    constexpr u64 SIGN = 1ull << 63;                      // signed order as unsigned
    const Best b = block_first_min<NT>(Best{w, (u64)c ^ SIGN}, red);
    return DirectBest{b.d, (i64)(b.x ^ SIGN)};
}

// The first minimum over candidates [e0, e1) (entry i of row p is candidate p * R + i), K of a thread at a time.  SPLIT: the
// waves share out the workers instead of the candidates (many workers, few candidates: a wave's walk over all of them would
// be the whole time), and add their sums up.
template <int NT, int PM, int K, bool SPLIT>
__device__ __forceinline__ DirectBest direct_search(DirectSmem<NT, PM, SPLIT>& sm, const DirectFacts& f, const i64* __restrict__ le,
                                                    const i64* __restrict__ iv, int P, int R, int e0, int e1)
{
    constexpr int NW = NT / WAVE, STRIDE = SPLIT ? WAVE : NT;
    static_assert(!SPLIT || NT == WAVE * K, "a thread adds up one candidate's sums");
    const int tid = threadIdx.x, at = SPLIT ? tid & (WAVE - 1) : tid, wave = tid >> 6;
    if (__builtin_expect(f.fits, 1)) {
        const double top = (double)(R - 1), dP = (double)P, none = __builtin_inf();
        const int p0 = SPLIT ? wave * P / NW : 0, p1 = SPLIT ? (wave + 1) * P / NW : P;
        double dw = none, dc = none;
        int row = (e0 + at) / R, i = e0 + at - row * R;    // of the thread's next candidate
        const int drow = STRIDE / R, di = STRIDE - drow * R;
        for (int base = e0; base < e1; base += STRIDE * K) {
            double c[K], sum[K];                           // (c: none where there is no candidate)
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const int p = row < P ? row : 0;
                const double v = __builtin_fma((double)i, sm.step[p], sm.first[p]);
                c[j] = base + j * STRIDE + at < e1 && v >= f.thr ? v : none;
                sum[j] = 0.0;
                row += drow;
                i += di;
                if (i >= R) { i -= R; ++row; }
            }
#pragma unroll 4
            for (int p = p0; p < p1; ++p) {
                const DirectRow r = sm.row[p];
                const double s = sm.step[p];
#pragma unroll
                for (int j = 0; j < K; ++j) sum[j] = __builtin_fma(direct_quotient(c[j], r.rcp, r.shift, top), s, sum[j]);
            }
            double w = none;
            if constexpr (SPLIT) {
                if (base > e0) __syncthreads();            // the sums before are added up
#pragma unroll
                for (int j = 0; j < K; ++j) sm.part[wave][j * WAVE + at] = sum[j];
                __syncthreads();
                double all = 0.0, mine = c[0];
#pragma unroll
                for (int k = 0; k < NW; ++k) all += sm.part[k][tid];
#pragma unroll
                for (int j = 1; j < K; ++j) mine = j == wave ? c[j] : mine;
                w = __builtin_fma(dP, mine, -all);
                if (w < dw || (w == dw && mine < dc)) { dw = w; dc = mine; }
            } else {
                // the smallest wait first, then which candidates have it
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    sum[j] = __builtin_fma(dP, c[j], -sum[j]);
                    w = __builtin_fmin(w, sum[j]);
                }
                if (w <= dw) {
                    if (w < dw) { dw = w; dc = none; }
#pragma unroll
                    for (int j = 0; j < K; ++j)
                        if (sum[j] == w) dc = __builtin_fmin(dc, c[j]);
                }
            }
        }
        const bool any = dw < none;
        return direct_first_min<NT>(any ? (u64)(i64)(dw - f.sum) : U64_MAX, any ? (i64)dc : INT64_MAX, sm.red);
    }
    if (f.flags) return DirectBest{0ull, 0};               // (no results then)
    u64 bw = U64_MAX;
    i64 bc = INT64_MAX;
    const u64 thr = sm.red[2 * NW];
    auto first = [&](int p) -> u64 { return (u64)__double_as_longlong(sm.first[p]); };
    auto step = [&](int p) -> u64 { return (u64)__double_as_longlong(sm.step[p]); };
    constexpr int KF = SPLIT ? 1 : K;                      // (a split search has NT candidates a workgroup)
    for (int base = e0 + tid; base < e1; base += NT * KF) {
        u64 c[KF], w[KF];
#pragma unroll
        for (int j = 0; j < KF; ++j) {
            const int e = base + j * NT < e1 ? base + j * NT : e1 - 1, row = e / R;
            c[j] = first(row) + (u64)(e - row * R) * step(row);
            w[j] = 0;
        }
        for (int p = 0; p < P; ++p) {
            const u64 a = first(p), s = step(p);
            const double rcp = sm.row[p].rcp;
#pragma unroll
            for (int j = 0; j < KF; ++j) w[j] += direct_remainder(c[j] - a, s, rcp, (u32)(R - 1));
        }
#pragma unroll
        for (int j = 0; j < KF; ++j)
            if (c[j] >= thr && (w[j] < bw || (w[j] == bw && (i64)c[j] < bc))) { bw = w[j]; bc = (i64)c[j]; }
    }
    return direct_first_min<NT>(bw, bc, sm.red);
}

// Entries of every row up to the barrier c.
template <int NT, int PM, bool SPLIT>
__device__ __forceinline__ void direct_iters(const DirectSmem<NT, PM, SPLIT>& sm, const DirectFacts& f, const i64* __restrict__ le,
                                             const i64* __restrict__ iv, int P, int R, i64 c, int* __restrict__ iters)
{
    for (int p = threadIdx.x; p < P; p += NT) {
        if (f.fits) {
            const double q = direct_quotient((double)c, sm.row[p].rcp, sm.row[p].shift, (double)(R - 1));
            iters[p] = sm.step[p] == 0.0 ? R : (int)q + 1;
        } else
            iters[p] = zl_iters_pred(le ? le[p] : 0, iv[p], R, (i64)((u64)f.ref + (u64)c));
    }
}

// Searches `at0` .. of one kind, G workgroups each.  Single searches: `at` is the instance.  Runs of supersteps: at =
// superstep * B + instance.  From the second superstep on all workers start at the barrier before, and relative to that
// time a superstep's rows (i + 1) * interval depend on nothing before it, so all of them are searched side by side;
// barrier[at] is then the time since the superstep's start until zl_direct_starts_kernel adds that.  (Superstep 0 has
// start times of its own, and its barrier is final.)
// G > 1: every workgroup leaves its best in the search's iters (16 bytes; G <= P / 4) for zl_direct_finish_kernel.
template <int NT, int PM, int K, bool SPLIT>
__global__ __launch_bounds__(NT, (PM > 64 ? 1 : 4)) void zl_direct_kernel(
    const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, i64 at0, int P, int R, int G, int per,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    __shared__ DirectSmem<NT, PM, SPLIT> sm;
    const i64 at = at0 + (i64)(blockIdx.x / (u32)G);
    const int g = (int)(blockIdx.x % (u32)G);
    le = at < B ? le + at * (i64)P : nullptr;
    iv += at * (i64)P;
    iters += at * (i64)P;
    const DirectFacts f = direct_rows(sm, le, iv, P, R);
    const int n = P * R, e0 = g * per, e1 = n - e0 < per ? n : e0 + per;
    const DirectBest best = direct_search<NT, PM, K, SPLIT>(sm, f, le, iv, P, R, e0, e1);
    if (G > 1) {
        if (threadIdx.x < 4) {
            const u64 word = threadIdx.x < 2 ? best.wait : (u64)best.c;
            iters[4 * g + threadIdx.x] = (int)(u32)(word >> (threadIdx.x & 1 ? 32 : 0));
        }
        return;
    }
    if (threadIdx.x == 0) {
        barrier[at] = (i64)((u64)f.ref + (u64)best.c);
        wait[at] = (i64)best.wait;
        if (status) status[at] = (int)f.flags;
    }
    direct_iters(sm, f, le, iv, P, R, best.c, iters);
}

template <int NT, int PM>
__global__ __launch_bounds__(NT) void zl_direct_finish_kernel(
    const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, i64 at0, int P, int R, int G,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    __shared__ DirectSmem<NT, PM> sm;
    const i64 at = at0 + (i64)blockIdx.x;
    le = at < B ? le + at * (i64)P : nullptr;
    iv += at * (i64)P;
    iters += at * (i64)P;
    u64 w = U64_MAX;
    i64 c = INT64_MAX;
    for (int g = threadIdx.x; g < G; g += NT) {
        const u32* from = (const u32*)iters + 4 * g;
        const u64 ow = (u64)from[0] | ((u64)from[1] << 32);
        const i64 oc = (i64)((u64)from[2] | ((u64)from[3] << 32));
        if (ow < w || (ow == w && oc < c)) { w = ow; c = oc; }
    }
    const DirectFacts f = direct_rows(sm, le, iv, P, R);
    const DirectBest best = direct_first_min<NT>(w, c, sm.red);
    __syncthreads();                                      // the results are read: iters may be written
    if (threadIdx.x == 0) {
        barrier[at] = (i64)((u64)f.ref + (u64)best.c);
        wait[at] = (i64)best.wait;
        if (status) status[at] = (int)f.flags;
    }
    direct_iters(sm, f, le, iv, P, R, best.c, iters);
}

// The supersteps' start times: a running sum of the times to the barrier and the synchronisation, a wave per instance.  A
// superstep whose search raised a status bit has no barrier: the next one starts where it did.  If that is so from
// superstep 0 on, the workers keep start times of their own, and those supersteps are searched again here.
// Those are few, or flagged like the first (and then not searched), but may be large: NT threads.
template <int NT, int PM, int K>
__global__ __launch_bounds__(NT) void zl_direct_starts_kernel(
    const i64* __restrict__ le, const i64* __restrict__ iv, i64 sync_cost, int S, i64 B, int P, int R,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    __shared__ DirectSmem<NT, PM> sm;
    const i64 b = blockIdx.x;
    const int lane = threadIdx.x;
    int s = 1;
    bool flagged = status && status[b] != 0;
    u64 start = (u64)barrier[b] + (u64)sync_cost;         // of superstep s
    for (; flagged && s < S; ++s) {
        const i64 at = (i64)s * B + b;
        const i64* from = le + b * (i64)P;
        const i64* step = iv + at * (i64)P;
        __syncthreads();
        const DirectFacts f = direct_rows(sm, from, step, P, R);
        const DirectBest best = direct_search<NT, PM, K, false>(sm, f, from, step, P, R, 0, P * R);
        const i64 bar = (i64)((u64)f.ref + (u64)best.c);
        if (lane == 0) {
            barrier[at] = bar;
            wait[at] = (i64)best.wait;
            status[at] = (int)f.flags;
        }
        direct_iters(sm, f, from, step, P, R, best.c, iters + at * (i64)P);
        flagged = f.flags != 0;
        start = (u64)bar + (u64)sync_cost;
    }
    if (lane >= WAVE) return;
    for (; s < S; s += WAVE) {
        const int mine = s + lane;
        const i64 at = (i64)mine * B + b;
        u64 len = 0, add = 0;
        if (mine < S) {
            len = (u64)barrier[at];
            add = status && status[at] != 0 ? 0ull : len + (u64)sync_cost;
        }
        const u64 sum = wave_incl_scan(add);
        if (mine < S) barrier[at] = (i64)(start + (sum - add) + len);
        start += last_lane(sum);
    }
}

}  // namespace
