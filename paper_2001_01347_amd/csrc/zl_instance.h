// One workgroup per instance: the whole search in LDS.
// Part of the ZipLine library (see zipline.hip); device code for gfx950.
#pragma once
#include "zl_walk.h"

namespace {

// Where an instance's rows come from, and what a search of it found.
struct Source {
    const i64* inst;    // stored rows, or
    const i64* le;      // predicted ones: le[p] + (i + 1) * iv[p],
    const i64* iv;
    i64 start;          // (RUN) start + (i + 1) * iv[p] if `common`
    bool common;
};
struct Found {
    i64 bar;
    u64 wait;
    u32 flags;
};

template <bool PRED>
__device__ __forceinline__ Source source_of(const i64* ts, const i64* le, const i64* iv, i64 b, int P, int R)
{
    Source s;
    s.inst = PRED ? nullptr : ts + b * (i64)(P * R);
    s.le = PRED ? le + b * (i64)P : nullptr;
    s.iv = PRED ? iv + b * (i64)P : nullptr;
    s.start = 0;
    s.common = false;
    return s;
}

// An instance's outputs, or the mark that leaves it to zl_instance_general_kernel.
template <int NT>
struct StoreFound {
    const Source& src;
    i64 b;
    int P, R;
    i64* __restrict__ barrier;
    int* __restrict__ iters;
    i64* __restrict__ wait;
    int* __restrict__ status;
    __device__ __forceinline__ void none() const { if (threadIdx.x == 0) wait[b] = DEFERRED; }
    __device__ __forceinline__ void operator()(const Found& f) const
    {
        if (threadIdx.x == 0) {
            barrier[b] = f.bar;
            wait[b] = (i64)f.wait;
            if (status) status[b] = (int)f.flags;
        }
        for (int p = threadIdx.x; p < P; p += NT)
            iters[b * (i64)P + p] = zl_iters_of(src.inst, src.le, src.iv, p, R, f.bar);
    }
};
// The same kept for the caller.
struct KeepFound {
    bool& found;
    Found& f;
    __device__ __forceinline__ void none() const { found = false; }
    __device__ __forceinline__ void operator()(const Found& g) const { found = true; f = g; }
};

// One workgroup per instance (P*R <= NT*ITEMS): the whole search in LDS (smem: HotCfg::BYTES of it).  out
// gets what it found, or none(): left to the general search.  On return some threads may still be reading LDS.
template <int NT, int ITEMS, bool PRED, bool RUN, class Out>        // PRED: rows are predicted; RUN: src.common may be set
__device__ __forceinline__ void zl_instance_search(unsigned char* smem, const Source& src, int P, int R, int rshift, const Out& out)
{
    using H = HotCfg<NT, ITEMS>;
    const Smem sm = carve_hot<NT, ITEMS>(smem);

    const int tid = threadIdx.x;
    const int n = P * R;
    const i64* __restrict__ inst = src.inst;
    const i64* __restrict__ lep = src.le;
    const i64* __restrict__ ivp = src.iv;
    auto at = [&](int e) -> i64 {                       // element e of the instance
        if (!PRED) return inst[e];
        const int p = rshift >= 0 ? (e >> rshift) : (e / R);
        const i64 from = RUN && src.common ? src.start : lep[p];
        return (i64)((u64)from + (u64)(e - p * R + 1) * (u64)ivp[p]);
    };

    // zl_delta.  Every element is loaded once, all loads of a thread in flight
    // together: wave w takes elements [w*64*items, (w+1)*64*items), 64 consecutive
    // ones per round, so the previous element sits in the neighbouring lane.
    // The instance minimum is not known yet, so keys are first taken relative to
    // the instance's first element t00 (mod 2^32) and shifted afterwards.
    {
        u64* bsum = sm.recs + H::BSUM_AT;
        bsum[tid] = 0; bsum[tid + NT] = 0;
    }
    const int lane = tid & (WAVE - 1), wave = tid >> 6;
    const int items = (n + NT - 1) / NT;
    const int wbase = wave * WAVE * items;
    const i64 t00 = at(0);
    i64 v[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int e = wbase + j * WAVE + lane;
        v[j] = (j < items && e < n) ? at(e) : 0;
    }
    i64 carry = (wbase > 0 && wbase < n) ? at(wbase - 1) : 0;   // element ahead of the wave's first
    i64 mn = INT64_MAX, mxf = INT64_MIN, mxl = INT64_MIN;         // min first, max first, max last of the rows
    int bad = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int e = wbase + j * WAVE + lane;
        i64 prv = __shfl_up(v[j], 1, WAVE);
        if (lane == 0) prv = carry;
        carry = __shfl(v[j], WAVE - 1, WAVE);
        if (j < items && e < n) {
            const int i = rshift >= 0 ? (e & (R - 1)) : (e % R);
            const u32 rel = (u32)((u64)v[j] - (u64)t00);
            u32 dl = rel;                                          // a row's first entry: completed below
            if (i == 0) { mn = v[j] < mn ? v[j] : mn; mxf = v[j] > mxf ? v[j] : mxf; }
            else { dl = (u32)((u64)v[j] - (u64)prv); bad |= (v[j] < prv); }
            if (i == R - 1) mxl = v[j] > mxl ? v[j] : mxl;
            sm.recs[e] = (u64)rel | ((u64)dl << 32);
        }
    }
    i64 base, first_max, last_max;
    block_bounds<NT>(mn, mxf, mxl, (i64*)sm.red, base, first_max, last_max);   // also orders the record writes
    const u64 range = (u64)last_max - (u64)base;
    const u64 thr = (u64)first_max - (u64)base;
    const u32 shift = (u32)((u64)t00 - (u64)base);                 // key relative to base = stored key + shift

    u32 flags = 0;
    if (range > (u64)INT64_MAX / (u64)P) flags |= EBSP_STATUS_OVERFLOW;

    if (range >> 32) { out.none(); return; }          // deltas need more than 32 bits
    // a row's first delta is its key relative to base
    for (int p = tid; p < P; p += NT) {
        const u64 r = sm.recs[(size_t)p * R];
        sm.recs[(size_t)p * R] = (u64)(u32)r | ((u64)((u32)(r >> 32) + shift) << 32);
    }
    if (__syncthreads_or(bad)) flags |= EBSP_STATUS_UNSORTED;
    // the records go to registers for the bucket search (which reuses the record area)
    u32 key[ITEMS], dl[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int q = j * NT + tid;
        if (q < n) {
            const u64 r = sm.recs[q];
            key[j] = (u32)r + shift;
            dl[j] = (u32)(r >> 32);
        }
    }
    // the equalising bucket map: key counts of up to 256 coarse bins -> buckets per bin
    u32* coarse = sm.cnt;                                   // free until the bucket scan
    u64* tab = (u64*)(sm.cnt + H::NB);
    const int bl = bit_length(range);
    TableMap<(ITEMS >= 8)> bucket;                          // small instances: finding the bounds costs more than it saves
    bucket.tab = tab;
    bucket.cshift = bl > 8 ? (u32)(bl - 8) : 0u;
    bucket.cmask = (1u << bucket.cshift) - 1u;
    bucket.span = (u32)range;
    constexpr int CPT = H::COARSE / NT > 1 ? H::COARSE / NT : 1;      // coarse bins per thread
    for (int c = tid; c < H::COARSE; c += NT) coarse[c] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (j * NT + tid < n) atomicAdd(&coarse[bucket.coarse(key[j])], 1u);
    __syncthreads();
    {
        u32 c[CPT], mine = 0;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            c[i] = tid * CPT + i < H::COARSE ? coarse[tid * CPT + i] : 0u;
            mine += c[i];
        }
        u32 all;
        u32 below_c = block_excl_scan<u32, NT>(mine, (u32*)sm.red, all);
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            if (tid * CPT + i < H::COARSE) {
                u64 tw, iw;
                table_entry(below_c, c[i], (u32)n, (u32)H::NB, bucket.cshift, tw, iw);
                tab[tid * CPT + i] = tw;
                tab[H::COARSE + tid * CPT + i] = iw;
            }
            below_c += c[i];
        }
    }
    __syncthreads();
    u64 best_wait;
    u32 bkey;
    if (!zl_bucket_finish<NT, ITEMS, false>(sm, key, StoredDeltas<ITEMS>{dl}, bucket, SlotsBelow<NT>{n}, 0ull, thr, (u32)P, 0ull, best_wait, bkey)) {
        out.none();                            // clustered values
        return;
    }
    out(Found{(i64)((u64)base + bkey), best_wait, flags});
}

template <int NT, int ITEMS, bool PRED>
__global__ __launch_bounds__(NT) void zl_instance_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, int P, int R, int rshift,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait,
    int* __restrict__ status)
{
    __shared__ __align__(16) unsigned char smem[HotCfg<NT, ITEMS>::BYTES];
    const i64 b = blockIdx.x;
    const Source src = source_of<PRED>(ts, le, iv, b, P, R);
    zl_instance_search<NT, ITEMS, PRED, false>(smem, src, P, R, rshift, StoreFound<NT>{src, b, P, R, barrier, iters, wait, status});
}

// The same search for the larger single-workgroup instances (1024 < P*R <= NT*ITEMS) with the
// keys held in registers from the loads to the evaluation: LDS holds only the bucket words,
// the tables and a short list of the entries that survive the bounds, so that several
// workgroups share a CU and one loads while another searches.  The instance's bounds come first,
// from the ends of its rows, and stay in scalar registers; the keys are relative to base from
// the start.  Wave w holds elements [w*64*items, (w+1)*64*items), 64 consecutive ones per item,
// so an element's predecessor sits in the neighbouring lane and its delta is never stored.
template <int NT, int ITEMS>
struct WaveItems {            // which of a thread's items exist in that layout
    u32 mask;
    __device__ __forceinline__ bool operator()(int j) const { return (mask >> j) & 1u; }
};
template <int ITEMS>
struct NeighbourDeltas {      // an entry's delta is its key minus the key in the lane before, a row's first entry's its key
    const u32 (&key)[ITEMS];
    u32 heads;                // items that are a row's first entry
    u32 ahead;                // key of the element before the wave's first
    __device__ __forceinline__ u32 operator()(int j) const
    {
        u32 pk = dpp_take<DPP_WAVE_SHR1, 0xf>(0u, key[j]);
        const u32 edge = j > 0 ? last_lane(key[j > 0 ? j - 1 : 0]) : ahead;
        if ((threadIdx.x & (WAVE - 1)) == 0) pk = edge;
        return ((heads >> j) & 1u) ? key[j] : key[j] - pk;
    }
};
template <int NT, int ITEMS>
struct RegCfg {
    using H = HotCfg<NT, ITEMS>;
    static constexpr int LIST = NT >= 1024 ? 6144 : NT * ITEMS / 2;   // records of the short list: two, three or six workgroups fit a CU
    static constexpr size_t BYTES = (size_t)LIST * 8 + (size_t)H::NB * 8 + (size_t)H::RED_WORDS * 8 + (size_t)H::NB * 4 +
                                    (size_t)H::COARSE * 16;
};
template <int NT, int ITEMS, bool PRED>
__global__ __launch_bounds__(NT, (NT == 1024 ? 8 : (NT == 128 ? 5 : 6))) void zl_instance_reg_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, int P, int R, int rshift,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait,
    int* __restrict__ status)
{
    using H = HotCfg<NT, ITEMS>;
    using C = RegCfg<NT, ITEMS>;
    static_assert(ITEMS <= 32 && ITEMS % 8 == 0, "item masks are one word; loads go in batches of 8");
    __shared__ __align__(16) unsigned char smem[C::BYTES];
    Smem sm;
    sm.recs = (u64*)smem;                                  // the short list
    sm.dhi = nullptr;
    sm.red = sm.recs + C::LIST + H::NB;                    // the bucket words sit between the list and the scratch
    sm.cnt = (u32*)(sm.red + H::RED_WORDS);                // followed by the coarse tables

    const int tid = threadIdx.x;
    const i64 b = blockIdx.x;
    const int n = P * R;
    const i64* __restrict__ inst = PRED ? nullptr : ts + b * (i64)n;
    const i64* __restrict__ lep = PRED ? le + b * (i64)P : nullptr;
    const i64* __restrict__ ivp = PRED ? iv + b * (i64)P : nullptr;
    // e / R for e < 2^16 (n <= 16384 here): exact with the rounded-up reciprocal, R >= 3 where it is used
    const u32 rinv = rshift >= 0 ? 0u : 0xffffffffu / (u32)R + 1u;
    auto row_of = [&](int e) -> int { return rshift >= 0 ? (e >> rshift) : (int)__umulhi((u32)e, rinv); };
    auto at = [&](int e) -> i64 {                          // element e of the instance
        if (!PRED) return inst[e];
        const int p = row_of(e);
        return (i64)((u64)lep[p] + (u64)(e - p * R + 1) * (u64)ivp[p]);
    };
    {
        u64* bsum = sm.red - H::NB;
        bsum[tid] = 0; bsum[tid + NT] = 0;
    }
    // the equalising bucket map needs the key counts of up to 256 coarse bins: counted while the records load
    u32* coarse = sm.cnt;                                   // free until the bucket scan
    u64* tab = (u64*)(sm.cnt + H::NB);
    constexpr int CPT = H::COARSE / NT > 1 ? H::COARSE / NT : 1;      // coarse bins per thread
    static_assert(H::NB >= H::COARSE, "the counters' area holds the coarse counts first");
#pragma unroll
    for (int i = 0; i < CPT; ++i)
        if (tid * CPT + i < H::COARSE) coarse[tid * CPT + i] = 0;
    // the instance's bounds from the ends of its rows (the exchange also orders the zeroes above)
    i64 base, first_max, last_max;
    {
        i64 mn = INT64_MAX, mxf = INT64_MIN, mxl = INT64_MIN;      // min first, max first, max last of the rows
        for (int p = tid; p < P; p += NT) {
            const i64 f = at(p * R), l = at(p * R + R - 1);
            mn = f < mn ? f : mn;
            mxf = f > mxf ? f : mxf;
            mxl = l > mxl ? l : mxl;
        }
        block_bounds<NT>(mn, mxf, mxl, (i64*)sm.red, base, first_max, last_max);
        base = (i64)uniform((u64)base);                    // the same in every thread: scalar registers
        first_max = (i64)uniform((u64)first_max);
        last_max = (i64)uniform((u64)last_max);
    }
    const u64 range = (u64)last_max - (u64)base;
    const u64 thr = (u64)first_max - (u64)base;
    u32 flags = 0;
    if (range > (u64)INT64_MAX / (u64)P) flags |= EBSP_STATUS_OVERFLOW;
    if (range >> 32) {
        // deltas need more than 32 bits: left to zl_instance_general_kernel
        if (tid == 0) wait[b] = DEFERRED;
        return;
    }
    const int bl = bit_length(range);
    TableMap<true> bucket;
    bucket.tab = tab;
    bucket.cshift = bl > 8 ? (u32)(bl - 8) : 0u;
    bucket.cmask = (1u << bucket.cshift) - 1u;
    bucket.span = (u32)range;

    const int lane = tid & (WAVE - 1), wave = tid >> 6;
    const int items = (n + NT - 1) / NT;
    const int wbase = wave * WAVE * items;
    i64 carry = (wbase > 0 && wbase < n) ? at(wbase - 1) : base;  // element ahead of the wave's first
    const u32 ahead = (u32)((u64)carry - (u64)base);               // its key
    int bad = 0;
    u32 key[ITEMS];                                        // relative to base
    u32 have = 0, heads = 0;                               // items that exist; items that are a row's first entry
    constexpr int LB = 8;                                  // loads of a thread in flight together
#pragma unroll
    for (int g = 0; g < ITEMS; g += LB) {
#pragma unroll
        for (int j = 0; j < LB; ++j) key[g + j] = 0;
        if (g < items) {
            i64 v[LB];
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                const int e = wbase + (g + j) * WAVE + lane;
                v[j] = (g + j < items && e < n) ? at(e) : 0;
            }
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                const int e = wbase + (g + j) * WAVE + lane;
                i64 prv = dpp_take<DPP_WAVE_SHR1, 0xf>((i64)0, v[j]);
                if (lane == 0) prv = carry;
                carry = (i64)last_lane((u64)v[j]);
                if (g + j < items && e < n) {
                    const bool first = e == row_of(e) * R;
                    const u32 rel = (u32)((u64)v[j] - (u64)base);   // (beyond the range only in unsorted rows: the maps clamp)
                    have |= 1u << (g + j);
                    key[g + j] = rel;
                    if (first) heads |= 1u << (g + j);
                    else bad |= (v[j] < prv);
                    atomicAdd(&coarse[bucket.coarse(rel)], 1u);
                }
            }
        }
    }
    const WaveItems<NT, ITEMS> present{have};
    if (__syncthreads_or(bad)) flags |= EBSP_STATUS_UNSORTED;       // also: the coarse counts are complete
    {
        u32 c[CPT], mine = 0;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            c[i] = tid * CPT + i < H::COARSE ? coarse[tid * CPT + i] : 0u;
            mine += c[i];
        }
        u32 all;
        u32 below_c = block_excl_scan<u32, NT>(mine, (u32*)sm.red, all);
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            if (tid * CPT + i < H::COARSE) {
                u64 tw, iw;
                table_entry(below_c, c[i], (u32)n, (u32)H::NB, bucket.cshift, tw, iw);
                tab[tid * CPT + i] = tw;
                tab[H::COARSE + tid * CPT + i] = iw;
            }
            below_c += c[i];
        }
    }
    __syncthreads();
    u64 best_wait;
    u32 bkey;
    // the deltas are not stored: an entry's delta is its key minus the key in the lane before (a row's first
    // delta is its key relative to base)
    const bool found = zl_bucket_finish<NT, ITEMS, false, TableMap<true>, C::LIST, WaveItems<NT, ITEMS>, NeighbourDeltas<ITEMS>>(
        sm, key, NeighbourDeltas<ITEMS>{key, heads, ahead}, bucket, present, 0ull, thr, (u32)P, 0ull, best_wait, bkey);
    if (!found) {
        if (tid == 0) wait[b] = DEFERRED;      // clustered values: left to zl_instance_general_kernel
        return;
    }
    const i64 bar = (i64)((u64)base + bkey);
    if (tid == 0) {
        barrier[b] = bar;
        wait[b] = (i64)best_wait;
        if (status) status[b] = (int)flags;
    }
    for (int p = tid; p < P; p += NT)
        iters[b * (i64)P + p] = zl_iters_of(inst, lep, ivp, p, R, bar);
}

// Instances whose values spread over 2^32 and more (timestamps in nanoseconds) but evenly enough: the bucket search
// of zl_bucket_finish with 64-bit values.  Buckets and bounds come from the values shifted down to 32 bits (a bucket's
// bounds in whole values are its lowest shifted key with the lost bits zero, and its highest with them set), the
// buckets' words hold exact sums of exact deltas (P * range below 2^SUM_BITS: 18 minutes of nanoseconds at P = 64),
// the list holds whole values.  Values are read again for each of the passes instead of kept in registers (not all of
// them stay in the L2: 356 MiB fetched for 115).  `smem` has BYTES; false: nothing found out (the sort does it).  1021 instances of 61 x 241
// in nanoseconds: 820 us by the radix sort in 64-bit pieces, 297 us so.  Not for instances of at most 1024 entries:
// one piece of the sort, and the kernel that has both starts 1 us later where nothing is left to it.  What it gives up
// (a bucket too deep) has paid for two passes: rows that all jump by 2^40 half way, 17 to 29 % more than by the sort alone.
template <int NT, size_t BYTES, class RW>
__device__ __forceinline__ bool zl_wide_search(unsigned char* smem, const RW& rw, int P, int R, u64 range, u64 thr,
                                               u64& best_wait, u64& best_rel)
{
    constexpr int NB = 2 * NT, NW = NT / WAVE, COARSE = 256;
    constexpr int LIST = (int)((BYTES - NB * 12 - COARSE * 16 - (4 * NW + 8) * 8) / 16);
    static_assert(LIST >= 256 && NB >= COARSE, "room for a list worth the while; the counters' area holds the coarse counts first");
    u64* const bsum = (u64*)smem;
    u64* const tab = bsum + NB;
    u64* const red = tab + 2 * COARSE;
    u64* const lval = red + 4 * NW + 8;
    u64* const ldel = lval + LIST;
    u32* const cnt = (u32*)(ldel + LIST);
    u32* const misc = (u32*)(red + 4 * NW);               // entries listed; a bucket is too deep
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const int n = P * R;
    if (range >= (1ull << SUM_BITS) / (u64)P) return false;
    const u32 sh = (u32)bit_length(range) - 32u;          // 1 or more
    TableMap<true> bucket;
    bucket.tab = tab;
    bucket.cshift = 24;
    bucket.cmask = (1u << 24) - 1u;
    bucket.span = (u32)(range >> sh);
    bsum[2 * tid] = bsum[2 * tid + 1] = 0;
    for (int c = tid; c < COARSE; c += NT) cnt[c] = 0;
    if (tid == 0) { misc[0] = 0; misc[1] = 0; }
    __syncthreads();
    // every entry: f(value relative to base, delta, out of order)
    auto each = [&](auto f) {
        constexpr int U = 4;
        int p = tid / R, i = tid - p * R;
        const int dp = NT / R, di = NT - dp * R;
        for (int e = tid; e < n; e += U * NT) {
            u64 v[U], d[U];
            bool have[U], bad[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                have[k] = e + k * NT < n;
                v[k] = d[k] = 0;
                bad[k] = false;
                if (have[k]) {
                    v[k] = rw.rel(p, (u32)i);
                    d[k] = i > 0 ? rw.rel(p, (u32)i - 1u) : 0ull;
                }
                p += dp; i += di;
                if (i >= R) { i -= R; ++p; }
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                bad[k] = v[k] < d[k] || v[k] > range;
                if (have[k]) f(v[k], v[k] - d[k], bad[k]);
            }
        }
    };
    int bad = 0;
    each([&](u64 v, u64, bool b) { bad |= b; atomicAdd(&cnt[bucket.coarse((u32)(v >> sh))], 1u); });
    if (__syncthreads_or(bad)) return false;              // not sorted: the sums would not hold; the general search says so
    {
        constexpr int CPT = COARSE / NT > 1 ? COARSE / NT : 1;
        u32 c[CPT], mine = 0;
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            c[k] = tid * CPT + k < COARSE ? cnt[tid * CPT + k] : 0u;
            mine += c[k];
        }
        u32 all;
        u32 below = block_excl_scan<u32, NT>(mine, (u32*)red, all);
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            if (tid * CPT + k < COARSE) table_entry(below, c[k], (u32)n, (u32)NB, 24u, tab[tid * CPT + k], tab[COARSE + tid * CPT + k]);
            below += c[k];
        }
    }
    __syncthreads();
    each([&](u64 v, u64 d, bool) { atomicAdd(&bsum[bucket((u32)(v >> sh))], (1ull << SUM_BITS) | d); });
    __syncthreads();
    const u64 h0 = bsum[2 * tid], h1 = bsum[2 * tid + 1];
    const u32 c0 = (u32)(h0 >> SUM_BITS), c1 = (u32)(h1 >> SUM_BITS);
    u32 q0, q1, r0, r1;
    bucket.bounds_pair(2 * tid, q0, q1, r0, r1);
    const u64 rest = (1ull << sh) - 1;
    const u64 lo0 = (u64)q0 << sh, hi0 = ((u64)q1 << sh) | rest, lo1 = (u64)r0 << sh, hi1 = ((u64)r1 << sh) | rest;
    if ((c0 > c1 ? c0 : c1) > BUCKET_LIMIT) misc[1] = 1;
    u64 all;
    const u64 before = block_excl_scan<u64, NT>((h0 + h1) & SUM_MASK, red, all);     // sums stay below 2^SUM_BITS
    if (misc[1]) return false;
    const u64 e0 = before + (h0 & SUM_MASK), e1 = e0 + (h1 & SUM_MASK);
    i64 ub = INT64_MAX;
    if (c0 && lo0 >= thr) ub = (i64)((u64)P * hi0 - e0);
    if (c1 && lo1 >= thr) { const i64 u = (i64)((u64)P * hi1 - e1); ub = u < ub ? u : ub; }
    ub = block_reduce<i64, NT>(ub, (i64*)red, OpMin());
    // (a bucket whose values are all below thr holds no candidate at all)
    const bool live0 = c0 && hi0 >= thr && (i64)((u64)P * lo0 - e0) <= ub, live1 = c1 && hi1 >= thr && (i64)((u64)P * lo1 - e1) <= ub;
    constexpr u32 DROPPED = (1u << (64 - SUM_BITS)) - 1u;     // first slot of a bucket that is not listed
    static_assert(NT * 16 < (int)DROPPED, "behind every slot: an instance has at most 16 entries per thread");
    const u32 at0 = live0 ? atomicAdd(&misc[0], c0) : DROPPED, at1 = live1 ? atomicAdd(&misc[0], c1) : DROPPED;
    cnt[2 * tid] = at0; cnt[2 * tid + 1] = at1;
    bsum[2 * tid] = before | ((u64)at0 << SUM_BITS);
    bsum[2 * tid + 1] = e0 | ((u64)at1 << SUM_BITS);
    __syncthreads();
    const u32 live = misc[0];
    // More survivors than the list holds (few workers: the bounds are weak) are listed and evaluated in rounds of whole
    // buckets: a bucket belongs to the round that its first slot falls in; it has at most BUCKET_LIMIT entries.  300
    // instances of 6 x 2000 in ns: 381 us by the sort alone, 433 with the sort after a search in vain, 153 so.  One
    // round is kept apart, its entries need no test of the round (1021 of 61 x 241: 297 us, 300 as one of several).
    u64 bw = U64_MAX, bv = U64_MAX;
    auto evaluate = [&](u64 v, u64 below_b, u32 x, u32 e) {
        u64 S = below_b;
        for (; x < e; ++x) S += lval[x] <= v ? ldel[x] : 0ull;
        const u64 w = (u64)P * v - S;
        if (w < bw || (w == bw && v < bv)) { bw = w; bv = v; }
    };
    if (live <= (u32)LIST) {
        each([&](u64 v, u64 d, bool) {
            const u32 b = bucket((u32)(v >> sh));
            if (cnt[b] < DROPPED) {
                const u32 slot = atomicAdd(&cnt[b], 1u);
                lval[slot] = v;
                ldel[slot] = d;
            }
        });
        __syncthreads();
        for (u32 q = tid; q < live; q += NT) {
            const u64 v = lval[q];
            if (v < thr) continue;
            const u32 b = bucket((u32)(v >> sh));
            evaluate(v, bsum[b] & SUM_MASK, (u32)(bsum[b] >> SUM_BITS), cnt[b]);
        }
    } else {
        constexpr u32 ROUND = (u32)LIST - BUCKET_LIMIT;
        for (u32 from = 0; from < live; from += ROUND) {
            if (from) __syncthreads();                    // the list is written again
            each([&](u64 v, u64 d, bool) {
                const u32 b = bucket((u32)(v >> sh));
                if ((u32)(bsum[b] >> SUM_BITS) - from < ROUND) {
                    const u32 slot = atomicAdd(&cnt[b], 1u) - from;
                    lval[slot] = v;
                    ldel[slot] = d;
                }
            });
            __syncthreads();
            for (u32 q = tid; q < (u32)LIST && from + q < live; q += NT) {
                const u64 v = lval[q];
                const u32 b = bucket((u32)(v >> sh)), x = (u32)(bsum[b] >> SUM_BITS), e = cnt[b];
                // a slot that holds no entry of this round lies outside the bucket of whatever it holds
                if (v >= thr && x - from < ROUND && from + q >= x && from + q < e) evaluate(v, bsum[b] & SUM_MASK, x - from, e - from);
            }
        }
    }
    wave_argmin(bw, bv);
    __syncthreads();
    if (lane == WAVE - 1) { red[wave] = bw; red[NW + wave] = bv; }
    __syncthreads();
    bw = red[0]; bv = red[NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        const u64 ow = red[w], ov = red[NW + w];
        if (ow < bw || (ow == bw && ov < bv)) { bw = ow; bv = ov; }
    }
    best_wait = bw;
    best_rel = bv;
    return bw != U64_MAX;
}

// The general search over whole rows of one instance (value spread of 2^32 or more, or values too clustered for
// the bucket search): 64-bit keys and deltas, any spread in one piece (or as few as its entries need).
template <int NT, int ITEMS, bool TRY_WIDE, class RW>     // TRY_WIDE: zl_wide_search first
__device__ __forceinline__ void zl_instance_general_search(const Smem& sm, RW& rw, int P, int R, Found& out)
{
    rw.P = P; rw.R = R;
    rw.cr = nullptr; rw.narrow = false; rw.wide = false; rw.stride = 0; rw.k0 = rw.k1 = 0;
    i64 mn = INT64_MAX, mxf = INT64_MIN, mxl = INT64_MIN;
    for (int p = threadIdx.x; p < P; p += NT) {
        const i64 f = rw.value(p, 0), l = rw.value(p, (u32)R - 1);
        mn = f < mn ? f : mn;
        mxf = f > mxf ? f : mxf;
        mxl = l > mxl ? l : mxl;
    }
    i64 base, first_max, last_max;
    block_bounds<NT>(mn, mxf, mxl, (i64*)sm.red, base, first_max, last_max);
    const u64 range = (u64)last_max - (u64)base;
    const u64 thr = (u64)first_max - (u64)base;
    u32 flags = 0;
    if (range > (u64)INT64_MAX / (u64)P) flags |= EBSP_STATUS_OVERFLOW;
    rw.base = (u64)base;
    int bad = 0;
    u64 best_wait = U64_MAX, best_rel = 0;
    if constexpr (TRY_WIDE) {
        if ((range >> 32) != 0) {
            const bool found = zl_wide_search<NT, WinCfg<NT, ITEMS>::BYTES>((unsigned char*)sm.recs, rw, P, R, range, thr, best_wait, best_rel);
            __syncthreads();                              // everyone is done with LDS before it is written again
            if (found) {
                out.bar = (i64)((u64)base + best_rel);
                out.wait = best_wait;
                out.flags = flags;
                return;
            }
            best_wait = U64_MAX;
            best_rel = 0;
        }
    }
    zl_window<NT, ITEMS, true, true>(sm, rw, thr, 0ull, range, best_wait, best_rel, bad);
    if (__syncthreads_or(bad)) flags |= EBSP_STATUS_UNSORTED;
    out.bar = (i64)((u64)base + best_rel);
    out.wait = best_wait;
    out.flags = flags;
}

// The instances that zl_instance_kernel, zl_instance_reg_kernel and zl_cells_kernel deferred (value spread of 2^32
// or more, or values too clustered): the general window search over whole rows.  A small fixed grid; every workgroup looks through its share of
// wait[] for deferred marks and handles the marked instances one after the other.
template <int NT, int ITEMS>
__global__ __launch_bounds__(NT) void zl_instance_general_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, i64 B, int P, int R,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait,
    int* __restrict__ status)
{
    using C = WinCfg<NT, ITEMS>;
    __shared__ __align__(16) unsigned char smem[C::BYTES];
    const Smem sm = carve<NT, ITEMS>(smem);
    const int tid = threadIdx.x;
    const u32 total = (u32)B;
    const u32 share = (total + gridDim.x - 1) / gridDim.x;
    const u32 first = blockIdx.x * share;
    const u32 end = first + share < total ? first + share : total;

    int any = 0;                                          // mostly nothing is marked: out before anything is set up
    for (u32 idx = first + tid; idx < end; idx += NT) any |= wait[idx] == DEFERRED;
    if (!__syncthreads_or(any)) return;
    for (u32 base0 = first; base0 < end; base0 += NT) {
        const u32 idx = base0 + tid;
        bool mine = idx < end && wait[idx] == DEFERRED;
        for (;;) {
            const u32 b = block_reduce<u32, NT>(mine ? idx : 0xffffffffu, (u32*)sm.red, OpMin());
            if (b == 0xffffffffu) break;
            if (b == idx) mine = false;
            Rows rw;
            rw.inst = ts ? ts + (i64)b * P * R : nullptr; rw.le = le ? le + (i64)b * P : nullptr; rw.iv = iv ? iv + (i64)b * P : nullptr;
            Found f;
            zl_instance_general_search<NT, ITEMS, (ITEMS >= 16)>(sm, rw, P, R, f);
            if (tid == 0) {
                barrier[b] = f.bar;
                wait[b] = (i64)f.wait;
                if (status) status[b] = (int)f.flags;
            }
            for (int p = tid; p < P; p += NT) iters[(i64)b * P + p] = zl_iters_of(rw.inst, rw.le, rw.iv, p, R, f.bar);
        }
    }
}

// Both searches in one workgroup, over S supersteps: a workgroup takes an instance through all of them, the general
// search where the fast one gives up.  S == 1 is a single search (stored or predicted rows).  Batches that fit the
// chip at once are bound by launches and by the latency of one workgroup's chain, so one launch instead of three per
// superstep (search, general search, start times) is what counts; the general search's LDS costs occupancy that such
// batches do not use.  Registers (the general search's) leave room for three workgroups of 256 per CU: held to four
// by spilling, the 256 instances of 16 x 60 took 8.1 us per superstep instead of 7.6 (13.8 in three launches).
template <int NT, int ITEMS, int GITEMS, bool PRED>
__global__ __launch_bounds__(NT) void zl_run_kernel(
    const i64* __restrict__ ts, const i64* __restrict__ le, const i64* __restrict__ iv, i64 sync_cost, int S, i64 B, int P, int R,
    int rshift, i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    using H = HotCfg<NT, ITEMS>;
    using C = WinCfg<NT, GITEMS>;
    static_assert(C::CAP_WIDE >= NT * ITEMS, "the general search takes an instance in one piece");
    __shared__ __align__(16) unsigned char smem[H::BYTES > C::BYTES ? H::BYTES : C::BYTES];
    const int tid = threadIdx.x;
    const i64 b = blockIdx.x;
    Source src = source_of<PRED>(ts, le, iv, b, P, R);
    for (int s = 0; s < S; ++s) {
        // the next superstep's intervals are asked for a superstep ahead: they come from HBM
        i64 ahead = 0;
        if (PRED && s + 1 < S && tid < P) ahead = src.iv[B * (i64)P + tid];
        Found f;
        bool found;
        zl_instance_search<NT, ITEMS, PRED, PRED>(smem, src, P, R, rshift, KeepFound{found, f});
        RunRows rw;
        rw.inst = src.inst; rw.le = src.le; rw.iv = src.iv;
        rw.common = PRED && src.common; rw.start = src.start;
        rw.R = R;
        if (!found) {
            __syncthreads();                              // the fast search may still be reading LDS
            const Smem sm = carve<NT, GITEMS>(smem);
            zl_instance_general_search<NT, GITEMS, false>(sm, rw, P, R, f);
        }
        const i64 at = (i64)s * B + b;
        if (tid == 0) {
            barrier[at] = f.bar;
            wait[at] = (i64)f.wait;
            if (status) status[at] = (int)f.flags;
        }
        for (int p = tid; p < P; p += NT) iters[at * P + p] = rw.iters(p, f.bar);
        // after the barrier and the synchronisation every worker starts together; where the search raised a status
        // bit there is no barrier and the workers keep their start times
        if (PRED) {
            if (!status || f.flags == 0) { src.common = true; src.start = (i64)((u64)f.bar + (u64)sync_cost); }
            src.iv += B * (i64)P;
        }
        asm volatile("" :: "v"(ahead));
        if (s + 1 < S) __syncthreads();                   // LDS is written again
    }
}

}  // namespace
