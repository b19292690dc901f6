// One workgroup per stored instance of few rows: the summed-wait search over value cells.
// Part of the ZipLine library (see zipline.hip); device code for gfx950.
#pragma once
#include "zl_direct.h"

namespace {

// The entries are loaded once and stay in registers as 31-bit keys relative to the instance's smallest entry (wave w holds
// elements [w * 64 * items, (w + 1) * 64 * items), 64 neighbouring ones per item, so an element's predecessor sits in the
// neighbouring lane and its delta is never stored).  With W(c) = P * c - S(c), S(c) the sum of the deltas of all entries up
// to c:
//   1. C, the last value that can win.  lb(c) = sum_p max(0, c - last entry of row p) only grows; where lb(C) has reached some
//      wait that a candidate has, nothing behind C can win.  That wait is guessed: lb(thr), and what P rows at random wait is less
//      than half the sum of their mean iteration times; two and a half times that is allowed for (the mean of each row's quickest
//      quarter, so that a pause in a row does not count).  The guess is checked at the end.  Up to C all rows run on and
//      their entries lie evenly, so
//   2. cells of 2^sh values need no equalising table: one LDS atomic per entry up to C adds its delta to its cell's word,
//      and a scan makes S at the end of every cell of them.
//   3. Every entry reads its cell's word, D (the wait at the cell's first value if all its deltas were in, counted from
//      the smallest such) and the sum of its deltas: lb(x) = D + P * (x - first value) is short of W(x) by the deltas of
//      the cell's entries behind x, and lb(x) + sum - delta(x) is at least W(x).  The smallest upper bound is the answer unless
//      an entry has a smaller lower bound; the cells of such entries (a dozen entries in all: a cell holds two or three)
//      are listed and evaluated.  Where a cell is one value, lb is the wait.
// Values that spread over 2^31 and more are shifted down (ms bits) for all this, which makes the bounds wider by P units either
// way; the entries that remain are evaluated from the rows in 64 bits.
// What this gives up (too many entries to list: clustered values; sums beyond 32 bits; values behind C that may win) is left to
// zl_instance_general_kernel.
// Bound by the load of the entries where the batch is large (2 GiB: 2.2 TB/s; vector ALU busy 68 %: the passes over the keys are as long as the load),
// else by the workgroup's chain of steps.  The bucket search of zl_instance_reg_kernel counts the entries of coarse bins
// first, which is one more LDS atomic per entry, a table and 14 more instructions per entry to look a bucket up, and leaves
// spreads of 2^32 and more to the general search.  us, that one / this: 16384 of 64 x 256 1175 / 983, 8192 of 64 x 60
// 181 / 159, 1 of 64 x 60 25 / 16; 1021 of 61 x 241 in nanoseconds 277 / 98.  Tried and not kept: the first loads and C
// ahead of everything (in the shadow of the loads, but 80 registers spilled: 1270); 8 or 32 loads in flight instead of 16
// (1024 and 1006; in nanoseconds 102 and 99 against 98); all entries of a cell with D below the
// best bound listed without looking at them one by one (50 instead of 13: 1310); 1024 threads for large batches (1290).
template <int NT, int ITEMS, int NB>
struct CellSmem {
    static constexpr int LIST = 224;                      // (four workgroups of 256 threads per CU)
    static constexpr int CPT = NB / NT, CPT_LOG = __builtin_ctz((unsigned)(NB / NT));
    // Cell c is word c + c / CPT: the threads walk their CPT cells an odd number of words apart, without bank conflicts.
    __device__ static __forceinline__ u32 word_of(u32 c) { return c + (c >> CPT_LOG); }
    u64 cells[NB + NT + 2];                               // and a dead one
    u32 key[LIST], delta[LIST];                           // listed entries; of shifted values: key is the index,
    u64 acc[LIST];                                        // the wait evaluated from the rows
    u16 cell[LIST];
    u64 red[2 * (NT / WAVE) + 2];
    i64 first[WAVE], last[WAVE];                          // ends of the rows
    i64 bounds[5];
    u32 flag[NB / 32 + 1];                                // cells whose entries are listed
    u32 listed;
};

constexpr u64 DEAD = 0x80000000ull | 0x3fffffffull << 32;     // the word of a cell that cannot hold the minimum: D beyond every bound

// The rows of an instance.
struct InstRows {
    const i64* inst;
    int R, rshift;
    u32 rinv;           // e / R for e < 2^16: exact with the rounded-up reciprocal, R >= 3 where it is used
    __device__ __forceinline__ InstRows(const i64* inst_, int R_, int rshift_)
        : inst(inst_), R(R_), rshift(rshift_), rinv(rshift_ >= 0 ? 0u : 0xffffffffu / (u32)R_ + 1u) {}
    __device__ __forceinline__ int row_of(int e) const { return rshift >= 0 ? (e >> rshift) : (int)__umulhi((u32)e, rinv); }
    __device__ __forceinline__ i64 value(int p, int i) const { return inst[p * R + i]; }
    __device__ __forceinline__ i64 at(int e) const { return inst[e]; }
    // entries of row p up to v (relative to base)
    template <class S>
    __device__ __forceinline__ u32 upto(const S& sm, int p, u64 base, u64 v) const
    {
        return RowProbe(inst + p * R, (u32)R, base, (u64)sm.first[p] - base, (u64)sm.last[p] - base, v + 1).index();
    }
};

template <int NT, int ITEMS, int NB>
__global__ __launch_bounds__(NT, 4) void zl_cells_kernel(
    const i64* __restrict__ ts, int P, int R, int rshift,
    i64* __restrict__ barrier, int* __restrict__ iters, i64* __restrict__ wait, int* __restrict__ status)
{
    using S = CellSmem<NT, ITEMS, NB>;
    constexpr int LOG = __builtin_ctz((unsigned)NB), CPT = S::CPT, LB = ITEMS < 8 ? ITEMS : ITEMS > 16 ? 16 : 8;
    static_assert(ITEMS <= 32 && ITEMS % LB == 0, "item masks are one word; loads go in batches");
    static_assert(NB % NT == 0 && (CPT & (CPT - 1)) == 0 && NB <= 65536, "cells are numbered in 16 bits");
    __shared__ __align__(16) S sm;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const i64 b = blockIdx.x;
    const int n = P * R;
    const InstRows rows(ts + b * (i64)n, R, rshift);
    auto barrier_all = [] { __syncthreads(); };

    // the instance's bounds from the ends of its rows: wave 0's lanes
    i64 base;
    u64 thr, range, min_last, spans;
    {
        if (wave == 0) {
            const int p = lane < P ? lane : 0;             // (row 0 in lanes without one)
            const i64 f = rows.value(p, 0), l = rows.value(p, R - 1);
            // the mean iteration time, of the quickest quarter of the row (one long pause is not what the search is about)
            i64 least = l - f;
            if (R >= 16) {
                const i64 a = rows.value(p, R / 4), m = rows.value(p, R / 4 * 2), z = rows.value(p, R / 4 * 3), e = rows.value(p, R / 4 * 4 - 1);
                const i64 s0 = a - f < m - a ? a - f : m - a, s1 = z - m < e - z ? z - m : e - z;
                least = s0 < s1 ? s0 : s1;
            }
            sm.first[lane] = f;
            sm.last[lane] = l;
            const i64 mn = last_lane(wave_scan(f, OpMin())), mxf = last_lane(wave_scan(f, OpMax()));
            const i64 mxl = last_lane(wave_scan(l, OpMax())), mnl = last_lane(wave_scan(l, OpMin()));
            const i64 sp = last_lane(wave_scan(lane < P && R > 1 ? least : (i64)0, OpAdd()));
            if (lane == 0) { sm.bounds[0] = mn; sm.bounds[1] = mxf; sm.bounds[2] = mxl; sm.bounds[3] = mnl; sm.bounds[4] = sp; }
        }
        barrier_all();
        const i64 mn = sm.bounds[0], mxf = sm.bounds[1], mxl = sm.bounds[2], mnl = sm.bounds[3], sp = sm.bounds[4];
        base = (i64)uniform((u64)mn);
        thr = uniform((u64)mxf - (u64)mn);
        range = uniform((u64)mxl - (u64)mn);
        min_last = mnl < mn ? 0ull : uniform((u64)mnl - (u64)mn);      // (below in unsorted rows only)
        spans = uniform((u64)sp);
    }
    u32 flags = 0;
    if (range > (u64)INT64_MAX / (u64)P) flags |= EBSP_STATUS_OVERFLOW;

    // The entries: 31 bits of key (P * a cell's width is to stay below 2^30), a row's first entry marked; all ones: none.
    const int items = (n + NT - 1) / NT;
    const int wbase = wave * WAVE * items;
    const i64 ahead = (wbase > 0 && wbase < n) ? rows.at(wbase - 1) : base;      // the element before the wave's first
    constexpr u32 HEAD = 0x80000000u, KEY = 0x7fffffffu;
    u32 ms;
    {
        const int bl = bit_length(range), bp = bl + bit_length((u64)P) - LOG - 30;
        const int m = bl - 31 > bp ? bl - 31 : bp;
        ms = m > 0 ? (u32)m : 0u;
    }
    u32 key[ITEMS];
    int bad = 0;
    {
        i64 carry = ahead;
        u32 over = 0;
        int i = wbase + lane - rows.row_of(wbase + lane) * R;                    // index in the row
        const int step = WAVE % R;
#pragma unroll
        for (int g = 0; g < ITEMS; g += LB) {
            i64 v[LB];
            if constexpr (ITEMS > 16) __builtin_amdgcn_sched_barrier(0);      // (the next loads would spill keys)
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                const int e = wbase + (g + j) * WAVE + lane;
                v[j] = rows.at((g + j < items && e < n) ? e : n - 1);            // (the last element stands in for none)
            }
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                const int e = wbase + (g + j) * WAVE + lane;
                const i64 prv = dpp_take<DPP_WAVE_SHR1, 0xf>(carry, v[j]);       // lane 0: the item before's last
                carry = last_lane(v[j]);
                const bool is = g + j < items && e < n;
                const u64 rel = ((u64)v[j] - (u64)base) >> ms;
                over |= (u32)(rel >> 32) | ((u32)rel & HEAD);                    // beyond the range only in unsorted rows
                bad |= is && i != 0 && v[j] < prv;
                key[g + j] = is ? (u32)rel | (i == 0 ? HEAD : 0u) : ~0u;
                i += step;
                i = i >= R ? i - R : i;
            }
        }
        bad |= over != 0;
    }
    const u32 first_prev = (u32)(((u64)ahead - (u64)base) >> ms);

    Best best{U64_MAX, U64_MAX};                           // relative to base
    bool slow = false;
    if (__syncthreads_or(bad)) {
        flags |= EBSP_STATUS_UNSORTED;                     // (nothing below may rely on such rows)
    } else {
        // Nothing that one pass over the items computed is worth a register until the next.
        auto forget = [&] {
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) asm volatile("" : "+v"(key[j]));
        };
        auto delta_of = [&](int j) -> u32 {                // (all lanes together)
            const u32 p = dpp_take<DPP_WAVE_SHR1, 0xf>(j > 0 ? last_lane(key[j > 0 ? j - 1 : 0]) : first_prev, key[j]) & KEY;
            return (key[j] & KEY) - ((key[j] & HEAD) ? 0u : p);
        };
        u64 C = range, lbC = 0;
        do {                                               // (left where the slow search has to finish)
            // C (step 1): wave 0, by Newton's steps from above
            if (R > 1) {
                if (wave == 0) {
                    // in single precision, then what it found as it is in whole numbers
                    const u64 own = (u64)sm.last[lane] - (u64)base;
                    const float at = (float)(own - min_last);
                    auto lb_of = [&](u64 c) -> u64 { return last_lane(wave_scan(lane < P && own < c ? c - own : 0ull, OpAdd())); };
                    const float share = 1.25f * (float)spans / (float)(R >= 16 ? R / 4 : R - 1), G = share + (float)lb_of(thr);
                    float c = G;                                          // from min_last on: lb there is at least G
                    for (int it = 0; it < 12; ++it) {
                        const bool ended = lane < P && at < c;
                        const float lb = last_lane(wave_scan(ended ? c - at : 0.0f, OpAdd()));
                        const int rows_ended = __popcll(__ballot(ended));
                        const float over = lb - G;
                        if (!(over > 0.001f * G) || rows_ended == 0) break;
                        c -= over / (float)rows_ended;
                    }
                    u64 to = c < 9.0e18f && range - min_last > (u64)c ? min_last + (u64)c + 1 : range;
                    to = to > thr ? to : thr;
                    const u64 lb = lb_of(to);
                    if (lane == 0) { sm.red[0] = to; sm.red[1] = lb; }
                }
                barrier_all();
                C = uniform(sm.red[0]);
                lbC = uniform(sm.red[1]);
            }
            // cells (step 2): up to the one that C is in
            const u32 Ck = (u32)(C >> ms), thrk = (u32)(thr >> ms);
            const u32 sh = bit_length((u64)Ck) > LOG ? (u32)(bit_length((u64)Ck) - LOG) : 0u;
            const u32 mask = (1u << sh) - 1u, end = Ck >> sh;
            barrier_all();                                 // red is read
#pragma unroll
            for (int k = 0; k <= CPT; ++k) sm.cells[k * NT + tid] = 0;
            for (int k = tid; k <= NB / 32; k += NT) sm.flag[k] = 0;
            if (tid == 0) { sm.listed = 0; sm.cells[S::word_of(NB)] = DEAD; }
            barrier_all();
            u32 used = 0;                                  // items with entries up to C
            forget();
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const u32 d = delta_of(j), c = (key[j] & KEY) >> sh;
                if (c <= end) atomicAdd(&sm.cells[S::word_of(c)], (u64)d);
                if (__ballot(c <= end)) used |= 1u << j;
            }
            used = uniform(used);
            barrier_all();
            // S at the end of every cell; D and the cell's sum in its word
            i64 least_w;                                   // the smallest wait at a cell's first value with its deltas in
            u32 top;                                       // the smallest upper bound, counted from that
            int big = 0;
            {
                u64* const own = sm.cells + tid * (CPT + 1);
                u64 part = 0;
#pragma unroll
                for (int k = 0; k < CPT; ++k) part += own[k];
                u64 all;
                const u64 before = block_excl_scan<u64, NT>(part, sm.red, all);
                const u64 PL = (u64)P << sh;
                const u32 c_thr = thrk >> sh;              // cells before it hold no candidate
                u64 low = PL * (u32)(tid * CPT) - before;  // the wait at the next cell's first value, deltas before it in
                const u64 low0 = low;
                i64 least = INT64_MAX;
#pragma unroll
                for (int k = 0; k < CPT; ++k) {
                    const u32 c = (u32)(tid * CPT + k);
                    low -= own[k];
                    if (c >= c_thr && c <= end) least = (i64)low < least ? (i64)low : least;
                    low += PL;
                }
                least_w = block_reduce_any<i64, NT>(least, sm.red, OpMin());
                top = (u32)(PL - (u64)P);                  // (the wait at that cell's last value)
                low = low0 - (u64)least_w;
#pragma unroll
                for (int k = 0; k < CPT; ++k) {
                    const u32 c = (u32)(tid * CPT + k);
                    const u64 sum = own[k];
                    low -= sum;
                    const bool dead = c < c_thr || c > end || low > 0x40000000ull;
                    big |= !dead && sum > 0x3fffffffull;
                    // (in thr's cell an entry may be no candidate: its bound from above is not to count)
                    own[k] = dead ? DEAD : low | (c == c_thr ? 0x3fffffffull << 32 : sum << 32);
                    low += PL;
                }
            }
            if (__syncthreads_or(big || flags)) { slow = true; break; }      // (sums beyond 63 bits: left too)
            // entries (step 3); those behind C find a dead cell
            auto cell_of = [&](int j) -> u32 { const u32 c = (key[j] & KEY) >> sh; return c <= end ? c : end + 1u; };
            forget();
            u32 low = ~0u;
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                if (!((used >> j) & 1u)) continue;
                const u32 d = delta_of(j);
                const u64 w = sm.cells[S::word_of(cell_of(j))];
                const u32 lb = (u32)w + __umul24((u32)P, key[j] & mask), sum = (u32)(w >> 32);
                const u32 ub = lb + (sum > d ? sum - d : 0u);             // (sum < d in dead cells only)
                top = ub < top ? ub : top;
                low = lb < low ? lb : low;
            }
            low = last_lane(wave_scan(low, OpMin()));
            top = block_reduce_any<u32, NT>(top, sm.red, OpMin());
            if (sh == 0 && ms == 0) {                      // a cell is its only value, lb the wait
                u64 w = U64_MAX;
                forget();
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) {
                    const u64 one = (sm.cells[S::word_of(cell_of(j))] << 32) | (key[j] & KEY);
                    w = one < w ? one : w;
                }
                w = block_reduce_any<u64, NT>(w, sm.red, OpMin());
                best = Best{(u64)((i64)(w >> 32) + least_w), w & 0xffffffffull};
                slow = C != range && best.d > lbC;
                break;
            }
            // shifted values: a wait is known to P units either way
            const u32 limit = ms ? top + 2u * (u32)P : top;
            if (low <= limit) {
                forget();
                u32 first_index = (u32)(wbase + lane);
                asm volatile("" : "+v"(first_index));        // (or the loads' indices are kept till here, spilled)
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) {
                    if (!((used >> j) & 1u)) continue;
                    const u32 c = cell_of(j), lb = (u32)sm.cells[S::word_of(c)] + __umul24((u32)P, key[j] & mask);
                    if (lb <= limit) {
                        if (ms) {
                            const u32 at = atomicAdd(&sm.listed, 1u);
                            if (at < (u32)S::LIST) { sm.key[at] = first_index + (u32)(j * WAVE); sm.acc[at] = 0; }
                        } else
                            atomicOr(&sm.flag[c >> 5], 1u << (c & 31u));
                    }
                }
            }
            barrier_all();
            Best got{U64_MAX, U64_MAX};
            if (!ms) {
                // the flagged cells' entries, in rounds of neighbouring cells where the list does not hold them all
                u32 c0 = 0, per = end + 1, least = 0;
                u64 w = U64_MAX;
                while (c0 <= end) {
                    forget();
#pragma unroll
                    for (int j = 0; j < ITEMS; ++j) {
                        if (!((used >> j) & 1u)) continue;
                        const u32 d = delta_of(j), c = cell_of(j);
                        if (((sm.flag[c >> 5] >> (c & 31u)) & 1u) && c - c0 < per) {
                            const u32 at = atomicAdd(&sm.listed, 1u);
                            if (at < (u32)S::LIST) { sm.key[at] = key[j] & KEY; sm.delta[at] = d; sm.cell[at] = (u16)c; }
                        }
                    }
                    barrier_all();
                    const u32 total = sm.listed;
                    barrier_all();
                    if (tid == 0) sm.listed = 0;
                    if (total > (u32)S::LIST) {
                        if (per < end / 32 + 2) { slow = true; break; }
                        if (per > end) least = block_reduce_any<u32, NT>(low, sm.red, OpMin());
                        per /= 2 * ((total + S::LIST - 1) / S::LIST);
                        per = per ? per : 1u;
                        barrier_all();
                        continue;
                    }
                    for (u32 q = tid; q < total; q += NT) {
                        const u32 x = sm.key[q], c = sm.cell[q];
                        if (x < thrk) continue;
                        u32 w = (u32)sm.cells[S::word_of(c)] + __umul24((u32)P, x & mask);     // (the cell's deltas are below 2^30 in all)
                        for (u32 o = 0; o < total; ++o) w += sm.cell[o] == (u16)c && sm.key[o] > x ? sm.delta[o] : 0u;
                        const Best one{(u64)w, (u64)x};
                        if (one.before(got)) got = one;
                    }
                    const u64 one = got.d == U64_MAX ? U64_MAX : (got.d << 32) | got.x;
                    w = block_reduce_any<u64, NT>(one < w ? one : w, sm.red, OpMin());      // (the list may be written again)
                    if ((u32)(w >> 32) <= least) break;    // (a later one with this wait is not the first)
                    c0 += per;
                }
                if (slow) break;
                if (w == U64_MAX) { slow = true; break; }  // (never: the smallest upper bound is some entry's)
                best = Best{(u64)((i64)(w >> 32) + least_w), w & 0xffffffffull};
            } else {
                const u32 total = sm.listed;
                if (total > (u32)S::LIST || total * (u32)P > 65536u) { slow = true; break; }
                for (u32 q = tid; q < total * (u32)P; q += NT) {
                    const u32 ci = q / (u32)P;
                    const int p = (int)(q - ci * (u32)P);
                    const u64 x = (u64)rows.at((int)sm.key[ci]) - (u64)base;
                    if (x < thr) continue;
                    const u32 cnt = rows.upto(sm, p, (u64)base, x);
                    atomicAdd(&sm.acc[ci], x - ((u64)rows.value(p, (int)cnt - 1) - (u64)base));
                }
                barrier_all();
                for (u32 q = tid; q < total; q += NT) {
                    const u64 x = (u64)rows.at((int)sm.key[q]) - (u64)base;
                    const Best one{sm.acc[q], x};
                    if (x >= thr && one.before(got)) got = one;
                }
                best = block_first_min<NT>(got, sm.red);
                if (best.d == U64_MAX) { slow = true; break; }
            }
            slow = C != range && best.d > lbC;             // something behind C may win
        } while (false);
    }
    if (flags & EBSP_STATUS_UNSORTED)
        best = Best{0ull, 0ull};
    else if (slow) {
        if (tid == 0) wait[b] = DEFERRED;
        return;
    }
    const i64 bar = (i64)((u64)base + best.x);
    if (tid == 0) {
        barrier[b] = bar;
        wait[b] = (i64)best.d;
        if (status) status[b] = (int)flags;
    }
    if (tid < P) iters[b * (i64)P + tid] = (int)rows.upto(sm, tid, (u64)base, best.x);
}

}  // namespace
