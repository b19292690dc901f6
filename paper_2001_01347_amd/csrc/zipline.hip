// ZipLine barrier search for MI355X (gfx950, wave64).
//
// Implements the C ABI declared in include/ebsp_zipline.h.  The search is the
// sweep of Algorithm 2 of the ElasticBSP paper (arXiv 2001.01347) with the
// summed waiting time as objective (Section III; Fig. 1 caption), recast for
// a GPU:
//
//   * the set Z of Algorithm 2 (newest timestamp per worker) is never built.
//     With delta[p][i] = t[p][i] - t[p][i-1], the sum of the elements of Z
//     after the sweep has passed timestamp c is the prefix sum of the deltas
//     of all elements <= c in sorted order, so
//         wait(c) = P*c - prefix(c)
//     and the sweep becomes sort -> scan -> arg-min;
//   * every row of the input is already sorted (rows are iteration sequences,
//     Section III), so the merged set Omega can be cut into windows of
//     consecutive values without moving any data: a window takes one
//     contiguous segment of every row.  A window that fits in LDS is searched
//     by one workgroup, and the value of the prefix at the window start is
//     known from the row elements just before the segments, so windows need
//     no carry from one another;
//   * inside a window the sort is a counting sort into value buckets, exact
//     bounds per bucket drop the buckets that cannot hold the minimum, and
//     only the entries of the remaining buckets are ordered and evaluated;
//   * small instances (P*R <= 16384) are one window: one workgroup each, no
//     scratch memory.
//
// Device code, by header (each includes the one before it):
//   zl_common.h    types, records, wave/block primitives, the fine-bin map
//   zl_rows.h      rows of an instance (stored or predicted), zl_iters
//   zl_sort.h      general search of a window: radix sort, scan, arg-min
//   zl_bucket.h    fast search of a window: buckets, bounds, evaluation
//   zl_gather.h    zl_delta: row segments -> (key, delta) records in registers
//   zl_walk.h      general search of a value interval of any size
//   zl_instance.h  one workgroup per instance
//   zl_plan.h      zl_bounds, zl_partition, zl_bincount, zl_plan (the windows)
//   zl_window.h    window kernels of the summed-wait search
//   zl_range.h     the objective max(Z) - min(Z)
//   zl_finish.h    reduction over windows, zl_iters; the copy yardstick
//   zl_direct.h    predicted rows, every candidate evaluated; runs of supersteps side by side
//   zl_cells.h     one workgroup per stored instance of few rows: value cells
//   zl_slices.h    larger instances: value cells, in slices of an instance's values
//   zl_sweep.h     the frontier sweep: stored rows searched in one pass, no crossing table
//   zl_gridscan.h  GridScan and FullGridScan, the paper's comparators
// This file: the host side (plans, launches, the C entry points).
#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "ebsp_zipline.h"
#include "ebsp_zipline_bench.h"
#include "zl_gridscan.h"    // pulls in the other device headers, in dependency order

namespace {

// ---------------------------------------------------------------------------
// Host side.

thread_local char g_err[256] = "";

int fail(int code, const char* msg)
{
    snprintf(g_err, sizeof g_err, "%s", msg);
    return code;
}

// The kernels are built for gfx950 only: refuse any other device by name instead of
// letting a launch fail.  Asked once per device; the answer is kept.
int check_device()
{
    constexpr int KNOWN = 64;
    static std::atomic<signed char> seen[KNOWN];       // 0: not asked yet, 1: gfx950, -1: something else
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(EBSP_ERR_DEVICE, "no current HIP device");
    signed char state = dev >= 0 && dev < KNOWN ? seen[dev].load(std::memory_order_relaxed) : 0;
    if (state == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return fail(EBSP_ERR_DEVICE, "hipGetDeviceProperties failed");
        state = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : -1;
        if (dev >= 0 && dev < KNOWN) seen[dev].store(state, std::memory_order_relaxed);
    }
    if (state < 0) return fail(EBSP_ERR_DEVICE, "the current device is not a gfx950 (MI355X): this library has code for nothing else");
    return EBSP_OK;
}

enum KernelId { K_INSTANCE = 0, K_INSTANCE_GENERAL, K_BOUNDS, K_PARTITION, K_BINCOUNT, K_PLAN, K_WINDOW,
                K_WINDOW_GENERAL, K_FINISH, K_COPY, K_RANGE_INSTANCE, K_RANGE_FAST, K_PARTITION_PRED, K_RANGE_WINDOW, K_ADVANCE, K_SWEEP, K_SWEEP_FINISH, K_GRIDSCAN, K_GRIDSCAN_FINISH, K_READ, K_INSTANCE_REG, K_RUN, K_DIRECT, K_DIRECT_FINISH, K_CELLS, K_COUNT };
const char* const kKernelNames[K_COUNT] = {
    "zl_instance_kernel", "zl_instance_general_kernel", "zl_bounds_kernel", "zl_partition_kernel",
    "zl_bincount_kernel", "zl_plan_kernel", "zl_window_kernel", "zl_window_general_kernel",
    "zl_finish_kernel", "zl_copy_kernel", "zl_range_instance_kernel", "zl_range_fast_kernel",
    "zl_partition_pred_kernel", "zl_range_window_kernel", "zl_advance_kernel", "zl_sweep_kernel", "zl_sweep_finish_kernel", "zl_gridscan_kernel",
    "zl_gridscan_finish_kernel", "zl_read_kernel", "zl_instance_reg_kernel", "zl_run_kernel", "zl_direct_kernel",
    "zl_direct_finish_kernel", "zl_cells_kernel"};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Shape-dependent sizes of the multi-window path.
struct Tuning {          // 0: choose by shape
    int window_cap;
    int single_max;
    int window_fill;
    int sweep_min;       // smallest P*R that takes the frontier sweep (0: the default, < 0: never)
    int slice_keys;      // entries per slice of the sweep (0: chosen from the batch)
    int sweep_lines;     // lines of a plan of the sweep (0: chosen from P)
};
// Set before any thread calls a search (the header says so); read once per call, word by word.
std::atomic<int> g_tune_window_cap{0}, g_tune_single_max{0}, g_tune_window_fill{0}, g_tune_sweep_min{0}, g_tune_slice_keys{0}, g_tune_sweep_lines{0};
Tuning tuning()
{
    Tuning t;
    t.window_cap = g_tune_window_cap.load(std::memory_order_relaxed);
    t.single_max = g_tune_single_max.load(std::memory_order_relaxed);
    t.window_fill = g_tune_window_fill.load(std::memory_order_relaxed);
    t.sweep_min = g_tune_sweep_min.load(std::memory_order_relaxed);
    t.slice_keys = g_tune_slice_keys.load(std::memory_order_relaxed);
    t.sweep_lines = g_tune_sweep_lines.load(std::memory_order_relaxed);
    return t;
}

// The frontier sweep (zl_sweep.h) takes stored rows of these shapes under the summed-wait objective.
constexpr int SWEEP_NT = 512, SWEEP_LINES = 4096, SWEEP_BUCKETS = 4096, SWEEP_LIST = 2048;
constexpr int SWEEP_DEFAULT_ON = 1;              // 0: the sweep is the default for its shapes; 1: only where ebsp_zipline_tune_sweep asks for it
constexpr int SWEEP_MIN_DEFAULT = 8192;          // instances of fewer entries: one workgroup of zl_instance_kernel each
constexpr int SWEEP_PMAX = 1024;                 // every row with entries left needs a line of its own and one to spare

struct Plan {
    bool sweep;        // stored rows go through the frontier sweep
    int nslices;       // slices per instance there
    int lines;         // lines of a plan there
    size_t off_spartial, off_best, sweep_bytes;
    bool multi;
    int cap;           // records per window workgroup
    int fill;          // most entries of a window (unless a single fine bin holds more)
    int part_stored, part_pred;   // groups of rows whose column sums the partition kernels write (stored / predicted rows)
    int bins;          // fine bins per instance
    int stride;        // bins + 1 crossing indices per row
    int max_win;       // windows per instance <= max_win
    bool narrow;       // crossing indices fit 16 bits
    size_t off_info, off_seg, off_cross, off_part, off_below, off_winstart, off_winval, off_partial, off_rowpar, off_wide, bytes;
};

// single_limit: the most entries one workgroup takes whole on the path the plan is for;
// list_room: the scratch asked for under the range objective, whose size counts windows that leave a quarter or more of a
// workgroup's records free.  The kernels use range_rest_bytes of it; callers size buffers for several calls by it.
bool make_plan(i64 B, int P, int R, Plan& pl, int single_limit = SINGLE_MAX, bool list_room = false, bool stored_sum = false)
{
    if (B < 0 || P < 1 || R < 1) return false;
    const i64 n = (i64)P * (i64)R;
    if (n >= (1ll << 31)) return false;
    memset(&pl, 0, sizeof pl);
    const Tuning g_tune = tuning();
    {
        const i64 sweep_min = g_tune.sweep_min > 0 ? g_tune.sweep_min : SWEEP_MIN_DEFAULT;
        pl.sweep = stored_sum && g_tune.sweep_min >= SWEEP_DEFAULT_ON && n >= sweep_min && n < (1ll << 29) && P <= SWEEP_PMAX && B > 0;
        if (pl.sweep) {
            // about 2048 slices per batch (four rounds of two workgroups per CU), each long enough to pay for the
            // searches that open it (64 entries per row or more) and short enough to spread an instance over the chip
            i64 keys = g_tune.slice_keys > 0 ? g_tune.slice_keys : B * n / 2048;
            if (g_tune.slice_keys <= 0) {
                if (keys < 32768) keys = 32768;
                if (keys > 262144) keys = 262144;
                if (keys < 64ll * P) keys = 64ll * P;
            }
            i64 ns = (n + keys - 1) / keys;
            if (ns > 4096) ns = 4096;
            pl.nslices = (int)(ns < 1 ? 1 : ns);
            // four lines a row: a window then takes about forty entries of every row, most of what is loaded
            int lines = g_tune.sweep_lines > 0 ? g_tune.sweep_lines : 4 * P;
            lines = (lines + 31) / 32 * 32;
            if (lines < 2 * P) lines = (2 * P + 31) / 32 * 32;
            if (lines < 128) lines = 128;
            if (lines > SWEEP_LINES) lines = SWEEP_LINES;
            pl.lines = lines;
            size_t o = 0;                                       // (the first two as in the other layout below)
            pl.off_info = o;     o = align_up(o + (size_t)B * sizeof(InstInfo), 256);
            pl.off_seg = o;      o = align_up(o + (size_t)B * SEGS * sizeof(SegEntry), 256);
            pl.off_spartial = o; o = align_up(o + (size_t)B * pl.nslices * sizeof(Partial), 256);
            pl.off_best = o;     o = align_up(o + (size_t)B * sizeof(i64), 256);
            pl.sweep_bytes = o;
        }
    }
    int single_max = g_tune.single_max > 0 ? g_tune.single_max : SINGLE_MAX;
    if (single_max > single_limit) single_max = single_limit;
    pl.multi = n > single_max;
    if (!pl.multi) return true;
    // the per-window cost has a term proportional to P: larger windows for more rows
    pl.cap = g_tune.window_cap > 0 ? g_tune.window_cap : (P >= 1536 ? 16384 : (P >= 512 ? 8192 : 4096));
    const int fine_shift = (pl.cap == 16384 ? 14 : (pl.cap == 8192 ? 13 : 12)) - 3;       // fine bins of cap/8 keys on average
    pl.fill = g_tune.window_fill > 0 && g_tune.window_fill < pl.cap ? g_tune.window_fill : pl.cap;
    if (list_room) {
        // with few workers a larger share of a window's entries is min(Z) at some time and has to be listed
        const int room = P < 128 ? pl.cap / 2 : pl.cap / 4;
        if (pl.fill > pl.cap - room) pl.fill = pl.cap - room;
    }
    pl.bins = (int)((n + (1 << fine_shift) - 1) >> fine_shift);
    pl.stride = (pl.bins + 1 + 7) / 8 * 8;              // rows of cross start on 16-byte boundaries
    // two windows in a row hold more than `fill` keys, or they would be one; a whole number of workgroups per instance
    pl.max_win = (int)((2 * n / pl.fill + 3 + WINDOWS_PER_BLOCK - 1) / WINDOWS_PER_BLOCK * WINDOWS_PER_BLOCK);
    size_t o = 0;
    pl.off_info = o;     o = align_up(o + (size_t)B * sizeof(InstInfo), 256);
    pl.off_seg = o;      o = align_up(o + (size_t)B * SEGS * sizeof(SegEntry), 256);
    pl.narrow = R < 65536;
    pl.off_cross = o;    o = align_up(o + (size_t)B * P * pl.stride * (pl.narrow ? 2 : 4), 256);
    pl.part_stored = pl.stride <= PART_MAX_STRIDE ? (P + PART_ROWS - 1) / PART_ROWS : 0;     // 0: zl_bincount reads cross itself
    pl.part_pred = (P + PRED_ROWS_PER_BLOCK - 1) / PRED_ROWS_PER_BLOCK;
    const int part_rows = pl.part_stored > pl.part_pred ? pl.part_stored : pl.part_pred;
    pl.off_part = o;     o = align_up(o + (size_t)B * part_rows * pl.stride * sizeof(u32), 256);
    pl.off_below = o;    o = align_up(o + (size_t)B * pl.stride * sizeof(u32), 256);
    pl.off_winstart = o; o = align_up(o + (size_t)B * (pl.max_win + 1) * sizeof(u32), 256);
    pl.off_winval = o;   o = align_up(o + (size_t)B * pl.max_win * sizeof(WinVal), 256);
    pl.off_partial = o;  o = align_up(o + (size_t)B * pl.max_win * sizeof(Partial), 256);
    pl.off_rowpar = o;   o = align_up(o + (size_t)B * P * sizeof(uint2), 256);      // predicted rows only
    pl.off_wide = o;     o = align_up(o + (size_t)B * WIDE_MARKS * sizeof(u32), 256);
    pl.bytes = o;
    return true;
}

// Optional per-kernel timing: while a profile is open on this thread every
// launch is bracketed by two events taken from a pool created up front.
struct Profile {
    bool on = false;
    int max_calls = 0, calls = 0;
    hipEvent_t* ev = nullptr;      // [max_calls][K_COUNT][2]
    bool* used = nullptr;          // [max_calls][K_COUNT]
    float* share = nullptr;        // [max_calls]: what part of the durations recorded there the profile counts
};
thread_local Profile g_prof;

// The launches since the last count stood for n calls (the supersteps of a run that one launch takes whole).  Their
// durations are recorded with the first of them; of a run that passes max_calls the supersteps up to there count.
void prof_count(i64 n = 1)
{
    if (!g_prof.on || g_prof.calls >= g_prof.max_calls) return;
    const i64 left = g_prof.max_calls - g_prof.calls;
    g_prof.share[g_prof.calls] = n <= left ? 1.f : (float)left / (float)n;
    g_prof.calls += (int)(n <= left ? n : left);
}

hipEvent_t* prof_slot(int kid, int which)
{
    if (!g_prof.on || g_prof.calls >= g_prof.max_calls) return nullptr;
    if (which == 0) g_prof.used[g_prof.calls * K_COUNT + kid] = true;
    return &g_prof.ev[(g_prof.calls * K_COUNT + kid) * 2 + which];
}

#define LAUNCH(kid, kernel, grid, block, ...)                                              \
    do {                                                                                   \
        if (hipEvent_t* e0_ = prof_slot(kid, 0)) (void)hipEventRecord(*e0_, st);           \
        hipLaunchKernelGGL(kernel, grid, block, 0, st, __VA_ARGS__);                       \
        if (hipEvent_t* e1_ = prof_slot(kid, 1)) (void)hipEventRecord(*e1_, st);           \
        hipError_t e_ = hipGetLastError();                                                 \
        if (e_ != hipSuccess) {                                                            \
            snprintf(g_err, sizeof g_err, "%s: %s", kKernelNames[kid], hipGetErrorString(e_)); \
            return EBSP_ERR_LAUNCH;                                                        \
        }                                                                                  \
    } while (0)

// Batches of more planned windows than this (max_win is about twice the windows there are) first find out how far the
// values can win (zl_bounds).  What that saves grows with the batch and with how early some workers are through; what it
// costs hardly does: 7 to 25 us, with thousands of short-rowed instances more.  Calls without / with it, us, for workers
// of 95 to 105 ms, which leave nothing out | config 4's two groups | config 5's 20 to 200 ms:
//     68 x 1024 x 240   ( 4 352 planned)   164 / 172  |   160 / 170   |   164 / 140
//      8 x 1024 x 4096  ( 8 224)           288 / 290  |   298 / 250   |   287 / 170
//     64 x  256 x 1024  ( 8 448)           127 / 134  |   122 / 122   |   119 / 98
//    128 x  256 x 1024  (16 896)           207 / 211  |   200 / 187   |   199 / 140
//    273 x 1024 x 240   (17 472)           583 / 579  |   540 / 546   |   567 / 410
//     64 x 2048 x 1024  (16 640)          1226 / 1224 |  1206 / 1065  |  1191 / 620
//     64 x 1024 x 4096  (65 792)          1816 / 1785 |  1784 / 1555  |  1824 / 934
// The line lies where workers all alike
// lose no more than 2 % (the worst of some thousand drawn batches: predicted 8690 x 246 x 114, 1125 / 1164).
constexpr i64 CUT_MIN_WINDOWS = 16384;

// The front of the multi-window path: per-instance facts and fine-bin map, crossing indices, exact bin counts, windows.
int plan_windows(const Plan& pl, const i64* ts, const i64* le, const i64* iv, i64 B, int P, int R,
                 char* wsp, int* status, hipStream_t st)
{
    const bool pred = ts == nullptr;
    InstInfo* info = (InstInfo*)(wsp + pl.off_info);
    SegEntry* segtab = (SegEntry*)(wsp + pl.off_seg);
    void* cross = (void*)(wsp + pl.off_cross);
    u32* part = (u32*)(wsp + pl.off_part);
    u32* below = (u32*)(wsp + pl.off_below);
    u32* winstart = (u32*)(wsp + pl.off_winstart);
    WinVal* winval = (WinVal*)(wsp + pl.off_winval);
    uint2* rowpar = pred ? (uint2*)(wsp + pl.off_rowpar) : nullptr;
    u32* widebin = (u32*)(wsp + pl.off_wide);
    const i64 nrows = B * (i64)P;
    const i64 kblocks = (pl.stride + 255) / 256;
    const i64 widest = pl.part_stored > pl.part_pred ? pl.part_stored : pl.part_pred;
    if (kblocks * B > 0x7fffffffll || widest * B > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "batch too large for one call");
    const bool cut = B * (i64)pl.max_win > CUT_MIN_WINDOWS;
    // With the cut a thread's rows are chains of dependent loads and the workgroup steps through reductions.  512 threads
    // where the batch leaves CUs free anyway, fewer rows per chain; 256 beyond, more workgroups at once.  Calls with
    // 256 / 512 / 1024 threads, us: 64 x 1024 x 4096 939 / 932 / 942, 64 x 2048 x 1161 698 / 688 / 694, 192 x 600 x 654
    // 306 / 306 / 314, 320 x 600 x 392 349 / 351 / 362, 8000 x 300 x 60 1621 / 1629 / 1856, predicted 2542 x 378 x 239
    // 919 / 943 / 1032 (923 without the cut) and 3619 x 401 x 60 362 / 396 / 523 (472).
    if (cut && P > 512 && B <= GENERAL_GRID)
        LAUNCH(K_BOUNDS, (zl_bounds_kernel<512>), dim3((unsigned)B), dim3(512), ts, le, iv, P, R, pl.bins, info, segtab, rowpar, status,
               cut, (i64*)nullptr);
    else
        LAUNCH(K_BOUNDS, (zl_bounds_kernel<256>), dim3((unsigned)B), dim3(256), ts, le, iv, P, R, pl.bins, info, segtab, rowpar, status,
               cut, (i64*)nullptr);
    int part_rows;                                    // rows of partial column sums per instance (0: none, count from cross)
    if (pred) {
        part_rows = pl.part_pred;
        // two bins per thread where an instance's bins still make many workgroups
#define LAUNCH_PARTITION_PRED(CT_, KPT_)                                                                         \
    LAUNCH(K_PARTITION_PRED, (zl_partition_pred_kernel<CT_, KPT_>),                                              \
           dim3((unsigned)((pl.stride + 256 * KPT_ - 1) / (256 * KPT_) * B), (unsigned)part_rows), dim3(256),     \
           le, iv, P, R, info, segtab, (CT_*)cross, pl.stride, part)
        if (pl.stride >= 2048) {
            if (pl.narrow) LAUNCH_PARTITION_PRED(unsigned short, 2); else LAUNCH_PARTITION_PRED(u32, 2);
        } else {
            if (pl.narrow) LAUNCH_PARTITION_PRED(unsigned short, 1); else LAUNCH_PARTITION_PRED(u32, 1);
        }
#undef LAUNCH_PARTITION_PRED
    } else if (pl.part_stored > 0) {
        part_rows = pl.part_stored;
        if (pl.narrow)
            LAUNCH(K_PARTITION, zl_partition_sum_kernel<unsigned short>, dim3((unsigned)(B * part_rows)), dim3(PART_ROWS * WAVE),
                   ts, P, R, part_rows, info, widebin, segtab, (unsigned short*)cross, pl.stride, part, status);
        else
            LAUNCH(K_PARTITION, zl_partition_sum_kernel<u32>, dim3((unsigned)(B * part_rows)), dim3(PART_ROWS * WAVE),
                   ts, P, R, part_rows, info, widebin, segtab, (u32*)cross, pl.stride, part, status);
    } else {
        part_rows = 0;
        if (pl.narrow)
            LAUNCH(K_PARTITION, (zl_partition_kernel<256, unsigned short>), dim3((unsigned)((nrows + 3) / 4)), dim3(256),
                   ts, nrows, P, R, info, widebin, segtab, (unsigned short*)cross, pl.stride, status);
        else
            LAUNCH(K_PARTITION, (zl_partition_kernel<256, u32>), dim3((unsigned)((nrows + 3) / 4)), dim3(256),
                   ts, nrows, P, R, info, widebin, segtab, (u32*)cross, pl.stride, status);
    }
    if (part_rows > 0)        // the partial sums are exact counts already: nothing to clamp
        LAUNCH(K_BINCOUNT, zl_bincount_kernel<u32>, dim3((unsigned)(kblocks * B)), dim3(256),
               (const u32*)part, part_rows, 0x7fffffff, pl.stride, info, below);
    else if (pl.narrow)
        LAUNCH(K_BINCOUNT, zl_bincount_kernel<unsigned short>, dim3((unsigned)(kblocks * B)), dim3(256),
               (const unsigned short*)cross, P, R, pl.stride, info, below);
    else
        LAUNCH(K_BINCOUNT, zl_bincount_kernel<u32>, dim3((unsigned)(kblocks * B)), dim3(256),
               (const u32*)cross, P, R, pl.stride, info, below);
    if (pl.bins <= 1024)      // small instances, many of them: small workgroups
        LAUNCH(K_PLAN, (zl_plan_kernel<256, 1024>), dim3((unsigned)B), dim3(256), info, segtab, below, pl.stride, widebin, pred, winstart, winval,
               pl.max_win, (u32)pl.fill, (u32)(pl.cap / 8));
    else
        LAUNCH(K_PLAN, (zl_plan_kernel<1024, 4096>), dim3((unsigned)B), dim3(1024), info, segtab, below, pl.stride, widebin, pred, winstart, winval,
               pl.max_win, (u32)pl.fill, (u32)(pl.cap / 8));
    return EBSP_OK;
}

// Instances of 1024 entries or fewer take both searches in one launch, all supersteps of a run included
// (zl_run_kernel), where the batch's workgroups are on the chip together; a run's launches weigh more, so twice as
// many there.  Measured, us per superstep (64 of them) in separate launches / in one: 256 instances of 16 x 60 13.6 / 7.6,
// 1024 17.4 / 15.2, 1536 21.7 / 17.9, 2048 24.6 / 24.8, 3072 31.3 / 35.2; of 16 x 15 2048 16.5 / 8.2, 4096 21.4 / 15.8,
// 6144 (beyond the line) 27.9 / 23.0.  Single searches: 256 of 16 x 60 14.1 / 12.4, 1024 16.4 / 19.9, 1536 20.4 / 23.4;
// 2048 of 16 x 15 16.4 / 13.5, 3072 18.6 / 18.2, 4096 20.3 / 20.8.  Larger instances keep the separate kernels: with the
// general search in the same kernel 100 x 150 predicted took 55.6 us instead of 29.2.
bool takes_run_kernel(i64 S, i64 B, i64 n)
{
    if (n > 1024) return false;
    const i64 resident = (n <= 256 ? 8ll : 3ll) * GENERAL_GRID;
    return B <= (S > 1 ? 2 * resident : resident);
}

int launch_run(const i64* ts, const i64* le, const i64* iv, i64 sync_cost, i64 S, i64 B, int P, int R,
               i64* barrier, int* iters, i64* wait, int* status, hipStream_t st)
{
    const int rshift = (R & (R - 1)) == 0 ? __builtin_ctz((unsigned)R) : -1;
#define LAUNCH_RUN(NT_, ITEMS_, GITEMS_)                                                                    \
    do {                                                                                                    \
        if (ts) LAUNCH(K_RUN, (zl_run_kernel<NT_, ITEMS_, GITEMS_, false>), dim3((unsigned)B), dim3(NT_), ts, le, iv, \
                       sync_cost, (int)S, B, P, R, rshift, barrier, iters, wait, status);                   \
        else LAUNCH(K_RUN, (zl_run_kernel<NT_, ITEMS_, GITEMS_, true>), dim3((unsigned)B), dim3(NT_), ts, le, iv, \
                    sync_cost, (int)S, B, P, R, rshift, barrier, iters, wait, status);                      \
    } while (0)
    if (P * R <= 256) LAUNCH_RUN(128, 2, 4); else LAUNCH_RUN(256, 4, 8);
#undef LAUNCH_RUN
    return EBSP_OK;
}

// Which searches of predicted rows evaluate every candidate (zl_direct_kernel).  Its time goes with entries x workers, that
// of the bucket searches with the entries, so few workers are one reason, a batch that leaves the chip idle the other.
// Bucket searches / direct, us:
//   few workers    4096 of 16 x 64 34 / 18, of 32 x 32 33 / 25, of 40 x 25 36 / 28, of 48 x 20 35 / 32, of 64 x 16 34 / 41;
//                  4096 of 24 x 170 149 / 66, 2048 of 32 x 500 255 / 159, 1000 of 48 x 300 103 / 124;
//                  500 of 16 x 4096 228 / 102, 1000 of 24 x 2000 354 / 197, 100 of 32 x 4096 139 / 91
//                  (of more than 16384 entries the workers count: where some are through early, most windows are ruled out.
//                  Configuration 2's steady workers | configuration 5's 20 to 200 ms: 682 of 24 x 4096 440 / 239 | 277 / 234,
//                  3994 of 28 x 600 538 / 282 | 478 / 281, 585 of 28 x 4096 413 / 268 | 250 / 263, 2097 of 32 x 1000
//                  429 / 339 | 266 / 338, 2796 of 40 x 600 414 / 371 | 259 / 369, 409 of 40 x 4096 355 / 358 | 205 / 351;
//                  smaller batches of them 800 of 32 x 1000 224 / 130 | 200 / 133, 100 of 40 x 4096 181 / 110 | 135 / 108,
//                  200 of 40 x 4096 208 / 192 | 135 / 190)
//   small batches  one of 100 x 150 28.6 / 14.5, of 1024 x 15 26.7 / 22.6, 64 of 64 x 256 35 / 19, 40 of 200 x 60 26.5 / 25,
//                  128 of 100 x 150 31 / 41; one of 1000 x 150 60 / 45, 2 of 1000 x 100 101 / 52, 20 of 256 x 120 84 / 38;
//                  up to 1024 entries one of 100 x 10 10.6 / 10.9, of 128 x 8 11.4 / 12.1 (one launch as well)
//   supersteps     (per superstep, the searches side by side) 256 of 16 x 60 7.6 / 0.9, 1000 of 64 x 15 15 / 9.5, 500 of 100
//                  x 10 8.7 / 9; 64 of 64 x 60 29 / 2.5, 16 of 100 x 150 32 / 4.7, 8 of 1000 x 60 104 / 58
constexpr i64 DIRECT_NMAX = 1 << 18;             // a search has P / 4 workgroups at most: with more entries they are too few
bool takes_direct(i64 B, int P, i64 n, bool run)
{
    if (P > DIRECT_PMAX || n > DIRECT_NMAX) return false;
    if (P <= (n > 16384 ? 28 : n > 1024 ? 40 : run ? 64 : 48)) return true;
    if (P <= 40 && n > 16384) return B * n * P <= 900000000ll;
    return n > 1024 && B * n * P <= (n > 16384 ? 300000000ll : 100000000ll);
}

// Searches at0 .. at0 + count - 1 (zl_direct_kernel), recorded as kernel `kid`.  Batches that fill the chip: a wave per search of
// up to 4096 entries and 64 workers, four for larger ones (2048 of 16 x 1000 98 us with four, 109 with one; 4096 of 16 x 64
// 24 and 17).  Others: as many workgroups per search as its iters hold results for; with many workers, split among a
// workgroup's waves (one of 1000 x 150 45 us split, 55 not; of 256 x 60 14 and 20; of 256 x 240 22 and 20).
int launch_direct(int kid, const i64* le, const i64* iv, i64 B, i64 at0, i64 count, int P, int R, i64* barrier, int* iters, i64* wait,
                  int* status, hipStream_t st)
{
    const i64 n = (i64)P * R;
    const bool full = count * n >= 1 << 20;          // two waves of eight candidates a thread per SIMD
    const bool split = P > 64 && !full && count * n <= 1 << 18;
    const int nt = full && P <= 64 && n <= 4096 ? 64 : 256;
    int k = 4;
    if (nt == 64)                                    // as many candidates a thread as leave the fewest lanes empty
        for (const int more : {5, 8})
            if ((n + 64 * more - 1) / (64 * more) * more <= (n + 64 * k - 1) / (64 * k) * k) k = more;
    const i64 chunk = split ? 256 : (i64)nt * k;
    i64 G = (n + chunk - 1) / chunk;
    if (G > P / 4) G = P / 4;
    if (G < 1 || nt == 64 || count >= 2048 || n <= 1024) G = 1;
    const i64 per = ((n + G - 1) / G + chunk - 1) / chunk * chunk;
    G = (n + per - 1) / per;
#define LAUNCH_DIRECT(NT_, PM_, K_, SPLIT_)                                                                  \
    LAUNCH(kid, (zl_direct_kernel<NT_, PM_, K_, SPLIT_>), dim3((unsigned)(count * G)), dim3(NT_), le, iv, B, at0, P, R, \
           (int)G, (int)per, barrier, iters, wait, status)
    if (nt == 64) {
        if (k == 4) LAUNCH_DIRECT(64, 64, 4, false);
        else if (k == 5) LAUNCH_DIRECT(64, 64, 5, false);
        else LAUNCH_DIRECT(64, 64, 8, false);
    } else if (split) LAUNCH_DIRECT(256, DIRECT_PMAX, 4, true);
    else if (P <= 64) LAUNCH_DIRECT(256, 64, 4, false);
    else LAUNCH_DIRECT(256, DIRECT_PMAX, 4, false);
#undef LAUNCH_DIRECT
    if (G > 1) {
        if (P <= 64) LAUNCH(K_DIRECT_FINISH, (zl_direct_finish_kernel<64, 64>), dim3((unsigned)count), dim3(64), le, iv, B, at0, P, R, (int)G,
                            barrier, iters, wait, status);
        else LAUNCH(K_DIRECT_FINISH, (zl_direct_finish_kernel<256, DIRECT_PMAX>), dim3((unsigned)count), dim3(256), le, iv, B, at0, P, R, (int)G,
                    barrier, iters, wait, status);
    }
    return EBSP_OK;
}

// Which stored instances are searched over value cells (zl_cells_kernel): those of few rows (their ends are one wave's
// work), whose cells are narrow enough: a cell of range / NB values blurs a wait by P times that, R * sqrt(12 P) / NB of the
// standard deviation of the waits, and where that nears 1 too many entries have to be listed.  Bucket search / cells, us:
//   NB = 4096, 16 P R^2 / NB^2 = 0.6: 4000 of 24 x 160 138 / 84;  1.0: 4000 of 16 x 256 134 / 85;
//   1.2: 1000 of 8 x 400 42 / 58;  1.4: 1000 of 4 x 600 37 / 67
//   NB = 8192, 0.7: 4000 of 32 x 300 269 / 231;  1.0: 8000 of 64 x 256 588 / 494 (2000 of them 159 / 146);
//   1.4: 1000 of 24 x 500 85 / 105;  3.8: 1000 of 16 x 1000 170 / 358
// More rows: 8000 of 100 x 24 123 / 143, of 200 x 40 289 / 383, of 200 x 60 488 / 549.  Up to 2048 entries there is
// little to save (16384 of 64 x 30 162 / 179); between 4097 and 8192, with a chip's worth of instances or less (1 of 64 x 100
// 20.5 / 17, 300 27 / 27, 8192 of 64 x 128 310 / 364).
bool takes_cells(i64 B, int P, int R)
{
    const i64 n = (i64)P * R, nb = n <= 8192 ? 4096 : 8192;
    if (P > WAVE || 16 * n * R > nb * nb) return false;
    return (n > 2048 && n <= 4096) || n > 8192 || (n > 4096 && B <= GENERAL_GRID);
}

constexpr i64 RANGE_SMALL = 32768;               // entries of a slice that is small

// The search over value cells in slices (zl_slices_kernel), for instances of several windows.  Windows / slices, us, with
// configuration 2's steady workers | 5's 20 to 200 ms (one number: as named):
//   predicted rows   64 of 1024 x 4096 775 / 284 | 390 / 141, 1024 of 256 x 1024 764 / 287 | 391 / 173, 2542 of 378 x 239 930 / 424,
//                    8690 of 246 x 114 1150 / 824, 2000 of 1000 x 17 626 / 302, 1500 of 45 x 400 186 / 116, 500 of 100 x 200 110 / 66,
//                    100 of 300 x 100 73 / 50, 16 of 1000 x 150 69 / 63, 4 of 1000 x 100 64 / 57
//   stored rows      64 of 1024 x 4096 1517 / 866 | 933 / 663, 1024 of 256 x 1024 1141 / 854 | 779 / 663 (configuration 4 1158 / 909,
//                    in nanoseconds 1167 / 960), 512 of 64 x 4096 766 / 410 | 455 / 340, 2000 of 32 x 1024 597 / 479, 100 of 512 x
//                    1024 345 / 275, 900 of 64 x 1000 243 / 227 (5's)
//   windows with a cut (CUT_MIN_WINDOWS) leave out what lies behind the last value that can win, which for 5's workers is most, while
//                    every slice searches every row for its ends: of short rows, up to 100 million entries, 64 of 1024 x 1024 491 / 454 |
//                    285 / 328, 120 of 900 x 620 474 / 455 | 284 / 457, 100 of 768 x 1000 511 / 484 | 304 / 382, 200 of 600 x 600
//                    465 / 511 | 296 / 406, 300 of 400 x 600 442 / 537 | 287 / 317, 600 of 300 x 520 541 / 554 | 363 / 409; beyond
//                    (not short) 128 of 512 x 1024 415 / 376 | 252 / 265, 160 of 448 x 1000 430 / 340 | 262 / 272, 36 of 1024 x 2048
//                    574 / 401 | 328 / 321, (more) 400 of 600 x 520 780 / 700 | 511 / 512, 128 of 1024 x 1024 901 / 662 | 502 / 465,
//                    (no cut) 48 of 1021 x 1031 377 / 340 | 382 / 280, 100 of 1024 x 600 466 / 466 | 462 / 358
//   not those: fewer stored entries (64 of 256 x 1024 127 / 152) or instances (16 of 1024 x 4096 442 / 401 | 292 / 353), whose
//   slices are short; short rows, whose searches are most of it (273 of 1024 x 240 545 / 700, 8000 of 300 x 60 1622 / 2197); few
//   workers, whose cells have to be wide (100 of 12 x 4000 137 / 1750).
// Slower where waits repeat and all cells are alike, whose instances are searched again by windows without a table.  Workers of two
// intervals | of almost one: predicted 64 of 1024 x 4096 1135 / 2224 | 1241 / 2406, 1024 of 256 x 1024 1146 / 2504 | 1331 / 3100, 1000
// of 60 x 1000 438 / 909 | 493 / 987, 300 of 48 x 4000 415 / 1429 | 467 / 1617, 100 of 300 x 100 87 / 105 | 82 / 100 (nanoseconds: 14331 /
// 2298 | 14522 / 2401, 9130 / 2544 | 10482 / 3145, 2555 / 1146 | 2634 / 1240, 3102 / 2169 | 2815 / 2221, 289 / 107 | 285 / 102);
// stored rows without any jitter 256 of 256 x 1024 400 / 926 | 444 / 1245, 512 of 64 x 4096 1032 / 2080 | 1148 / 2485, 900 of 64 x 1000
// 481 / 999 | 515 / 1091.  One interval, predicted, is searched over one interval alone: 1296 / 57, 1351 / 91, 496 / 73, 470 / 44,
// 83 / 38.  Stored rows in step within 20 us | in nanoseconds: 256 of 256 x 1024 4470 / 3247 | 5245 / 3596, 1024 of 256 x 1024 9439
// / 11794 | 10907 / 13179, 60 of 1021 x 1031 3262 / 2246 | 3832 / 5003, 512 of 64 x 4096 2591 / 3800 | 2370 / 3970.
struct Slices {
    i64 count;           // per instance; 0: the search by windows
    u32 room;            // cells listed per slice
};
Slices plan_slices(const Plan& pl, i64 B, int P, int R, bool pred)
{
    Slices s{0, 0};
    const Tuning t = tuning();
    if (t.window_cap || t.single_max || t.window_fill || P < 8 || P > SLICE_PMAX || R < 8) return s;
    const i64 n = (i64)P * R;
    if (!pred && (P < 32 || R < 512 || B < 32 || B * n < 50000000)) return s;
    if (!pred && R < 2 * P && B * n < 100000000 && B * (i64)pl.max_win > CUT_MIN_WINDOWS) return s;
    // Two workgroups on every CU; one where that leaves a slice few entries.  More than 64 slices list more cells than they save time.
    i64 slices = 2 * GENERAL_GRID / B;
    if (slices > 1 && n / slices <= RANGE_SMALL) slices = GENERAL_GRID / B;
    const i64 most = n / 2048 < R / 4 ? n / 2048 : R / 4;
    if (slices > most) slices = most;
    if (slices > 64) slices = 64;
    if (slices < 1) slices = 1;
    for (;; slices = (slices + 1) / 2) {             // (callers size the workspace by the windows')
        const size_t fixed = slice_space_fixed(B, slices, pred ? 0 : P);
        const i64 room = fixed < pl.bytes ? (i64)((pl.bytes - fixed) / SLICE_CELL_BYTES) / (B * slices) : 0;
        if (room >= 64) { s.count = slices; s.room = (u32)(room < 4096 ? room : 4096); break; }
        if (slices == 1) break;
    }
    if (s.count * B * s.room > 0xfffffffell || s.count * B > 0x7fffffffll) s.count = 0;      // (cells are numbered in 32 bits)
    return s;
}

int launch_slices(const Slices& sl, const i64* ts, const i64* le, const i64* iv, i64 B, int P, int R, void* workspace,
                  i64* barrier, int* iters, i64* wait, int* status, hipStream_t st)
{
    const i64 n = (i64)P * R;
    const dim3 grid((unsigned)(B * sl.count));
#define LAUNCH_SLICES(NT_, NB_)                                                                              \
    do {                                                                                                     \
        if (ts) LAUNCH(K_WINDOW, (zl_slices_kernel<NT_, NB_, false>), grid, dim3(NT_), ts, le, iv, B, P, R, (u32)sl.count, workspace, sl.room); \
        else LAUNCH(K_WINDOW, (zl_slices_kernel<NT_, NB_, true>), grid, dim3(NT_), ts, le, iv, B, P, R, (u32)sl.count, workspace, sl.room); \
    } while (0)
    const bool many = n / sl.count > RANGE_SMALL;
    if (many) LAUNCH_SLICES(512, 16384);
    else LAUNCH_SLICES(512, 4096);
#undef LAUNCH_SLICES
#define LAUNCH_CELLS_OF(KERNEL_, KID_, NT_, GRID_)                                                           \
    LAUNCH(KID_, KERNEL_, dim3((unsigned)(GRID_)), dim3(NT_), ts, le, iv, B, P, R, (u32)sl.count, workspace, sl.room, barrier, iters, wait, status)
    const i64 cells_grid = 4 * GENERAL_GRID, rest_grid = 2 * GENERAL_GRID;
    if (ts) LAUNCH_CELLS_OF((zl_slices_queue_kernel<256, false>), K_PLAN, 256, B);
    else LAUNCH_CELLS_OF((zl_slices_queue_kernel<256, true>), K_PLAN, 256, B);
    if (ts) LAUNCH_CELLS_OF(zl_slices_cells_kernel<false>, K_FINISH, 256, cells_grid);
    else LAUNCH_CELLS_OF(zl_slices_cells_kernel<true>, K_FINISH, 256, cells_grid);
    if (ts) LAUNCH_CELLS_OF((zl_slices_rest_kernel<512, 8, false>), K_WINDOW_GENERAL, 512, rest_grid);
    else LAUNCH_CELLS_OF((zl_slices_rest_kernel<512, 8, true>), K_WINDOW_GENERAL, 512, rest_grid);
#undef LAUNCH_CELLS_OF
    return EBSP_OK;
}

// The rows are either stored (ts != nullptr) or predicted: t[p][i] = le[p] + (i + 1) * iv[p] (ts == nullptr; direct: every
// candidate may be evaluated).
int run_batch(const i64* ts, const i64* le, const i64* iv, i64 B, int P, int R,
              i64* barrier, int* iters, i64* wait, int* status,
              void* workspace, size_t workspace_bytes, hipStream_t st, bool direct = true)
{
    Plan pl;
    const bool pred = ts == nullptr;
    if (!make_plan(B, P, R, pl, SINGLE_MAX, false, !pred)) return fail(EBSP_ERR_SHAPE, "invalid shape: need B >= 0, P >= 1, R >= 1, P*R < 2^31");
    if (B == 0) return EBSP_OK;
    if ((pred && (!le || !iv)) || !barrier || !iters || !wait)
        return fail(EBSP_ERR_NULL, "the input arrays, barrier, iters and wait must not be NULL");
    if (B > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "B must be below 2^31");
    const int n = P * R;

    if (pl.sweep) {
        // stored rows in one pass: instance facts and slices, the sweep, the reduction over slices with zl_iters
        if (!workspace) return fail(EBSP_ERR_NULL, "this shape needs a workspace");
        if (workspace_bytes < pl.sweep_bytes) return fail(EBSP_ERR_WORKSPACE, "workspace smaller than ebsp_zipline_workspace_bytes()");
        if (((uintptr_t)workspace & 255u) != 0) return fail(EBSP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
        const i64 pblocks = (P + 255) / 256;
        if (B * (i64)pl.nslices > 0x7fffffffll || pblocks * B > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "batch too large for one call");
        if (int rc = check_device()) return rc;
        char* wsp = (char*)workspace;
        InstInfo* info = (InstInfo*)(wsp + pl.off_info);
        SegEntry* segtab = (SegEntry*)(wsp + pl.off_seg);
        Partial* spartial = (Partial*)(wsp + pl.off_spartial);
        i64* best = (i64*)(wsp + pl.off_best);
        LAUNCH(K_BOUNDS, (zl_bounds_kernel<256>), dim3((unsigned)B), dim3(256), ts, le, iv, P, R, pl.nslices, info, segtab,
               (uint2*)nullptr, status, false, best);
        const dim3 sgrid((unsigned)(B * (i64)pl.nslices));
        LAUNCH(K_SWEEP, (zl_sweep_kernel<SWEEP_NT, SWEEP_LINES, SWEEP_BUCKETS, SWEEP_LIST, SWEEP_PMAX>), sgrid, dim3(SWEEP_NT),
               ts, B, P, R, pl.nslices, pl.lines, info, segtab, best, spartial, status);
        LAUNCH(K_SWEEP_FINISH, (zl_sweep_finish_kernel<256>), dim3((unsigned)(pblocks * B)), dim3(256),
               ts, P, R, pl.nslices, info, spartial, barrier, iters, wait);
        return EBSP_OK;
    }

    if (!pl.multi) {
        if (int rc = check_device()) return rc;
        if (pred && direct && takes_direct(B, P, n, false)) return launch_direct(K_DIRECT, le, iv, B, 0, B, P, R, barrier, iters, wait, status, st);
        const int rshift = (R & (R - 1)) == 0 ? __builtin_ctz((unsigned)R) : -1;
        const dim3 grid((unsigned)B);
        if (takes_run_kernel(1, B, n)) return launch_run(ts, le, iv, 0, 1, B, P, R, barrier, iters, wait, status, st);
#define LAUNCH_INSTANCE(NT_, ITEMS_)                                                                        \
    do {                                                                                                    \
        if (pred) LAUNCH(K_INSTANCE, (zl_instance_kernel<NT_, ITEMS_, true>), grid, dim3(NT_), ts, le, iv, P, R, rshift, \
                         barrier, iters, wait, status);                                                     \
        else LAUNCH(K_INSTANCE, (zl_instance_kernel<NT_, ITEMS_, false>), grid, dim3(NT_), ts, le, iv, P, R, rshift, \
                    barrier, iters, wait, status);                                                          \
    } while (0)
#define LAUNCH_CELLS(NT_, ITEMS_, NB_)                                                                      \
    LAUNCH(K_CELLS, (zl_cells_kernel<NT_, ITEMS_, NB_>), grid, dim3(NT_), ts, P, R, rshift, barrier, iters, wait, status)
        // larger instances keep their records in registers: less LDS, several workgroups per CU
#define LAUNCH_INSTANCE_REG(NT_, ITEMS_)                                                                    \
    do {                                                                                                    \
        if (pred) LAUNCH(K_INSTANCE_REG, (zl_instance_reg_kernel<NT_, ITEMS_, true>), grid, dim3(NT_), ts, le, iv, P, R, rshift, \
                         barrier, iters, wait, status);                                                     \
        else LAUNCH(K_INSTANCE_REG, (zl_instance_reg_kernel<NT_, ITEMS_, false>), grid, dim3(NT_), ts, le, iv, P, R, rshift, \
                    barrier, iters, wait, status);                                                          \
    } while (0)
        if (n <= 256) LAUNCH_INSTANCE(128, 2);
        else if (!pred && takes_cells(B, P, R)) {
            // small batches: the shorter chain per thread wins (1 of 64 x 60 15.6 us, with 256 threads 17.4; 8000 178 / 156)
            if (n <= 4096 && B <= GENERAL_GRID) LAUNCH_CELLS(512, 8, 4096);
            else if (n <= 4096) LAUNCH_CELLS(256, 16, 4096);
            else if (n <= 8192) LAUNCH_CELLS(512, 16, 4096);
            else if (B <= GENERAL_GRID) LAUNCH_CELLS(1024, 16, 8192);
            else LAUNCH_CELLS(512, 32, 8192);
        } else if (n <= 1024) LAUNCH_INSTANCE(256, 4);       // (batches of so small instances are often small too: the shorter chain per thread wins)
        else if (n <= 2048) LAUNCH_INSTANCE_REG(256, 8);
        else if (n <= 4096) LAUNCH_INSTANCE_REG(256, 16);
        else if (n <= 8192) LAUNCH_INSTANCE_REG(512, 16);
        else LAUNCH_INSTANCE_REG(1024, 16);
#undef LAUNCH_INSTANCE_REG
#undef LAUNCH_CELLS
#undef LAUNCH_INSTANCE
        // what the kernel above left: the general search in the smallest workgroup whose records hold an
        // instance (half of NT * ITEMS with 64-bit deltas), as many workgroups as fit the chip at once
#define LAUNCH_GENERAL(NT_, ITEMS_, PER_CU_)                                                                 \
    LAUNCH(K_INSTANCE_GENERAL, (zl_instance_general_kernel<NT_, ITEMS_>),                                    \
           dim3((unsigned)(B < PER_CU_ * GENERAL_GRID ? B : PER_CU_ * GENERAL_GRID)), dim3(NT_),            \
           ts, le, iv, B, P, R, barrier, iters, wait, status)
        if (n <= 1024) LAUNCH_GENERAL(256, 8, 7);
        else if (n <= 2048) LAUNCH_GENERAL(256, 16, 4);
        else if (n <= 4096) LAUNCH_GENERAL(512, 16, 2);
        else LAUNCH_GENERAL(LARGE_NT, LARGE_ITEMS, 1);
#undef LAUNCH_GENERAL
        return EBSP_OK;
    }

    if (!workspace) return fail(EBSP_ERR_NULL, "this shape needs a workspace");
    if (workspace_bytes < pl.bytes) return fail(EBSP_ERR_WORKSPACE, "workspace smaller than ebsp_zipline_workspace_bytes()");
    if (((uintptr_t)workspace & 255u) != 0) return fail(EBSP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    const i64 total_win = B * (i64)pl.max_win;
    if (total_win + 8 > 0x7fffffffll || B * (i64)P > (0x7fffffffll * 4)) return fail(EBSP_ERR_SHAPE, "batch too large for one call");

    char* wsp = (char*)workspace;
    InstInfo* info = (InstInfo*)(wsp + pl.off_info);
    void* cross = (void*)(wsp + pl.off_cross);
    u32* winstart = (u32*)(wsp + pl.off_winstart);
    WinVal* winval = (WinVal*)(wsp + pl.off_winval);
    u32* below = (u32*)(wsp + pl.off_below);
    Partial* partial = (Partial*)(wsp + pl.off_partial);
    uint2* rowpar = pred ? (uint2*)(wsp + pl.off_rowpar) : nullptr;

    const i64 pblocks = (P + 255) / 256;
    if (pblocks * B > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "batch too large for one call");
    if (int rc = check_device()) return rc;
    if (pred && direct && takes_direct(B, P, n, false)) return launch_direct(K_DIRECT, le, iv, B, 0, B, P, R, barrier, iters, wait, status, st);
    if (const Slices sl = plan_slices(pl, B, P, R, pred); sl.count)
        return launch_slices(sl, ts, le, iv, B, P, R, workspace, barrier, iters, wait, status, st);
    if (int rc = plan_windows(pl, ts, le, iv, B, P, R, wsp, status, st)) return rc;
    // Batches whose windows are all on the chip at once (two workgroups per CU; max_win is about twice the windows
    // there are) are as fast as one workgroup: a window each instead of two.
    const bool one_each = pl.narrow && total_win <= 4 * GENERAL_GRID;
    const u32 groups = (u32)(one_each ? pl.max_win : pl.max_win / WINDOWS_PER_BLOCK);
    const u32 groups_inv = groups > 1 ? (u32)((1ull << 32) / groups) : 0xffffffffu;
    const unsigned wgrid = (unsigned)((B * (i64)groups + 7) / 8 * 8);
#define LAUNCH_WINDOW(NT_, CT_, W_)                                                                          \
    do {                                                                                                     \
        if (pred) LAUNCH(K_WINDOW, (zl_window_kernel<NT_, 16, CT_, true, W_>), dim3(wgrid), dim3(NT_), ts, rowpar, B, P, R, info, \
                         (const CT_*)cross, pl.stride, winstart, winval, pl.max_win, groups, groups_inv, below, partial); \
        else LAUNCH(K_WINDOW, (zl_window_kernel<NT_, 16, CT_, false, W_>), dim3(wgrid), dim3(NT_), ts, rowpar, B, P, R, info, \
                    (const CT_*)cross, pl.stride, winstart, winval, pl.max_win, groups, groups_inv, below, partial);  \
    } while (0)
#define LAUNCH_WINDOWS(NT_)                                                                                  \
    do {                                                                                                     \
        if (one_each) LAUNCH_WINDOW(NT_, unsigned short, 1);                                                 \
        else if (pl.narrow) LAUNCH_WINDOW(NT_, unsigned short, WINDOWS_PER_BLOCK);                           \
        else LAUNCH_WINDOW(NT_, u32, WINDOWS_PER_BLOCK);                                                     \
    } while (0)
    if (pl.cap == 16384) LAUNCH_WINDOWS(1024);
    else if (pl.cap == 8192) LAUNCH_WINDOWS(512);
    else LAUNCH_WINDOWS(256);
#undef LAUNCH_WINDOWS
#undef LAUNCH_WINDOW
    if (pl.cap <= 4096)       // such windows fit a 512-thread workgroup's general search: two workgroups per CU
        LAUNCH(K_WINDOW_GENERAL, (zl_window_general_kernel<512, 16>),
               dim3((unsigned)(total_win < 2 * GENERAL_GRID ? total_win : 2 * GENERAL_GRID)), dim3(512),
               ts, le, iv, B, P, R, info, cross, pl.narrow, pl.stride, winstart, winval, pl.max_win, partial, status);
    else
        LAUNCH(K_WINDOW_GENERAL, (zl_window_general_kernel<LARGE_NT, LARGE_ITEMS>),
               dim3((unsigned)(total_win < GENERAL_GRID ? total_win : GENERAL_GRID)), dim3(LARGE_NT),
               ts, le, iv, B, P, R, info, cross, pl.narrow, pl.stride, winstart, winval, pl.max_win, partial, status);
    LAUNCH(K_FINISH, (zl_finish_kernel<256>), dim3((unsigned)(pblocks * B)), dim3(256),
           ts, le, iv, P, R, info, (const SegEntry*)(wsp + pl.off_seg), (const void*)cross, pl.narrow, pl.stride,
           partial, pl.max_win, barrier, iters, wait);
    return EBSP_OK;
}

// The search under the paper's formal objective: small instances in registers, others in slices of their values.
constexpr int RANGE_SINGLE_MAX = WinCfg<LARGE_NT, LARGE_ITEMS>::CAP_WIDE;      // larger ones need a workspace

int run_range_batch(const i64* ts, i64 B, int P, int R, i64* barrier, int* iters, i64* dmin, int* status,
                    void* workspace, size_t workspace_bytes, hipStream_t st)
{
    Plan pl;
    if (!make_plan(B, P, R, pl, RANGE_SINGLE_MAX, true))
        return fail(EBSP_ERR_SHAPE, "invalid shape: need B >= 0, P >= 1, R >= 1, P*R < 2^31");
    if (B == 0) return EBSP_OK;
    if (!ts || !barrier || !iters || !dmin) return fail(EBSP_ERR_NULL, "ts, barrier, iters and dmin must not be NULL");
    if (B > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "B must be below 2^31");
    const i64 n = (i64)P * R, pblocks = (P + 255) / 256;
    if (pl.multi) {
        if (!workspace) return fail(EBSP_ERR_NULL, "this shape needs a workspace");
        if (workspace_bytes < pl.bytes) return fail(EBSP_ERR_WORKSPACE, "workspace smaller than ebsp_zipline_range_workspace_bytes()");
        if (((uintptr_t)workspace & 255u) != 0) return fail(EBSP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
        if (B * (i64)pl.max_win + 8 > 0x7fffffffll || pblocks * B > 0x7fffffffll)
            return fail(EBSP_ERR_SHAPE, "batch too large for one call");
    }
    if (int rc = check_device()) return rc;
    const int knob = tuning().single_max;
    // In registers where an instance has at most 4096 entries and eight cells or more per iteration (fewer leave too many
    // entries to evaluate).  In registers / as one slice, us: 8192 of 64 x 64 128 / 214, 16384 of 64 x 30 160 / 261, 8000 of
    // 200 x 20 135 / 202; larger ones 8192 of 64 x 128 316 / 262, 4096 of 64 x 256 513 / 172 (32 waves of 64 registers per
    // CU, spilling); long rows 8192 of 4 x 1000 with 4096 cells in registers 1110, as a slice of 8192 cells 333.
    if (n <= 4096 && n <= (knob > 0 ? knob : SINGLE_MAX) && 8ll * R <= (n <= 256 && R <= 64 ? 512 : n <= 1024 ? 2048 : 4096)) {
        const int rshift = (R & (R - 1)) == 0 ? __builtin_ctz((unsigned)R) : -1;
#define LAUNCH_RANGE(NT_, ITEMS_, NB_, REST_)                                                                \
    LAUNCH(K_RANGE_INSTANCE, (zl_range_instance_kernel<NT_, ITEMS_, NB_, REST_>), dim3((unsigned)B), dim3(NT_), \
           ts, P, R, rshift, barrier, iters, dmin, status)
        // Two waves for up to 1024 entries: with one / two / four, us: 4096 of 16 x 64 28.9 / 23.6 / 34.7, 16384 of them
        // 73 / 69 / 109, 512 of them 19.6 / 15.0 / 16.5; with half the cells 32.3 / 29.3 and more.
        if (n <= 256 && R <= 64) { LAUNCH_RANGE(64, 4, 512, false); return EBSP_OK; }
        if (n <= 1024) { LAUNCH_RANGE(128, 8, 2048, false); return EBSP_OK; }      // (they never give up)
        LAUNCH_RANGE(256, 16, 4096, true);
#undef LAUNCH_RANGE
        LAUNCH(K_RANGE_WINDOW, (zl_range_window_kernel<512, 16, 16384, false>), dim3((unsigned)(B < 2 * GENERAL_GRID ? B : 2 * GENERAL_GRID)),
               dim3(512), ts, B, P, R, 1u, 0, (RangePart*)nullptr, barrier, iters, dmin, status);
        return EBSP_OK;
    }
    RangePart* part = pl.multi ? (RangePart*)workspace : nullptr;        // (one slice needs none)
    i64 slices = 1;
    if (pl.multi) {
        // Two workgroups on every CU; one where that leaves a slice little to read against what it pays per row (its ends
        // and two searches), and four entries of a row or more.  Slices 4 / 8 / 16 / 32 / 64, us: 64 of 1024 x 4096 804 / 604
        // / 767 / 1066 / 1651, 8 of them - / - / 251 / 226 / 243; 16 of 1000 x 150 116 / 83 / 74 / 92 / -, one of them 87 /
        // 53 / 41 / 38 / -.
        slices = 2 * GENERAL_GRID / B;
        if (slices > 1 && n / slices <= RANGE_SMALL) slices = GENERAL_GRID / B;
        const i64 most = n / 2048 < R / 4 ? n / 2048 : R / 4;
        if (slices > most) slices = most;
        if (slices < (R + 2047) / 2048) slices = (R + 2047) / 2048;      // eight cells per iteration
        if (slices > 0x7fffffffll / B) slices = 0x7fffffffll / B;
        while (slices > 1 && range_rest_bytes(B, slices) > pl.bytes) --slices;
        if (slices < 1) slices = 1;
    }
    // whole waves walk a row's stretch where it is long enough
    int lanes_log = 6;
    while (lanes_log > 0 && (1ll << lanes_log) * slices * 4 > 5 * (i64)R) --lanes_log;
    const i64 cells = 8 * (R / slices);
    const dim3 grid((unsigned)(B * slices));
#define LAUNCH_SLICE(NT_, NB_)                                                                               \
    LAUNCH(K_RANGE_FAST, (zl_range_fast_kernel<NT_, NB_>), grid, dim3(NT_), ts, P, R, (u32)slices, lanes_log, part, \
           barrier, iters, dmin, status)
    // Workgroups of 512 threads and 16384 cells (two per CU) for slices of many entries, of 256 and 4096 (six) for others,
    // of 512 where few of them have many rows to search.  512 x 16384 / 256 x 4096, us: 1024 of 256 x 1024 518 / 830 (8192
    // cells), 1000 of 300 x 300 244 / 283, 1000 of 500 x 100 223 / 244; 2000 of 300 x 60 254 / 225, 4096 of 64 x 256 258 /
    // 172.  256 / 512 threads, 4096 cells: one of 1000 x 150 41.8 / 38.1, 8000 of 300 x 30 422 / 497.
    const bool many = n / slices > RANGE_SMALL || cells > 8192;
    if (many) LAUNCH_SLICE(512, 16384);
    else if (cells > 4096) LAUNCH_SLICE(256, 8192);
    else if (P > 256 && B * slices <= 2 * GENERAL_GRID) LAUNCH_SLICE(512, 4096);
    else LAUNCH_SLICE(256, 4096);
#undef LAUNCH_SLICE
#define LAUNCH_REST(NB_)                                                                                     \
    LAUNCH(K_RANGE_WINDOW, (zl_range_window_kernel<512, 16, NB_, true>),                                     \
           dim3((unsigned)(slices > 1 ? B * slices : B < 2 * GENERAL_GRID ? B : 2 * GENERAL_GRID)),          \
           dim3(512), ts, B, P, R, (u32)slices, lanes_log, part, barrier, iters, dmin, status)
    if (many || cells > 4096) LAUNCH_REST(16384);
    else LAUNCH_REST(4096);
#undef LAUNCH_REST
    return EBSP_OK;
}

// Scratch of the entry point that allocates nothing: a file-scope device array that every GPU the
// library runs on holds until the process ends.  In host code the array's name is only a handle
// for hipGetSymbolAddress; its device address is asked for once per device and kept.
static __device__ __align__(256) unsigned char scratch[EBSP_STATIC_SCRATCH_BYTES];

int static_scratch(void** out)
{
    constexpr int KNOWN = 64;
    static std::atomic<void*> base[KNOWN];             // per device: where that GPU's copy of the array lives
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(EBSP_ERR_DEVICE, "no current HIP device");
    if (dev < 0 || dev >= KNOWN) return fail(EBSP_ERR_DEVICE, "device ordinal beyond what the static scratch table holds");
    void* ptr = base[dev].load(std::memory_order_acquire);
    if (!ptr) {
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            snprintf(g_err, sizeof g_err, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
            return EBSP_ERR_DEVICE;
        }
        base[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return EBSP_OK;
}

}  // namespace

extern "C" {

size_t ebsp_zipline_static_scratch_bytes(void) { return (size_t)EBSP_STATIC_SCRATCH_BYTES; }

int ebsp_zipline_batch_static(const int64_t* ts, int64_t B, int32_t P, int32_t R,
                              int64_t* barrier, int32_t* iters, int64_t* wait, int32_t* status, void* stream)
{
    if (!ts && B > 0) return fail(EBSP_ERR_NULL, "ts must not be NULL");
    Plan pl;
    if (!make_plan(B, P, R, pl, SINGLE_MAX, false, true)) return fail(EBSP_ERR_SHAPE, "invalid shape: need B >= 0, P >= 1, R >= 1, P*R < 2^31");
    const size_t need = pl.sweep ? pl.sweep_bytes : (pl.multi ? pl.bytes : 0);
    if (need > (size_t)EBSP_STATIC_SCRATCH_BYTES) {
        snprintf(g_err, sizeof g_err, "this batch needs %zu bytes of scratch, the static scratch holds %zu: "
                 "use fewer instances per call or ebsp_zipline_batch with a workspace", need, (size_t)EBSP_STATIC_SCRATCH_BYTES);
        return EBSP_ERR_WORKSPACE;
    }
    void* ptr = nullptr;
    if (B > 0)
        if (int rc = static_scratch(&ptr)) return rc;
    const int rc = run_batch((const i64*)ts, nullptr, nullptr, B, P, R, (i64*)barrier, iters, (i64*)wait, status,
                             ptr, (size_t)EBSP_STATIC_SCRATCH_BYTES, (hipStream_t)stream);
    if (rc == EBSP_OK && B > 0) prof_count();
    return rc;
}

size_t ebsp_zipline_workspace_bytes(int64_t B, int32_t P, int32_t R)
{
    Plan pl;
    if (!make_plan(B, P, R, pl, SINGLE_MAX, false, true)) return 0;
    if (pl.sweep) return pl.sweep_bytes;
    return pl.multi ? pl.bytes : 0;
}

size_t ebsp_predict_zipline_workspace_bytes(int64_t B, int32_t P, int32_t R)
{
    Plan pl;
    if (!make_plan(B, P, R, pl)) return 0;
    return pl.multi ? pl.bytes : 0;
}

int ebsp_zipline_batch(const int64_t* ts, int64_t B, int32_t P, int32_t R,
                       int64_t* barrier, int32_t* iters, int64_t* wait,
                       int32_t* status, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!ts && B > 0) return fail(EBSP_ERR_NULL, "ts must not be NULL");
    const int rc = run_batch((const i64*)ts, nullptr, nullptr, B, P, R, (i64*)barrier, iters, (i64*)wait, status,
                             workspace, workspace_bytes, (hipStream_t)stream);
    if (rc == EBSP_OK && B > 0) prof_count();
    return rc;
}

int ebsp_predict_zipline_batch(const int64_t* last_end, const int64_t* interval, int64_t B, int32_t P, int32_t R,
                               int64_t* barrier, int32_t* iters, int64_t* wait,
                               int32_t* status, void* workspace, size_t workspace_bytes, void* stream)
{
    if ((!last_end || !interval) && B > 0) return fail(EBSP_ERR_NULL, "last_end and interval must not be NULL");
    const int rc = run_batch(nullptr, (const i64*)last_end, (const i64*)interval, B, P, R, (i64*)barrier, iters,
                             (i64*)wait, status, workspace, workspace_bytes, (hipStream_t)stream);
    if (rc == EBSP_OK && B > 0) prof_count();
    return rc;
}

size_t ebsp_simulate_workspace_bytes(int64_t B, int32_t P, int32_t R)
{
    Plan pl;
    if (!make_plan(B, P, R, pl)) return 0;
    return align_up(pl.multi ? pl.bytes : 0, 256) + align_up((size_t)B * P * sizeof(i64), 256);   // + the workers' current start times
}

int ebsp_simulate_supersteps(const int64_t* last_end0, const int64_t* interval, int64_t sync_cost,
                             int64_t S, int64_t B, int32_t P, int32_t R, int64_t* barrier, int32_t* iters, int64_t* wait, int32_t* status,
                             void* workspace, size_t workspace_bytes, void* stream)
{
    Plan pl;
    if (S < 0 || sync_cost < 0 || !make_plan(B, P, R, pl))
        return fail(EBSP_ERR_SHAPE, "invalid shape: need S >= 0, sync_cost >= 0, B >= 0, P >= 1, R >= 1, P*R < 2^31");
    if (S == 0 || B == 0) return EBSP_OK;
    if (!last_end0 || !interval) return fail(EBSP_ERR_NULL, "last_end0 and interval must not be NULL");
    if (!barrier || !iters || !wait) return fail(EBSP_ERR_NULL, "barrier, iters and wait must not be NULL");
    if (!workspace) return fail(EBSP_ERR_NULL, "the simulation needs a workspace");
    if (((uintptr_t)workspace & 255u) != 0) return fail(EBSP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    const size_t search_bytes = align_up(pl.multi ? pl.bytes : 0, 256);
    if (workspace_bytes < search_bytes + (size_t)B * P * sizeof(i64))
        return fail(EBSP_ERR_WORKSPACE, "workspace smaller than ebsp_simulate_workspace_bytes()");
    if ((B * (i64)P + 255) / 256 > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "batch too large for one call");
    hipStream_t st = (hipStream_t)stream;
    i64* start = (i64*)((char*)workspace + search_bytes);
    const i64 per = B * (i64)P;
    const i64 n = (i64)P * R;
    // All supersteps side by side (zl_direct_kernel, timed as zl_run_kernel like the other launch that takes a run whole); of
    // instances of more than 1024 entries the first one, whose workers have start times of their own, by a bucket search.
    if (S > 1 && S * B * (P / 4 + 1) <= 0x7fffffffll && takes_direct(B, P, n, true)) {
        if (int rc = check_device()) return rc;
        const i64 s0 = n > 1024 ? 1 : 0;
        if (s0 == 1) {
            if (int rc = run_batch(nullptr, (const i64*)last_end0, (const i64*)interval, B, P, R, (i64*)barrier, iters, (i64*)wait, status,
                                   workspace, search_bytes, st, false)) return rc;
            prof_count();
        }
        if (int rc = launch_direct(K_RUN, (const i64*)last_end0, (const i64*)interval, B, s0 * B, (S - s0) * B, P, R, (i64*)barrier, iters,
                                   (i64*)wait, status, st)) return rc;
#define LAUNCH_STARTS(NT_, PM_)                                                                              \
    LAUNCH(K_ADVANCE, (zl_direct_starts_kernel<NT_, PM_, 4>), dim3((unsigned)B), dim3(NT_), (const i64*)last_end0, \
           (const i64*)interval, (i64)sync_cost, (int)S, B, P, R, (i64*)barrier, iters, (i64*)wait, status)
        if (P <= 64 && n <= 4096) LAUNCH_STARTS(64, 64);
        else LAUNCH_STARTS(1024, DIRECT_PMAX);
#undef LAUNCH_STARTS
        prof_count(S - s0);
        return EBSP_OK;
    }
    if (!pl.multi && S <= 0x7fffffffll && B <= 0x7fffffffll && takes_run_kernel(S, B, (i64)P * R)) {
        if (int rc = check_device()) return rc;
        if (int rc = launch_run(nullptr, (const i64*)last_end0, (const i64*)interval, (i64)sync_cost, S, B, P, R, (i64*)barrier,
                                iters, (i64*)wait, status, st)) return rc;
        prof_count(S);
        return EBSP_OK;
    }
    for (i64 s = 0; s < S; ++s) {
        const i64* from = s == 0 ? (const i64*)last_end0 : start;
        int* flags = status ? status + s * B : nullptr;
        const int rc = run_batch(nullptr, from, (const i64*)interval + s * per, B, P, R, (i64*)barrier + s * B, iters + s * per,
                                 (i64*)wait + s * B, flags, workspace, search_bytes, st);
        if (rc != EBSP_OK) return rc;
        if (s + 1 < S)       // the workers' start times of the next superstep (after the last one barrier[S-1] says it all)
            LAUNCH(K_ADVANCE, zl_advance_kernel, dim3((unsigned)((per + 255) / 256)), dim3(256),
                   (const i64*)barrier + s * B, (const int*)flags, from, start, (i64)sync_cost, B, P);
        prof_count();
    }
    return EBSP_OK;
}

size_t ebsp_gridscan_workspace_bytes(int64_t B, int32_t P, int32_t R, int32_t full)
{
    if (B < 0 || P < 1 || R < 1 || (i64)P * R >= (1ll << 31)) return 0;
    return align_up((size_t)B * (full ? (size_t)P : 1) * sizeof(GridBest), 256);
}

int ebsp_gridscan_batch(const int64_t* ts, int64_t B, int32_t P, int32_t R, int32_t full,
                        int64_t* barrier, int32_t* iters, int64_t* dz, int32_t* status,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    if (B < 0 || P < 1 || R < 1 || (i64)P * R >= (1ll << 31))
        return fail(EBSP_ERR_SHAPE, "invalid shape: need B >= 0, P >= 1, R >= 1, P*R < 2^31");
    if (B == 0) return EBSP_OK;
    if (!ts || !barrier || !iters || !dz) return fail(EBSP_ERR_NULL, "ts, barrier, iters and dz must not be NULL");
    const i64 blocks = B * (full ? (i64)P : 1);
    if (blocks > 0x7fffffffll) return fail(EBSP_ERR_SHAPE, "batch too large for one call");
    if (!workspace) return fail(EBSP_ERR_NULL, "the scans need a workspace");
    if (workspace_bytes < ebsp_gridscan_workspace_bytes(B, P, R, full))
        return fail(EBSP_ERR_WORKSPACE, "workspace smaller than ebsp_gridscan_workspace_bytes()");
    if (((uintptr_t)workspace & 255u) != 0) return fail(EBSP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    if (int rc = check_device()) return rc;
    hipStream_t st = (hipStream_t)stream;
    GridBest* best = (GridBest*)workspace;
    i64 pieces = full ? P : 1;                       // results per instance, in (row, point) order
    if (R <= GRID_RMAX) {
        const i64 points = full ? (i64)P * R : R;
        int least = 1024, per_thread = 4;
        auto count = [&] {
            const i64 per = (i64)grid_point_threads(points, R, least, per_thread) * per_thread;
            return (points + per - 1) / per;         // no more than there are designated rows: a piece has R points or more
        };
        // Four consecutive points per thread, each search going on from the one before; one where the chip is not full and
        // rows are short: a chain of one search instead of four, and no wave whose threads pass the end of a row and search
        // anew.  Four / one, us: FullGridScan of 63 of 11 x 198 25.5 / 20.3, 2 of 233 x 119 98 / 54, 64 of 100 x 15 56 / 30;
        // GridScan of one of 185 x 15 32.0 / 19.7, one of 1000 x 150 206 / 185, one of 1000 x 240 234 / 245.
        if (R <= (full ? 256 : 192) && B * count() < 2 * GENERAL_GRID) per_thread = 1;
        // Pieces of 1024 points; smaller ones, whose threads share out the rows as well, where those would leave CUs idle.
        // FullGridScan with pieces of 1024 / 256, us: one of 497 x 113 719 / 200, one of 100 x 15 111 / 37, 8 of 46 x 61
        // 72 / 30 (128: the same); with a workgroup on every CU, 256 of 10 x 60 in pieces of 1024 / 512, 19.4 / 21.3.
        while (least > 256 && B * count() < GENERAL_GRID) least /= 2;
        pieces = count();
        // Workgroups of 1024 threads that would have no second row for a thread, and more of them than the chip takes at
        // once: as many threads as the points need, so that more share a CU.  1024 / 256 threads, us: 16384 of 4 x 15
        // 316 / 89, FullGridScan of them 350 / 105, 1024 of 10 x 15 27.4 / 19.7, 520 of 8 x 512 31.9 / 25.7; with more
        // rows 520 of 100 x 15 43.8 / 54.2, FullGridScan of 520 of 16 x 60 42.9 / 50.9.
        const int pthreads = grid_point_threads(points, R, least, per_thread);
        const bool small = B * pieces > 2 * GENERAL_GRID && (i64)pthreads * P <= 1024;
#define LAUNCH_GRIDSCAN(NT_, PER_)                                                                                        \
    LAUNCH(K_GRIDSCAN, (zl_gridscan_kernel<NT_, PER_>), dim3((unsigned)(B * pieces)), dim3(NT_), (const i64*)ts, P, R,   \
           full ? 1 : 0, (int)pieces, pthreads, best, status)
        if (full && per_thread == 4 && !small && R <= GRID_FULL_RMAX && P >= GRID_FULL_PMIN && P <= GRID_FULL_PMAX &&
            (P >= 128 || B * pieces > 3 * GENERAL_GRID))
            LAUNCH(K_GRIDSCAN, (zl_fullgridscan_kernel<1024, 4>), dim3((unsigned)(B * pieces)), dim3(1024), (const i64*)ts, P, R, (int)pieces,
                   pthreads, best, status);
        else if (per_thread == 1) LAUNCH_GRIDSCAN(1024, 1);
        else if (small && pthreads <= 256) LAUNCH_GRIDSCAN(256, 4);
        else if (small && pthreads <= 512) LAUNCH_GRIDSCAN(512, 4);
        else LAUNCH_GRIDSCAN(1024, 4);
#undef LAUNCH_GRIDSCAN
    } else
        LAUNCH(K_GRIDSCAN, zl_gridscan_long_kernel, dim3((unsigned)blocks), dim3(GRID_NT), (const i64*)ts, P, R, full ? 1 : 0, best, status);
    LAUNCH(K_GRIDSCAN_FINISH, zl_gridscan_finish_kernel, dim3((unsigned)B), dim3(GRID_NT), (const i64*)ts, P, R, (int)pieces,
           (const GridBest*)best, (i64*)barrier, iters, (i64*)dz);
    prof_count();
    return EBSP_OK;
}

size_t ebsp_zipline_range_workspace_bytes(int64_t B, int32_t P, int32_t R)
{
    Plan pl;
    if (!make_plan(B, P, R, pl, RANGE_SINGLE_MAX, true)) return 0;
    return pl.multi ? pl.bytes : 0;
}

int ebsp_zipline_range_batch(const int64_t* ts, int64_t B, int32_t P, int32_t R,
                             int64_t* barrier, int32_t* iters, int64_t* dmin,
                             int32_t* status, void* workspace, size_t workspace_bytes, void* stream)
{
    const int rc = run_range_batch((const i64*)ts, B, P, R, (i64*)barrier, iters, (i64*)dmin, status,
                                   workspace, workspace_bytes, (hipStream_t)stream);
    if (rc == EBSP_OK && B > 0) prof_count();
    return rc;
}

int ebsp_zipline_shape_info(int64_t B, int32_t P, int32_t R, int64_t* info)
{
    Plan pl;
    if (!info) return fail(EBSP_ERR_NULL, "info must not be NULL");
    if (!make_plan(B, P, R, pl)) return fail(EBSP_ERR_SHAPE, "invalid shape: need B >= 0, P >= 1, R >= 1, P*R < 2^31");
    info[0] = pl.multi ? 1 : 0;
    info[1] = pl.multi ? pl.cap : 0;
    info[2] = pl.multi ? pl.bins : 0;
    info[3] = pl.multi ? pl.max_win : 0;
    info[4] = pl.multi ? pl.fill : 0;
    Plan stored;
    info[5] = make_plan(B, P, R, stored, SINGLE_MAX, false, true) && stored.sweep ? stored.nslices : 0;
    return EBSP_OK;
}

int ebsp_zipline_tune(int32_t window_cap, int32_t single_max, int32_t window_fill)
{
    if (window_fill < 0 || (window_fill > 0 && window_fill < 512))
        return fail(EBSP_ERR_SHAPE, "window_fill must be 0 or at least 512");
    if (window_cap != 0 && window_cap != 4096 && window_cap != 8192 && window_cap != 16384)
        return fail(EBSP_ERR_SHAPE, "window_cap must be 0, 4096, 8192 or 16384");
    if (single_max < 0 || single_max > SINGLE_MAX)
        return fail(EBSP_ERR_SHAPE, "single_max must be in 0..16384");
    g_tune_window_cap.store(window_cap, std::memory_order_relaxed);
    g_tune_single_max.store(single_max, std::memory_order_relaxed);
    g_tune_window_fill.store(window_fill, std::memory_order_relaxed);
    return EBSP_OK;
}

int ebsp_zipline_tune_sweep(int32_t sweep_min, int32_t slice_keys, int32_t lines)
{
    if (lines < 0 || lines > SWEEP_LINES) return fail(EBSP_ERR_SHAPE, "lines must be in 0..4096");
    if (slice_keys < 0 || (slice_keys > 0 && slice_keys < 256)) return fail(EBSP_ERR_SHAPE, "slice_keys must be 0 or at least 256");
    g_tune_sweep_min.store(sweep_min, std::memory_order_relaxed);
    g_tune_sweep_lines.store(lines, std::memory_order_relaxed);
    g_tune_slice_keys.store(slice_keys, std::memory_order_relaxed);
    return EBSP_OK;
}

int ebsp_zipline_copy_probe(const void* src, void* dst, size_t bytes, void* stream)
{
    if (!src || !dst) return fail(EBSP_ERR_NULL, "src and dst must not be NULL");
    if (bytes == 0 || bytes % 16 != 0 || (((uintptr_t)src | (uintptr_t)dst) & 15u))
        return fail(EBSP_ERR_SHAPE, "copy probe needs a positive multiple of 16 bytes and 16-byte aligned pointers");
    if (int rc = check_device()) return rc;
    hipStream_t st = (hipStream_t)stream;
    const i64 n = (i64)(bytes / 16);
    i64 blocks = (n + 2047) / 2048;                     // pieces of 32 KiB or more
    if (blocks > 256 * 256) blocks = 256 * 256;
    LAUNCH(K_COPY, zl_copy_kernel, dim3((unsigned)blocks), dim3(256), (const uint4*)src, (uint4*)dst, n);
    prof_count();
    return EBSP_OK;
}

static_assert(READ_SINK_WORDS == EBSP_READ_SINK_WORDS, "the header's word count is the kernel's");

int ebsp_zipline_read_probe(const void* src, size_t bytes, uint64_t* sink, void* stream)
{
    if (!src || !sink) return fail(EBSP_ERR_NULL, "src and sink must not be NULL");
    if (bytes == 0 || bytes % 16 != 0 || ((uintptr_t)src & 15u) || ((uintptr_t)sink & 7u))
        return fail(EBSP_ERR_SHAPE, "read probe needs a positive multiple of 16 bytes, a 16-byte aligned source and an 8-byte aligned sink of 256 words");
    if (int rc = check_device()) return rc;
    hipStream_t st = (hipStream_t)stream;
    const i64 n = (i64)(bytes / 16);
    i64 blocks = (n + 2047) / 2048;                     // pieces of 32 KiB or more
    if (blocks > 256 * 256) blocks = 256 * 256;
    LAUNCH(K_READ, zl_read_kernel, dim3((unsigned)blocks), dim3(256), (const uint4*)src, n, (u64*)sink);
    prof_count();
    return EBSP_OK;
}

int ebsp_zipline_memory_info(int32_t* clock_khz, int32_t* bus_bits)
{
    if (!clock_khz || !bus_bits) return fail(EBSP_ERR_NULL, "clock_khz and bus_bits must not be NULL");
    int dev = 0, clk = 0, bus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(EBSP_ERR_DEVICE, "no current HIP device");
    if (hipDeviceGetAttribute(&clk, hipDeviceAttributeMemoryClockRate, dev) != hipSuccess ||
        hipDeviceGetAttribute(&bus, hipDeviceAttributeMemoryBusWidth, dev) != hipSuccess)
        return fail(EBSP_ERR_DEVICE, "hipDeviceGetAttribute failed");
    *clock_khz = clk;
    *bus_bits = bus;
    return EBSP_OK;
}

int ebsp_zipline_profile_begin(int32_t max_calls)
{
    if (g_prof.on) return fail(EBSP_ERR_SHAPE, "a profile is already open on this thread");
    if (max_calls < 1 || max_calls > 100000) return fail(EBSP_ERR_SHAPE, "max_calls must be in 1..100000");
    const size_t n = (size_t)max_calls * K_COUNT;
    g_prof.ev = new hipEvent_t[2 * n];
    g_prof.used = new bool[n]();
    g_prof.share = new float[max_calls]();
    for (size_t i = 0; i < 2 * n; ++i)
        if (hipEventCreate(&g_prof.ev[i]) != hipSuccess) {
            for (size_t k = 0; k < i; ++k) (void)hipEventDestroy(g_prof.ev[k]);
            delete[] g_prof.ev; delete[] g_prof.used; delete[] g_prof.share;
            g_prof = Profile();
            return fail(EBSP_ERR_LAUNCH, "hipEventCreate failed");
        }
    g_prof.max_calls = max_calls;
    g_prof.calls = 0;
    g_prof.on = true;
    return EBSP_OK;
}

int ebsp_zipline_profile_end(float* kernel_ms, int32_t* calls)
{
    if (!g_prof.on) return fail(EBSP_ERR_SHAPE, "no profile is open on this thread");
    int rc = EBSP_OK;
    if (hipDeviceSynchronize() != hipSuccess) rc = fail(EBSP_ERR_LAUNCH, "hipDeviceSynchronize failed");
    const size_t n = (size_t)g_prof.max_calls * K_COUNT;
    for (int k = 0; k < K_COUNT && kernel_ms; ++k) kernel_ms[k] = 0.f;
    if (rc == EBSP_OK && kernel_ms)
        for (int c = 0; c < g_prof.calls; ++c)
            for (int k = 0; k < K_COUNT; ++k)
                if (g_prof.used[c * K_COUNT + k]) {
                    float ms = 0.f;
                    const size_t i = ((size_t)c * K_COUNT + k) * 2;
                    if (hipEventElapsedTime(&ms, g_prof.ev[i], g_prof.ev[i + 1]) == hipSuccess) kernel_ms[k] += ms * g_prof.share[c];
                }
    if (calls) *calls = g_prof.calls;
    for (size_t i = 0; i < 2 * n; ++i) (void)hipEventDestroy(g_prof.ev[i]);
    delete[] g_prof.ev;
    delete[] g_prof.used;
    delete[] g_prof.share;
    g_prof = Profile();
    return rc;
}

int ebsp_zipline_kernel_count(void) { return K_COUNT; }

const char* ebsp_zipline_kernel_name(int i) { return (i >= 0 && i < K_COUNT) ? kKernelNames[i] : nullptr; }

const char* ebsp_last_error(void) { return g_err; }

}  // extern "C"
