"""Parity of the HIP path with the CPU oracle for the paper's formal objective
d_Z = max(Z) - min(Z) (``ebsp_zipline_range_batch``), through the C ABI (needs an MI355X).

Bar: bit-exact on barrier (int64), dmin (int64) and iters (int32); the result is unique
(first minimum), also for instances whose value spread does not fit 32 bits.
"""
import json
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2001_01347_amd import workloads  # noqa: E402

EPOCH = 1_700_000_000_000_000


@pytest.fixture(scope="module")
def zl():
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2001_01347_amd import zipline
    zipline.load()
    return zipline


def gpu_run(zl, ts):
    d = torch.from_numpy(np.ascontiguousarray(ts)).cuda()
    bar, it, dm, st = zl.ebsp_zipline_range_batch(d)
    torch.cuda.synchronize()
    return bar.cpu().numpy(), it.cpu().numpy(), dm.cpu().numpy(), st.cpu().numpy()


def assert_same(zl, oracle, ts, label=""):
    bar, it, dm, st = gpu_run(zl, ts)
    ob, oi, od, rc, _ = oracle.zipline_range(ts, "sweep", threads=16)
    assert (rc == 0).all()
    assert (st == 0).all(), f"{label}: status {np.unique(st)}"
    assert np.array_equal(dm, od), f"{label}: dmin differs at {np.nonzero(dm != od)[0][:5]}"
    assert np.array_equal(bar, ob), f"{label}: barrier differs at {np.nonzero(bar != ob)[0][:5]}"
    assert np.array_equal(it, oi), f"{label}: iters differ at {np.nonzero((it != oi).any(axis=1))[0][:5]}"


def test_hand_worked_examples(zl):
    path = os.path.join(os.path.dirname(__file__), "golden", "worked_examples_range.json")
    for c in json.load(open(path))["cases"]:
        bar, it, dm, st = gpu_run(zl, np.array([c["t"]], dtype=np.int64))
        assert (int(bar[0]), int(dm[0]), list(it[0]), int(st[0])) == (c["barrier"], c["dmin"], c["iters"], 0), c["name"]


def test_config1_and_config2_full(zl, oracle):
    assert_same(zl, oracle, workloads.make(1), "config 1")
    assert_same(zl, oracle, workloads.make(2), "config 2")
    assert_same(zl, oracle, workloads.make(2, instances=range(64)) + EPOCH, "config 2 shifted")


@pytest.mark.parametrize("P,R", [(1, 1), (1, 9), (6, 1), (2, 3), (3, 5), (7, 9), (4, 16), (13, 19), (64, 64),
                                 (8, 1024), (8192, 1), (100, 81), (16, 64), (1, 1024), (1025, 1), (30, 60), (2, 1024),
                                 (2049, 1), (33, 100), (64, 64), (4097, 1), (90, 90)])
def test_single_workgroup_shapes(zl, oracle, P, R):
    rng = np.random.default_rng(1000 * P + R)
    ts = np.stack([workloads.random_small(rng, P, R, 1, 1000, ties=(i % 2 == 0)) for i in range(6)])
    assert_same(zl, oracle, ts, f"P={P} R={R}")
    assert_same(zl, oracle, ts * 1000 + EPOCH, f"P={P} R={R} scaled and shifted")


@pytest.mark.parametrize("P,R", [(1, 8193), (8193, 1), (64, 257), (5, 4000), (300, 100), (128, 512), (1100, 40)])
def test_multi_window_shapes(zl, oracle, P, R):
    rng = np.random.default_rng(77 * P + R)
    ts = np.stack([workloads.random_small(rng, P, R, 1, 1000, ties=(i % 2 == 0)) for i in range(3)])
    assert_same(zl, oracle, ts * 1000 + EPOCH, f"P={P} R={R}")


@pytest.mark.parametrize("P,R", [(8, 1024), (16, 4096), (600, 64)])
def test_equal_minima_far_apart(zl, oracle, P, R):
    # staggered workers of one period: d = (P-1)*g at every time once all have started;
    # worker 0 joins k periods late, so the first admissible time wins
    g, k = 7, R // 3
    T = P * g
    i = np.arange(R, dtype=np.int64)
    t = np.stack([p * g + i * T for p in range(P)])
    t[0] = (i + k) * T
    ts = np.stack([t, t + 3 + EPOCH])
    bar, it, dm, st = gpu_run(zl, ts)
    assert (st == 0).all()
    assert list(bar) == [k * T, k * T + 3 + EPOCH] and list(dm) == [(P - 1) * g] * 2
    assert_same(zl, oracle, ts, f"staggered P={P} R={R}")


def test_configs_3_to_5_samples(zl, oracle):
    assert_same(zl, oracle, workloads.make(3, instances=range(96)), "config 3 sample")
    assert_same(zl, oracle, workloads.make(4, instances=range(6)), "config 4 sample")
    assert_same(zl, oracle, workloads.make(5, instances=range(2)), "config 5 sample")
    assert_same(zl, oracle, workloads.make(4, instances=range(2)) + EPOCH, "config 4 shifted")


def test_skew_and_ties(zl, oracle):
    t = workloads.make(4, instances=range(2)).copy()
    t[:, 7, :] = t[:, 7, :1] + (t[:, 7, :] - t[:, 7, :1]) * 20        # one worker 20x slower
    assert_same(zl, oracle, t, "straggler x20")
    assert_same(zl, oracle, np.full((3, 8, 16), 42, dtype=np.int64), "all equal")
    assert_same(zl, oracle, np.full((2, 64, 512), -7, dtype=np.int64), "all equal, more than a workgroup holds")
    rng = np.random.default_rng(12)
    few = np.sort(rng.integers(0, 4, size=(2, 64, 1024)), axis=2).astype(np.int64) * 1_000_003
    assert_same(zl, oracle, few, "four distinct values")
    c = np.sort(rng.integers(0, 50_000, size=(1, 40, 1000)), axis=2).astype(np.int64)
    c[0, 0, -1] = 10 ** 9
    assert_same(zl, oracle, c, "cluster and outlier")
    row = np.cumsum(np.arange(1, 301, dtype=np.int64))
    assert_same(zl, oracle, np.tile(row, (2, 20, 1)), "identical workers")


def test_status_flags(zl, oracle):
    ts = workloads.make(2, instances=range(8)).copy()
    ts[3, 5, 10] = ts[3, 5, 9] - 1                      # one row of one instance goes backwards
    bar, it, dm, st = gpu_run(zl, ts)
    assert st[3] & zl.STATUS_UNSORTED and (np.delete(st, 3) == 0).all()
    ob, oi, od, rc, _ = oracle.zipline_range(np.delete(ts, 3, axis=0), "sweep", threads=8)
    assert np.array_equal(np.delete(bar, 3), ob) and np.array_equal(np.delete(dm, 3), od)
    # a spread of 2^32 or more is no reason for a flag
    wide = workloads.make(2, instances=range(4)).copy()
    wide[2] *= 1 << 20
    bar, it, dm, st = gpu_run(zl, wide)
    assert (st == 0).all()
    ms = workloads.make(3, instances=range(4)).copy()
    ms[1, 9, 100] = ms[1, 9, 99] - 5
    bar, it, dm, st = gpu_run(zl, ms)
    assert st[1] & zl.STATUS_UNSORTED and (np.delete(st, 1) == 0).all()


def _properties_hold(ts, bar, it, dm):
    """Checks that hold at any size (torch, on the GPU): each worker stops at its last timestamp
    <= barrier, the barrier is some worker's stop, and dmin is the barrier minus the earliest stop."""
    B, P, R = ts.shape
    assert int(it.min()) >= 1 and int(it.max()) <= R
    idx = (it.long() - 1).unsqueeze(-1)
    stop = torch.gather(ts, 2, idx).squeeze(-1)                        # [B, P]
    assert bool((stop <= bar.unsqueeze(-1)).all())
    nxt = torch.gather(ts, 2, torch.clamp(idx + 1, max=R - 1)).squeeze(-1)
    beyond = (it.long() == R) | (nxt > bar.unsqueeze(-1))
    assert bool(beyond.all())
    assert bool((stop.max(dim=1).values == bar).all())
    assert bool((bar - stop.min(dim=1).values == dm).all())
    first_all = ts[:, :, 0].max(dim=1).values
    assert bool((bar >= first_all).all())
    # never worse than the classic barrier after one iteration of every worker
    lag = torch.searchsorted(ts.contiguous(), first_all.view(B, 1, 1).expand(B, P, 1).contiguous(), right=True).squeeze(-1)
    classic = first_all - torch.gather(ts, 2, (lag - 1).unsqueeze(-1)).squeeze(-1).min(dim=1).values
    assert bool((dm <= classic).all())


@pytest.mark.parametrize("k", [3, 4, 5])
def test_full_size_configs(zl, oracle, k):
    # every instance of the 2 GiB configurations against the oracle
    host = workloads.make(k, threads=16)
    ts = torch.from_numpy(host).cuda()
    bar, it, dm, st = zl.ebsp_zipline_range_batch(ts)
    torch.cuda.synchronize()
    assert int(st.max().item()) == 0
    _properties_hold(ts, bar, it, dm)
    ob, oi, od, rc, _ = oracle.zipline_range(host, "sweep", threads=16)
    assert (rc == 0).all()
    assert np.array_equal(bar.cpu().numpy(), ob), f"barrier differs at {np.nonzero(bar.cpu().numpy() != ob)[0][:5]}"
    assert np.array_equal(dm.cpu().numpy(), od), f"dmin differs at {np.nonzero(dm.cpu().numpy() != od)[0][:5]}"
    assert np.array_equal(it.cpu().numpy(), oi)


def test_value_spread_beyond_32_bits(zl, oracle):
    # keys, successors and the distance back to a worker's previous value no longer fit 32 bits:
    # one workgroup per instance (config 2), windows (configs 3 to 5), a mix of both kinds in one batch
    assert_same(zl, oracle, workloads.make(2, instances=range(64)) * 1000 + EPOCH, "config 2 in ns")
    mixed = workloads.make(2, instances=range(16)).copy()
    mixed[::2] *= 1 << 20
    assert_same(zl, oracle, mixed, "config 2, every other instance x 2^20")
    assert_same(zl, oracle, workloads.make(3, instances=range(6)) * 1000, "config 3 in ns")
    assert_same(zl, oracle, workloads.make(4, instances=range(2)) * 1000, "config 4 in ns")
    assert_same(zl, oracle, workloads.make(5, instances=[0]) * 1000, "config 5 in ns")
    rng = np.random.default_rng(5)
    # every waiting time itself is beyond 2^32: two to five workers with iteration times near 2^33
    for P, R in ((2, 3), (3, 40), (5, 700), (2, 5000)):
        steps = rng.integers(2 ** 33, 2 ** 33 + 2 ** 31, size=(7, P, R), dtype=np.int64)
        assert_same(zl, oracle, np.cumsum(steps, axis=2), f"steps near 2^33, P={P} R={R}")
    # dense stretches far apart: most pieces of 2^32 are empty, some hold more than a workgroup takes
    for P, R in ((8, 600), (64, 512), (300, 100)):
        steps = rng.integers(1, 50, size=(3, P, R), dtype=np.int64)
        steps[:, :, R // 3] += 2 ** 40
        steps[:, :, 2 * R // 3] += 2 ** 34
        steps[:, ::3, R // 2] += 2 ** 36
        assert_same(zl, oracle, np.cumsum(steps, axis=2) - 2 ** 41, f"clusters far apart, P={P} R={R}")
    # the widest values the precondition allows for two workers
    big = np.array([[[0, 2 ** 61, 2 ** 62 - 1], [5, 2 ** 61 + 7, 2 ** 62 - 3]]], dtype=np.int64)
    assert_same(zl, oracle, big, "values up to 2^62")
    assert_same(zl, oracle, big - 2 ** 61, "values from -2^61")


def _steps(rng, B, P, R, spread):
    mean = rng.uniform(80, 120, size=(B, P, 1)) * spread
    steps = np.maximum(1, np.rint(mean * rng.lognormal(0, 0.15, size=(B, P, R)))).astype(np.int64)
    return np.cumsum(steps, axis=2) + rng.integers(0, 100 * spread, size=(B, P, 1))


# (B, P, R): one wave and two, items that end inside a wave and rows that end inside an item, the last entries of the
# register form and the first of the slices, of one slice and several, fewer lanes than a wave per row, rows one longer
# than a wave's step, more rows than threads, rows too long for the register form, rows that end long before the others
@pytest.mark.parametrize("B,P,R", [(9, 4, 64), (9, 5, 51), (9, 4, 65), (9, 16, 64), (9, 4, 256), (9, 3, 257), (9, 8, 128), (5, 8, 512),
                                   (5, 7, 513), (5, 64, 64), (5, 241, 17), (3, 63, 130), (3, 64, 256), (600, 33, 300), (3, 130, 127),
                                   (2, 520, 33), (1, 1030, 40), (3, 20, 3000), (1, 3, 9000), (1, 7, 5000)])
@pytest.mark.parametrize("spread", [10, 1000, 3_000_000])
def test_edges_of_the_search_by_successors(zl, oracle, B, P, R, spread):
    # spreads below 2^31, and (where rows are long) between 2^31 and 2^32 or beyond 2^32
    rng = np.random.default_rng(B + 31 * P + R + spread)
    ts = _steps(rng, B, P, R, spread)
    assert_same(zl, oracle, ts + EPOCH, f"B={B} P={P} R={R} spread {spread}")
    ts[:, ::3] = ts[:, ::3, :1] + (ts[:, ::3] - ts[:, ::3, :1]) // 7      # every third worker is through early: lim is small
    assert_same(zl, oracle, ts, f"B={B} P={P} R={R} spread {spread}, some workers through early")
    ts -= ts % (20 * spread)                                              # ties between workers and inside rows
    assert_same(zl, oracle, ts, f"B={B} P={P} R={R} spread {spread}, ties")


# values that cells do not resolve: more entries in a cell than its list holds, in more cells than may wait (520 x 150);
# more candidates than are tried in registers (20 x 150); intervals cut again and again
@pytest.mark.parametrize("B,P,R", [(520, 520, 150), (7, 20, 150), (3, 100, 30), (2, 700, 60), (1, 300, 400)])
def test_clusters_that_cells_do_not_resolve(zl, oracle, B, P, R):
    rng = np.random.default_rng(B + P)
    ts = np.arange(R, dtype=np.int64)[None, None, :] * 1_000_000_007 + rng.integers(0, 900, size=(B, P, R))
    assert_same(zl, oracle, ts, f"an iteration of every worker at a time, P={P} R={R}")
    near = rng.integers(0, 40, size=(min(B, 8), P, R), dtype=np.int64).cumsum(axis=2)
    near[:, :, R // 2:] += 1 << 40
    assert_same(zl, oracle, near, f"two dense stretches, P={P} R={R}")


@pytest.mark.parametrize("B,P,R", [(3, 16, 60), (3, 60, 60), (3, 30, 600), (520, 30, 600), (1, 700, 90)])
def test_rows_out_of_order_anywhere(zl, oracle, B, P, R):
    # one step back, at the start, in the middle, at the end and behind the earliest end of the rows, small and large
    rng = np.random.default_rng(P * R)
    ts = _steps(rng, B, P, R, 1000)
    ts[:, 1] = ts[:, 1, :1] + (ts[:, 1] - ts[:, 1, :1]) // 4              # through early
    for k, i in enumerate((1, R // 2, R - 1, R - 2, R // 3)):
        bad = ts.copy()
        p = P - 1 if k % 2 else P // 2
        bad[0, p, i] = bad[0, p, i - 1] - (1 if k < 3 else 50_000_000)
        st = gpu_run(zl, bad)[3]
        assert st[0] & zl.STATUS_UNSORTED and (st[1:] == 0).all(), (k, i)


# the answer is the earliest end of the rows, alone in a cell that begins there: that cell's two bounds are one value.  One
# iteration of all workers at a time, equally far apart but for the last; the ends lie 1 apart from instance to
# instance, or where cells of 2^shift values begin.  Workgroups of 256 and 512 threads, one slice and several, all numbers
# of cells, small instances
@pytest.mark.parametrize("B,P,R,ends", [(1100, 300, 30, 2_899_500), (64, 300, 30, 250_000), (300, 1100, 40, 3_900_000), (600, 300, 300, 16 * 2048 * 100),
                                        (64, 40, 30, 200_000), (64, 16, 30, 6000), (4, 300, 30, 2832 << 33), (4, 40, 30, 2832 << 33), (4, 40, 30, 2832 << 15)])
def test_the_answer_is_the_earliest_end(zl, oracle, B, P, R, ends):
    rng = np.random.default_rng(B + P + R)
    lim = ends + np.arange(B, dtype=np.int64) if ends < 1 << 25 else ends * (1 + np.arange(B, dtype=np.int64) % 2)
    period = lim // (R - 1)
    apart = np.minimum(period // 20, 1 << 30)
    ts = np.arange(R, dtype=np.int64) * period[:, None, None] + (rng.random((B, P, R)) * apart[:, None, None]).astype(np.int64)
    ts[:, 1, :] = np.arange(R, dtype=np.int64) * period[:, None]
    ts[:, 2, :] = ts[:, 1, :] + apart[:, None]
    ts[:, :, -1] = lim[:, None] + (rng.random((B, P)) * (apart - 4)[:, None]).astype(np.int64) + 1
    ts[:, 1, -1] = lim
    ts[:, 2, -1] = lim + apart - 3                         # (less than a cell is wide: others' lower bounds are smaller)
    assert_same(zl, oracle, ts, f"B={B} P={P} R={R}")


# workers in step, whose cells are given up, and one step back, anywhere and of any size, in every instance: the sort-based
# search that takes over cuts such rows into pieces by value and may never see it.  Instances in slices, in registers
@pytest.mark.parametrize("B,P,R,unit", [(64, 520, 1000, 0), (64, 520, 1000, 24), (64, 1030, 1000, 30), (64, 100, 40, 30)])
@pytest.mark.parametrize("apart", [0, 20])
def test_rows_out_of_order_where_cells_are_given_up(zl, B, P, R, unit, apart):
    rng = np.random.default_rng(5)
    ts = np.arange(R, dtype=np.int64) * (100_000 << unit) + (rng.random((B, P, R)) * (apart << unit)).astype(np.int64)
    back = [1, 100, 1 << 30, 1 << 36, 1 << 40, 1 << 45] if unit else [1, 10, 100_000, 5_000_000, 50_000_000]
    for b in range(B):
        p, i = int(rng.integers(P)), int(rng.integers(1, R - 1))
        ts[b, p, i] = ts[b, p, i - 1] - back[b % len(back)]
    st = gpu_run(zl, ts)[3]
    assert (st == zl.STATUS_UNSORTED).all(), np.nonzero(st != zl.STATUS_UNSORTED)[0]


# workers in step: more entries of a round in one cell than its list holds, which the cell's first entry settles; two
# iterations in quick succession, where it does not and the cells are cut further, few of them or (more than a level keeps)
# in pieces; three in a row with a pause of their own, where that repeats.  Several slices and one, workgroups of 256 and 512
# threads, narrow and wide values
@pytest.mark.parametrize("unit", [0, 33])
@pytest.mark.parametrize("B,P,R", [(64, 300, 400), (600, 300, 240), (1100, 300, 60), (4, 1100, 300), (16, 600, 24)])
def test_workers_in_step(zl, oracle, B, P, R, unit):
    rng = np.random.default_rng(B + P + R)
    round_ = np.arange(R, dtype=np.int64) * 100_000
    pairs = np.arange(R, dtype=np.int64) // 2 * 100_000 + np.arange(R, dtype=np.int64) % 2 * 40
    triples = np.arange(R, dtype=np.int64) // 3 * 100_000 + np.arange(R, dtype=np.int64) % 3 ** 2 // 3 * 30 + np.arange(R, dtype=np.int64) % 3
    for steps in (round_, pairs, triples):
        for apart in (1, 30, 1000):
            ts = steps + rng.integers(0, apart, size=(B, P, R))
            ts = np.sort(ts, axis=2) << unit
            if unit:
                ts += np.sort(rng.integers(0, 1 << unit, size=(B, P, R)), axis=2)
            assert_same(zl, oracle, np.sort(ts, axis=2), f"B={B} P={P} R={R} apart={apart}")
