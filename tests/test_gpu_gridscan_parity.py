"""GridScan / FullGridScan on the GPU (``ebsp_gridscan_batch``) against their CPU oracle, bit for bit: the
smallest max(Z) - min(Z) found, the barrier max(Z*) and the position of every worker's point in Z*
(Section IV, Algorithm 1 and the FullGridScan paragraph).  Needs an MI355X."""
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


def gpu_run(zl, ts, full):
    d = torch.from_numpy(np.ascontiguousarray(ts)).cuda()
    out = zl.ebsp_gridscan_batch(d, full)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


def assert_same(zl, oracle, ts, label, method="bisect"):
    for full in (False, True):
        bar, it, dz, st = gpu_run(zl, ts, full)
        ob, oi, od, rc, _ = oracle.gridscan(ts, full, method, threads=16)
        assert (rc == 0).all() and (st == 0).all(), label
        assert np.array_equal(dz, od), f"{label} full={full}: d_Z differs at {np.nonzero(dz != od)[0][:5]}"
        assert np.array_equal(bar, ob), f"{label} full={full}: barrier differs at {np.nonzero(bar != ob)[0][:5]}"
        assert np.array_equal(it, oi), f"{label} full={full}: Z* differs at {np.nonzero((it != oi).any(axis=1))[0][:5]}"


def test_hand_worked_examples(zl):
    path = os.path.join(os.path.dirname(__file__), "golden", "worked_examples_gridscan.json")
    for c in json.load(open(path))["cases"]:
        for full, key in ((False, "gridscan"), (True, "fullgridscan")):
            bar, it, dz, st = gpu_run(zl, np.array([c["t"]], dtype=np.int64), full)
            assert (int(dz[0]), int(bar[0]), list(it[0]), int(st[0])) == (c[key]["dz"], c[key]["barrier"], c[key]["iters"], 0), c["name"]


@pytest.mark.parametrize("P,R", [(1, 1), (1, 9), (6, 1), (2, 3), (3, 5), (7, 9), (13, 19), (33, 31), (64, 64), (17, 241),
                                 (300, 40), (5, 4096), (3, 5000), (2, 70001), (1100, 3)])
def test_shapes(zl, oracle, P, R):
    rng = np.random.default_rng(31 * P + R)
    ts = np.stack([workloads.random_small(rng, P, R, 1, 1000, ties=(i % 2 == 0)) for i in range(4)])
    small = P * R * R * P <= 4_000_000
    assert_same(zl, oracle, ts, f"P={P} R={R}", "scan" if small else "bisect")
    assert_same(zl, oracle, ts + EPOCH, f"P={P} R={R} shifted")
    assert_same(zl, oracle, ts - 5_000_000, f"P={P} R={R} negative")


@pytest.mark.parametrize("P,R,n", [(10, 15, 64), (10, 150, 32), (100, 15, 16), (100, 150, 8), (1000, 15, 4), (1000, 150, 2)])
def test_the_shapes_of_table_two(zl, oracle, P, R, n):
    assert_same(zl, oracle, workloads.make_workers(P, R, n), f"{P} workers, R={R}")


def test_configs(zl, oracle):
    assert_same(zl, oracle, workloads.make(1), "config 1", "scan")
    assert_same(zl, oracle, workloads.make(2, instances=range(256)), "config 2")
    assert_same(zl, oracle, workloads.make(3, instances=range(8)), "config 3")
    assert_same(zl, oracle, workloads.make(4, instances=range(1)), "config 4 (ties)")


def test_degenerate_and_extreme_values(zl, oracle):
    assert_same(zl, oracle, np.full((3, 8, 16), 42, dtype=np.int64), "all equal", "scan")
    rng = np.random.default_rng(17)
    base = np.stack([workloads.random_small(rng, 9, 33, 1, 1000, ties=True) for _ in range(3)])
    assert_same(zl, oracle, base + (1 << 62) - 40_000, "near the top of int64 / 2", "scan")
    assert_same(zl, oracle, base - (1 << 62), "near the bottom of int64 / 2", "scan")
    wide = base.copy()
    wide[:, ::2, :] += (1 << 61)                     # every other worker far away: the nearest point is a row's first or last
    assert_same(zl, oracle, wide, "two groups of workers 2^61 apart", "scan")
    far = np.sort(rng.integers(-(1 << 61), 1 << 61, size=(2, 5, 40)), axis=2)
    assert_same(zl, oracle, far, "values all over +-2^61", "scan")


def test_empty_batch_and_buffers_passed_in(zl, oracle):
    empty = torch.zeros((0, 4, 8), dtype=torch.int64, device="cuda")
    out = zl.ebsp_gridscan_batch(empty, True)
    torch.cuda.synchronize()
    assert [tuple(t.shape) for t in out] == [(0,), (0, 4), (0,), (0,)]
    ts = workloads.make_workers(12, 30, 5)
    d = torch.from_numpy(ts).cuda()
    bufs = (torch.full((5,), -1, dtype=torch.int64, device="cuda"), torch.full((5, 12), -1, dtype=torch.int32, device="cuda"),
            torch.full((5,), -1, dtype=torch.int64, device="cuda"), torch.full((5,), -1, dtype=torch.int32, device="cuda"))
    ws = torch.empty(zl.ebsp_gridscan_workspace_bytes(5, 12, 30, True), dtype=torch.uint8, device="cuda")
    got = zl.ebsp_gridscan_batch(d, True, *bufs, workspace=ws)
    torch.cuda.synchronize()
    assert all(a is b for a, b in zip(got, bufs))
    ob, oi, od, rc, _ = oracle.gridscan(ts, True, "scan")
    assert np.array_equal(bufs[0].cpu().numpy(), ob) and np.array_equal(bufs[1].cpu().numpy(), oi)
    assert np.array_equal(bufs[2].cpu().numpy(), od) and (bufs[3].cpu().numpy() == 0).all()
    with pytest.raises(ValueError):
        zl.ebsp_gridscan_batch(d, True, bufs[0].to(torch.int32))
    with pytest.raises(ValueError):
        zl.ebsp_gridscan_batch(d, True, workspace=ws[:ws.numel() - 256])


def test_never_below_the_exact_search(zl):
    # both scans build sets of one timestamp per worker: ebsp_zipline_range_batch's optimum bounds them from below
    ts = torch.from_numpy(workloads.make(2, instances=range(512))).cuda()
    exact = zl.ebsp_zipline_range_batch(ts)[2]
    heur = zl.ebsp_gridscan_batch(ts, False)[2]
    full = zl.ebsp_gridscan_batch(ts, True)[2]
    torch.cuda.synchronize()
    assert bool((full >= exact).all()) and bool((heur >= full).all())


def test_unsorted_row_is_flagged(zl):
    rng = np.random.default_rng(5)
    ts = np.stack([workloads.random_small(rng, 12, 80, 1, 100) for _ in range(4)])
    ts[1, 3, 40] = ts[1, 3, 39] - 1
    for full in (False, True):
        st = gpu_run(zl, ts, full)[3]
        assert st[1] == zl.STATUS_UNSORTED and (np.delete(st, 1) == 0).all()


def test_argument_errors(zl):
    lib = zl.load()
    ts = torch.zeros((1, 2, 2), dtype=torch.int64, device="cuda")
    assert lib.ebsp_gridscan_batch(ts.data_ptr(), 1, 0, 2, 0, ts.data_ptr(), ts.data_ptr(), ts.data_ptr(), None, None, 0, None) == -2
    assert lib.ebsp_gridscan_batch(None, 1, 2, 2, 0, ts.data_ptr(), ts.data_ptr(), ts.data_ptr(), None, None, 0, None) == -1
    assert lib.ebsp_gridscan_batch(ts.data_ptr(), 1, 2, 2, 1, ts.data_ptr(), ts.data_ptr(), ts.data_ptr(), None, ts.data_ptr(), 0, None) == -3
    assert zl.ebsp_gridscan_workspace_bytes(4, 100, 15, True) >= 4 * 100 * 16 and zl.ebsp_gridscan_workspace_bytes(4, 0, 15, True) == 0


@pytest.mark.parametrize("P,R", [(8, 128), (9, 128), (1, 1023), (3, 1025), (2, 2049), (3, 4096), (41, 100), (60, 257)])
@pytest.mark.parametrize("scale", [1, 1 << 22])
def test_pieces_and_batches(zl, oracle, P, R, scale):
    """Points at the edges of the workgroups' pieces, rows of more than one staging, values of 32 and 64 bits."""
    rng = np.random.default_rng(77 * P + R)
    ts = np.stack([workloads.random_small(rng, P, R, 1, 5000, ties=(i == 0)) for i in range(3)]) * scale
    assert_same(zl, oracle, ts + EPOCH, f"P={P} R={R} scale={scale}")


@pytest.mark.parametrize("P,R", [(1, 1), (2, 4), (4, 15), (8, 128), (9, 128), (16, 60), (4, 1024), (2, 1025), (2, 2048), (1, 2049)])
@pytest.mark.parametrize("scale", [1, 1 << 22])
def test_batches_of_more_workgroups_than_the_chip_takes(zl, oracle, P, R, scale):
    """Workgroups of 256, 512 and 1024 threads, at the largest rows and points of each; values of 32 and 64 bits."""
    rng = np.random.default_rng(91 * P + R)
    ts = np.cumsum(rng.integers(0, 2000, size=(513, P, R)), axis=2) + rng.integers(0, 2000, size=(513, P, 1))
    assert_same(zl, oracle, ts * scale + EPOCH, f"P={P} R={R} scale={scale}")


# FullGridScan of many rows, most points ruled out by a few of them (512 workgroups of 1024 points or more): rows that all
# continue, that end and begin at very different times, that are alike (too many points left), values beyond 32 bits
@pytest.mark.parametrize("B,P,R", [(64, 96, 90), (60, 100, 151), (37, 129, 130), (40, 97, 512), (200, 96, 33)])
def test_full_scan_of_many_rows(zl, oracle, B, P, R):
    rng = np.random.default_rng(P * R)
    mean = rng.integers(20_000, 200_000, size=(B, P, 1))
    d = rng.integers(80, 121, size=(B, P, R)) * (mean // 100)
    spread = np.cumsum(d, axis=2) + (rng.random((B, P, 1)) * mean).astype(np.int64)
    alike = np.arange(R) * 1000 + rng.integers(0, 900, size=(B, P, R))
    late = spread + (rng.random((B, P, 1)) < 0.05) * int(spread.max() // 2)
    for label, ts in (("spread", spread), ("ties", spread // 5000 * 5000), ("alike", alike), ("late", late), ("wide", spread * 100_003),
                      ("one value", np.zeros_like(spread))):
        ts = np.ascontiguousarray(ts + EPOCH)
        bar, it, dz, st = gpu_run(zl, ts, True)
        ob, oi, od, rc, _ = oracle.gridscan(ts, True, "bisect", threads=16)
        assert (rc == 0).all() and (st == 0).all(), label
        assert np.array_equal(dz, od) and np.array_equal(bar, ob) and np.array_equal(it, oi), label
    spread[5, 7, R - 1] = spread[5, 7, R - 2] - 1
    assert gpu_run(zl, spread, True)[3].tolist() == [1 if b == 5 else 0 for b in range(B)]


# the edges of its rule: the fewest rows, the longest ones, the most, small batches that do not take it, and of all of them a few rows
# much longer than the others, which rule points out, and as many as still do
@pytest.mark.parametrize("B,P,R", [(100, 96, 90), (60, 100, 151), (34, 127, 256), (20, 128, 255), (12, 511, 100), (13, 512, 97), (30, 100, 180), (12, 513, 100)])
@pytest.mark.parametrize("slow", [5, 51, 60])
def test_full_scan_of_rows_a_few_of_which_are_long(zl, oracle, B, P, R, slow):
    rng = np.random.default_rng(P * R + slow)
    mean = rng.integers(90_000, 110_000, size=(B, P, 1))
    mean[np.argsort(rng.random((B, P)), axis=1) < slow] *= 2
    ts = np.cumsum(rng.integers(90, 111, size=(B, P, R)) * (mean // 100), axis=2) + (rng.random((B, P, 1)) * mean).astype(np.int64)
    ts[B // 2:] *= 50_021                                                    # values beyond 32 bits
    ts = np.ascontiguousarray(ts + EPOCH)
    bar, it, dz, st = gpu_run(zl, ts, True)
    ob, oi, od, rc, _ = oracle.gridscan(ts, True, "bisect", threads=16)
    assert (rc == 0).all() and (st == 0).all()
    assert np.array_equal(dz, od) and np.array_equal(bar, ob) and np.array_equal(it, oi)
