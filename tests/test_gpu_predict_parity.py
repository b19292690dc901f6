"""Parity of ``ebsp_predict_zipline_batch`` (prediction folded into the search: rows
``last_end + (i + 1) * interval`` that are never stored) with the CPU oracle run on the rows
written out, through the C ABI (needs an MI355X).  Bar: bit-exact on all three outputs.
"""
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


def gpu_run(zl, le, iv, R):
    out = zl.ebsp_predict_zipline_batch(torch.from_numpy(np.ascontiguousarray(le)).cuda(),
                                        torch.from_numpy(np.ascontiguousarray(iv)).cuda(), R)
    torch.cuda.synchronize()
    return tuple(x.cpu().numpy() for x in out)


def assert_same(zl, oracle, le, iv, R, label=""):
    bar, it, w, st = gpu_run(zl, le, iv, R)
    ob, oi, ow, rc, _ = oracle.zipline(oracle.predicted_rows(le, iv, R), "sweep", threads=16)
    assert (rc == 0).all()
    assert (st == 0).all(), f"{label}: status {np.unique(st)}"
    assert np.array_equal(w, ow), f"{label}: wait differs at {np.nonzero(w != ow)[0][:5]}"
    assert np.array_equal(bar, ob), f"{label}: barrier differs at {np.nonzero(bar != ob)[0][:5]}"
    assert np.array_equal(it, oi), f"{label}: iters differ at {np.nonzero((it != oi).any(axis=1))[0][:5]}"


def random_inputs(rng, n, P, lo, hi, ties):
    iv = rng.integers(lo, hi + 1, size=(n, P)).astype(np.int64)
    if ties:
        iv = (iv // 10 + 1) * 10
    le = rng.integers(0, hi, size=(n, P)).astype(np.int64)
    if ties:
        le = le // 10 * 10
    return le, iv


@pytest.mark.parametrize("P,R", [(1, 1), (1, 9), (6, 1), (2, 3), (3, 5), (7, 9), (4, 16), (13, 19), (16, 64),
                                 (64, 64), (64, 256), (100, 163)])
def test_single_workgroup_shapes(zl, oracle, P, R):
    rng = np.random.default_rng(1000 * P + R)
    for ties in (False, True):
        le, iv = random_inputs(rng, 6, P, 1, 1000, ties)
        assert_same(zl, oracle, le, iv, R, f"P={P} R={R} ties={ties}")
        assert_same(zl, oracle, le + EPOCH, iv, R, f"P={P} R={R} shifted")


@pytest.mark.parametrize("P,R", [(1, 16385), (16385, 1), (64, 257), (5, 4000), (300, 100), (128, 512),
                                 (1100, 40), (1024, 64)])
def test_multi_window_shapes(zl, oracle, P, R):
    rng = np.random.default_rng(77 * P + R)
    for ties in (False, True):
        le, iv = random_inputs(rng, 3, P, 1, 1000, ties)
        assert_same(zl, oracle, le + EPOCH, iv, R, f"P={P} R={R} ties={ties}")
        assert_same(zl, oracle, le, iv, R, f"P={P} R={R} ties={ties}, small epoch")
        assert_same(zl, oracle, le - EPOCH, iv, R, f"P={P} R={R} ties={ties}, negative epoch")


def test_all_configurations(zl, oracle):
    for k, ids in ((1, None), (2, range(256)), (3, range(64)), (4, range(6)), (5, range(2))):
        le, iv = workloads.make_predicted(k, instances=ids, shift=EPOCH)
        assert_same(zl, oracle, le, iv, workloads.CONFIGS[k].R, f"config {k}")


def test_same_as_the_stored_path(zl, oracle):
    # the stored-rows entry point on the rows written out must give the very same outputs
    for k, ids in ((2, range(128)), (4, range(4))):
        le, iv = workloads.make_predicted(k, instances=ids)
        R = workloads.CONFIGS[k].R
        bar, it, w, st = gpu_run(zl, le, iv, R)
        ts = torch.from_numpy(oracle.predicted_rows(le, iv, R)).cuda()
        sb, si, sw, ss = zl.ebsp_zipline_batch(ts)
        torch.cuda.synchronize()
        assert np.array_equal(bar, sb.cpu().numpy()) and np.array_equal(w, sw.cpu().numpy())
        assert np.array_equal(it, si.cpu().numpy()) and (st == 0).all()


def test_degenerate_and_wide_inputs(zl, oracle):
    rng = np.random.default_rng(5)
    # zero intervals (all timestamps of a worker equal), identical workers, one very slow worker
    le, iv = random_inputs(rng, 4, 20, 1, 500, False)
    iv[:, ::3] = 0
    assert_same(zl, oracle, le, iv, 40, "zero intervals")
    assert_same(zl, oracle, np.full((2, 64), 7, dtype=np.int64), np.full((2, 64), 13, dtype=np.int64), 512, "identical workers")
    le, iv = random_inputs(rng, 2, 300, 100, 1000, False)
    iv[:, 5] *= 1000
    assert_same(zl, oracle, le, iv, 100, "one worker 1000x slower")
    # spreads of 2^32 and more (nanosecond units): the general search
    le, iv = random_inputs(rng, 3, 16, 1, 1000, True)
    assert_same(zl, oracle, le * 100_000_007, iv * 100_000_007, 64, "wide, single workgroup")
    le, iv = random_inputs(rng, 2, 128, 1, 1000, False)
    assert_same(zl, oracle, le * 100_000_007 + EPOCH, iv * 100_000_007, 512, "wide, multi-window")


@pytest.mark.parametrize("P,R", [(40, 26), (2, 1000), (6, 2000), (61, 241), (3, 5461)])
def test_wide_single_workgroup_instances(zl, oracle, P, R):
    # spreads around 2^35 in one workgroup: the bucket search of whole values, in one round and (few workers) in several
    rng = np.random.default_rng(P * R)
    le, iv = random_inputs(rng, 5, P, 50, 1000, False)
    iv[3] = 777                                            # every worker alike
    scale = (1 << 34) // (400 * R) + 7
    assert_same(zl, oracle, le * scale + EPOCH, iv * scale, R, f"P={P} R={R}")


def test_negative_interval_is_flagged(zl, oracle):
    for P, R in ((16, 64), (128, 512)):
        rng = np.random.default_rng(P)
        le, iv = random_inputs(rng, 6, P, 1, 1000, False)
        iv[2, 3] = -5
        bar, it, w, st = gpu_run(zl, le, iv, R)
        assert st[2] & zl.STATUS_UNSORTED and (np.delete(st, 2) == 0).all()
        keep = np.delete(np.arange(6), 2)
        ob, oi, ow, rc, _ = oracle.zipline(oracle.predicted_rows(le[keep], iv[keep], R), "sweep", threads=8)
        assert np.array_equal(bar[keep], ob) and np.array_equal(w[keep], ow) and np.array_equal(it[keep], oi)


@pytest.mark.parametrize("k", [3, 4, 5])
def test_full_size_configs(zl, oracle, k):
    # every instance of the 2 GiB shapes against the oracle on the written-out rows (a quarter of the batch at a time)
    cfg = workloads.CONFIGS[k]
    le, iv = workloads.make_predicted(k, shift=EPOCH)
    bar, it, w, st = gpu_run(zl, le, iv, cfg.R)
    assert (st == 0).all()
    for part in np.array_split(np.arange(cfg.B), 4):
        ob, oi, ow, rc, _ = oracle.zipline(oracle.predicted_rows(le[part], iv[part], cfg.R), "sweep", threads=16)
        assert (rc == 0).all()
        assert np.array_equal(bar[part], ob), f"barrier differs at {part[np.nonzero(bar[part] != ob)[0][:5]]}"
        assert np.array_equal(w[part], ow) and np.array_equal(it[part], oi)
    # properties that hold for every instance: each worker stops at its last predicted timestamp <= barrier,
    # the stops sum to the reported wait, some worker stops exactly at the barrier
    stop = le + it.astype(np.int64) * iv
    assert (it >= 1).all() and (it <= cfg.R).all()
    assert (stop <= bar[:, None]).all()
    assert ((it == cfg.R) | (stop + iv > bar[:, None])).all()
    assert (stop.max(axis=1) == bar).all()
    assert ((bar[:, None] - stop).sum(axis=1) == w).all()


# few workers or few instances: every candidate is evaluated.  A wave per search and four, with candidates that end inside a
# wave's step; several workgroups per search; workers split among waves; either side of the limits on workers and batch
DIRECT = [(2000, 4, 60), (2100, 16, 65), (1200, 40, 103), (4400, 16, 15), (300, 41, 90), (3, 48, 21), (3, 49, 20), (3, 49, 21), (300, 16, 300),
          (5, 12, 400), (3, 64, 500), (2, 65, 200), (1, 100, 163), (1, 101, 180), (1, 257, 61), (2, 1024, 17), (1, 1023, 30), (1, 1025, 20),
          (1, 1, 5000), (2, 3, 9000)]


@pytest.mark.parametrize("B,P,R", DIRECT)
def test_every_candidate_evaluated(zl, oracle, B, P, R):
    rng = np.random.default_rng(B + 7 * P + R)
    for ties in (False, True):
        le, iv = random_inputs(rng, B, P, 500, 1000, ties)
        assert_same(zl, oracle, le + EPOCH, iv, R, f"B={B} P={P} R={R} ties={ties}")
    iv[:, ::3] //= 50                                                      # through early, or standing still
    iv[: (B + 1) // 2, 0] = 0
    assert_same(zl, oracle, le, iv, R, f"B={B} P={P} R={R}, very different workers")
    assert_same(zl, oracle, np.zeros_like(le), np.full_like(iv, 12_345), R, f"B={B} P={P} R={R}, all alike")


@pytest.mark.parametrize("P,R", [(2, 3), (16, 60), (16, 300), (100, 150), (300, 60)])
def test_every_candidate_evaluated_at_the_limits_of_double_precision(zl, oracle, P, R):
    # the largest values that are divided in double precision, and beyond them, where they are divided as whole numbers
    rng = np.random.default_rng(P * R)
    most = (1 << 47) // P
    for first, step in ((most - most // R, most // R), (most, most // R + 1), (1 << 55 - P.bit_length(), 1 << 54 - (P * R).bit_length())):
        iv = step - rng.integers(0, 1 + step // 1000, size=(3, P)).astype(np.int64)
        le = first - rng.integers(0, 1 + step // 3, size=(3, P)).astype(np.int64)
        le[:, 0] = 0                                                       # the value that the others are taken relative to
        iv[1] -= iv[1] % 1000
        assert_same(zl, oracle, le, iv, R, f"P={P} R={R} first {first} step {step}")
        assert_same(zl, oracle, -le, iv, R, f"P={P} R={R} first -{first} step {step}")


# the same where the sums over the workers set the limit (2^51 / P) or the quotients do (2^47), one step inside and one beyond;
# and whole numbers of every size up to what P of them may spread over, workers that stand still and that step by 1 among them
@pytest.mark.parametrize("P,R", [(2, 3), (15, 65), (16, 60), (17, 300), (100, 150), (300, 60), (1000, 150)])
def test_every_candidate_evaluated_beyond_double_precision(zl, oracle, P, R):
    rng = np.random.default_rng(P * R)
    most = min(1 << 47, (1 << 51) // P)
    for first, step in ((most - most // R, most // R), (most - most // R + 1, most // R), (0, most // R), (0, most // R + 1)):
        iv = step - rng.integers(0, 1 + step // 1000, size=(2, P)).astype(np.int64)
        iv[:, P // 2] = step
        le = first - rng.integers(0, 1 + first // 3, size=(2, P)).astype(np.int64)
        le[:, 0], le[:, P - 1] = 0, first
        assert_same(zl, oracle, le, iv, R, f"P={P} R={R} first {first} step {step}")
        assert_same(zl, oracle, -le, iv, R, f"P={P} R={R} first -{first} step {step}")
    widest = (1 << 62) // (P * R)
    iv = (widest * 2.0 ** -rng.uniform(0, 50, size=(6, P))).astype(np.int64)
    le = (widest * 2.0 ** -rng.uniform(0, 50, size=(6, P))).astype(np.int64)
    iv[:, 0] = widest
    iv[2:4, 1::5] = 0
    iv[4:, 1::3] = 1
    iv[5, 1::2] = widest - 1
    assert_same(zl, oracle, le, iv, R, f"P={P} R={R} up to {widest}")
    assert_same(zl, oracle, le, np.sort(iv, axis=1) // 7 * 7, R, f"P={P} R={R} up to {widest}, sorted")


@pytest.mark.parametrize("P,R", [(16, 60), (16, 300), (100, 150)])
def test_every_candidate_evaluated_flags(zl, oracle, P, R):
    rng = np.random.default_rng(P)
    le, iv = random_inputs(rng, 4, P, 500, 1000, False)
    iv[1, P // 2] = -3
    iv[2, P - 1] = (1 << 62) // R
    st = gpu_run(zl, le, iv, R)
    assert st[3][1] & zl.STATUS_UNSORTED and st[3][2] & zl.STATUS_OVERFLOW and st[3][0] == 0 and st[3][3] == 0
    ob, oi, ow, rc, _ = oracle.zipline(oracle.predicted_rows(le[::3], iv[::3], R), "sweep", threads=4)
    assert np.array_equal(st[0][::3], ob) and np.array_equal(st[1][::3], oi) and np.array_equal(st[2][::3], ow)


@pytest.mark.parametrize("P,R", [(2, 1), (16, 60), (16, 300), (100, 150), (300, 60)])
def test_every_candidate_evaluated_flags_start_times_2_to_the_64_apart(zl, oracle, P, R):
    # no row overflows, but the distance of two start times does: modulo 2^64 it looks small
    rng = np.random.default_rng(P)
    le, iv = random_inputs(rng, 4, P, 500, 1000, False)
    for b, far in ((1, 1), (2, P - 1)):
        le[b] -= le[b].min()
        le[b, :far] += np.iinfo(np.int64).min
        le[b, far:] = np.iinfo(np.int64).max - R * iv[b, far:]
    st = gpu_run(zl, le, iv, R)
    assert st[3].tolist() == [0, zl.STATUS_OVERFLOW, zl.STATUS_OVERFLOW, 0]
    ob, oi, ow, rc, _ = oracle.zipline(oracle.predicted_rows(le[::3], iv[::3], R), "sweep", threads=4)
    assert np.array_equal(st[0][::3], ob) and np.array_equal(st[1][::3], oi) and np.array_equal(st[2][::3], ow)


# windows that are ruled out by what others of the instance have found: equal waits in all of them (the first is the answer),
# the best one in the last, in the first, in a window without a rival; workgroups of 256, 512 and 1024 threads
@pytest.mark.parametrize("B,P,R", [(2, 300, 1000), (1, 70, 4000), (3, 700, 400), (1, 1600, 170)])
def test_windows_that_rule_each_other_out(zl, oracle, B, P, R):
    rng = np.random.default_rng(P + R)
    le, iv = random_inputs(rng, B, P, 500, 1000, False)
    assert_same(zl, oracle, le + EPOCH, iv, R, f"P={P} R={R}")
    assert_same(zl, oracle, np.zeros_like(le), np.full_like(iv, 12_000), R, f"P={P} R={R}, all alike")
    group = 3000 * (1 << rng.integers(0, 3, size=(B, P))).astype(np.int64)
    assert_same(zl, oracle, np.zeros_like(le), group, R, f"P={P} R={R}, the same wait again and again")
    assert_same(zl, oracle, rng.integers(0, 40, size=(B, P)).astype(np.int64), group, R, f"P={P} R={R}, nearly the same wait")
    for at in (R - 1, R // 2, 3):                                     # all workers meet once, after `at` iterations
        iv = 2000 + rng.integers(-300, 300, size=(B, P)).astype(np.int64)
        assert_same(zl, oracle, 3000 * R - at * iv, iv, R, f"P={P} R={R}, they meet after {at}")
