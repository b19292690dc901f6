"""The summed-wait search over value cells in slices (``zl_slices_kernel`` and what follows it) against the CPU oracle, bit
for bit: the shapes at the edges of its rule, and the inputs that leave its common path (needs an MI355X)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPOCH = 1_700_000_000_000_000


@pytest.fixture(scope="module")
def zl():
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2001_01347_amd import zipline
    zipline.load()
    return zipline


def sliced(zl, call):
    """The call's outputs, and whether it went by slices (which need no zl_bounds_kernel)."""
    zl.ebsp_zipline_profile_begin(1)
    out = call()
    ms, _ = zl.ebsp_zipline_profile_end()
    return [x.cpu().numpy() for x in out], ms["zl_window_kernel"] > 0 and ms["zl_bounds_kernel"] == 0


def same_as(got, want, label):
    bar, it, w, st = got
    ob, oi, ow, rc, _ = want
    assert (rc == 0).all() and (st == 0).all(), f"{label}: status {np.unique(st)}"
    assert np.array_equal(w, ow), f"{label}: wait differs at {np.nonzero(w != ow)[0][:5]}"
    assert np.array_equal(bar, ob), f"{label}: barrier differs at {np.nonzero(bar != ob)[0][:5]}"
    assert np.array_equal(it, oi), f"{label}: iters differ at {np.nonzero((it != oi).any(axis=1))[0][:5]}"


# rows either side of a wave and of a workgroup's threads, one entry more than a chunk, the fewest and the most rows, short rows
@pytest.mark.parametrize("B,P,R", [(3, 8, 32769), (2, 63, 4200), (2, 64, 4097), (2, 65, 4099), (3, 511, 520), (40, 1024, 17), (24, 1023, 241),
                                   (30, 1000, 33), (300, 129, 128)])
def test_predicted_rows(zl, oracle, B, P, R):
    rng = np.random.default_rng(P * R)
    mean = rng.integers(20_000, 200_000, size=(B, P)).astype(np.int64)
    off = (rng.random((B, P)) * mean).astype(np.int64)
    some = rng.random((B, P)) < 0.1
    cases = {"spread": (off, mean),
             "ties": (off // 1000 * 1000, mean // 1000 * 1000),
             "nanoseconds": (off * 1000 + 7, mean * 1000 + rng.integers(0, 1000, size=(B, P))),
             "one iteration time": (off, np.full_like(mean, 100_000)),
             "one iteration time, starts far apart": ((rng.random((B, P)) ** 3 * 1.2 * R * 100_000).astype(np.int64), np.full_like(mean, 100_000)),
             "one iteration time, others in one": (off, np.where(np.arange(B)[:, None] % 2 == 0, 1, mean)),
             "in step": (off % 20, np.full_like(mean, 100_000)),
             "in step, nanoseconds": (off % 20_000, np.full_like(mean, 100_000_000)),
             "identical": (np.zeros_like(off), np.full_like(mean, 777)),
             "some stand still": (off, np.where(some, 0, mean)),
             "one late": (np.where(np.arange(P) == P // 2, off + 30 * mean.max(), off), mean),
             "one slow": (off, np.where(np.arange(P) == P // 3, mean * 10_000, mean)),
             "spreads of 2^45": (off << 24, mean << 24)}
    for label, (le, iv) in cases.items():
        for epoch in (0, EPOCH):
            le_, iv_ = torch.from_numpy(le + epoch).cuda(), torch.from_numpy(iv).cuda()
            got, is_sliced = sliced(zl, lambda: zl.ebsp_predict_zipline_batch(le_, iv_, R))
            assert is_sliced
            same_as(got, oracle.zipline(oracle.predicted_rows(le + epoch, iv, R), "sweep", threads=16), f"{B} x {P} x {R} {label} from {epoch}")


def stored_rows(B, P, R, kind, seed):
    rng = np.random.default_rng(seed)
    mean = rng.integers(20_000, 200_000, size=(B, P, 1)) if kind != "alike" else rng.integers(95_000, 105_000, size=(B, P, 1))
    d = rng.integers(90, 111, size=(B, P, R), dtype=np.int64)
    if kind == "in step":
        return np.arange(1, R + 1) * 100_000 + rng.integers(0, 20, size=(B, P, R), dtype=np.int64)
    d *= mean // 100
    t = np.cumsum(d, axis=2) + (rng.random((B, P, 1)) * mean).astype(np.int64)
    if kind == "ties":
        t = t // 1000 * 1000
    if kind == "nanoseconds":
        t = t * 1000 + 321
    if kind == "pauses":
        t[:, :, R // 3:] += 3_000_000_000 * (rng.random((B, P, 1)) < 0.2)
    return t


# the fewest entries that go by slices: few instances of many rows (several slices each), and one workgroup per instance
@pytest.mark.parametrize("kind", ["spread", "alike", "ties", "nanoseconds", "pauses", "in step"])
@pytest.mark.parametrize("B,P,R", [(48, 1021, 1031), (640, 150, 523)])
def test_stored_rows(zl, oracle, B, P, R, kind):
    ts = stored_rows(B, P, R, kind, P + R) + EPOCH
    dev = torch.from_numpy(ts).cuda()
    got, is_sliced = sliced(zl, lambda: zl.ebsp_zipline_batch(dev))
    assert is_sliced
    same_as(got, oracle.zipline(ts, "sweep", threads=16), f"{B} x {P} x {R} {kind}")


def test_stored_rows_out_of_order_are_flagged_wherever_they_are(zl, oracle):
    B, P, R = 48, 1021, 1031
    ts = stored_rows(B, P, R, "spread", 5) + EPOCH
    where = [1, 2, 3, 60, R // 8, R // 4, R // 2, R - 200, R - 2, R - 1]      # before the first barrier, in the slices, behind the last value that can win
    for b, i in enumerate(where):
        for p in (int(ts[b, :, -1].argmin()), int(ts[b, :, -1].argmax())):
            ts[b, p, i] = ts[b, p, i - 1] - 1
    big = len(where)
    ts[big, 3, R // 2:] += 1 << 60                                           # P waits of that size do not fit
    bar, it, w, st = [x.cpu().numpy() for x in zl.ebsp_zipline_batch(torch.from_numpy(ts).cuda())]
    assert (st[:big] == 1).all() and st[big] == 2 and (st[big + 1:] == 0).all(), st
    rest = ts[big + 1:]
    same_as([x[big + 1:] for x in (bar, it, w, st)], oracle.zipline(rest, "sweep", threads=16), "the others")


# One common pause: with all workers in step after it, their steps over it fall into one or two cells, whose sums pass 2^32, and
# the slices there are left to the search by windows.  A quarter of the workers end early: values behind those that can win.
@pytest.mark.parametrize("B,P,R", [(512, 256, 768), (60, 1021, 1031)])       # one slice per instance, and several
def test_stored_rows_of_a_slice_that_is_left(zl, oracle, B, P, R):
    rng = np.random.default_rng(P)
    T, pause, early = 100_000, 100_000_000, np.arange(P) % 4 == 0
    assert (P - early.sum()) * pause // 2 > 1 << 32 and 0.7 * 0.6 * T / np.sqrt(12 * P) > 20      # wider than the workers are apart
    ts = np.where(early, 6 * T // 10, T)[:, None] * np.arange(1, R + 1) + rng.integers(0, 20, size=(B, P, R), dtype=np.int64)
    ts += np.where(ts > T * R // 5, pause, 0) + EPOCH
    dev = torch.from_numpy(ts).cuda()
    got, is_sliced = sliced(zl, lambda: zl.ebsp_zipline_batch(dev))
    assert is_sliced
    same_as(got, oracle.zipline(ts, "sweep", threads=16), f"{B} x {P} x {R} sorted")
    where = [R // 10, R // 5 + 3, R // 4, R // 3, 2 * R // 5, R // 2, 2 * R // 3, R - 2, R - 1]      # before the pause, after it, behind
    for b, i in enumerate(where):
        p = 1 + 4 * b                                                        # (a worker that ends late)
        ts[b, p, i] = ts[b, p, i - 1] - 1
    bar, it, w, st = [x.cpu().numpy() for x in zl.ebsp_zipline_batch(torch.from_numpy(ts).cuda())]
    n = len(where)
    assert (st[:n] == 1).all() and (st[n:] == 0).all(), st
    same_as([x[n:] for x in (bar, it, w, st)], oracle.zipline(ts[n:], "sweep", threads=16), "the others")


def test_rows_out_of_order_are_flagged_where_values_are_too_far_apart_too(zl):
    B, P, R = 60, 1021, 1031
    ts = stored_rows(B, P, R, "spread", 7) + EPOCH
    ts[::2, 3, R // 2:] += 1 << 60                                           # P waits of that size do not fit
    where = [(b, (37 * b + 5) % P, 1 + (97 * b) % (R - 1)) for b in range(0, B, 4)]
    for b, p, i in where:
        ts[b, p, i] = ts[b, p, i - 1] - 1
    (_, _, _, st), is_sliced = sliced(zl, lambda: zl.ebsp_zipline_batch(torch.from_numpy(ts).cuda()))
    assert is_sliced
    assert st.tolist() == [3 if b % 4 == 0 else 2 if b % 2 == 0 else 0 for b in range(B)]


# Workers whose waits repeat: every cell of one kind may win, and the instances are searched by windows.  In nanoseconds, and with
# the entries so far apart that almost every window of 2^32 values is empty.
def intervals_of(kind, rng, B, P):
    return {"one": np.full((B, P), 100_000), "two": np.where(rng.random((B, P)) < 0.3, 200_000, 100_000),
            "almost one": 100_000 + rng.integers(0, 3, size=(B, P))}[kind].astype(np.int64)


@pytest.mark.parametrize("unit", [1, 1000, 1 << 27])
@pytest.mark.parametrize("B,P,R", [(3, 8, 32769), (150, 64, 500), (24, 1023, 241)])
def test_predicted_rows_whose_waits_repeat(zl, oracle, B, P, R, unit):
    rng = np.random.default_rng(P + R)
    for kind in ("two", "almost one"):
        iv = intervals_of(kind, rng, B, P) * unit
        for label, off in (("anywhere", (rng.random((B, P)) * 100_000).astype(np.int64) * unit), ("in step", rng.integers(0, 20 * unit, size=(B, P)))):
            le = off + EPOCH
            got, is_sliced = sliced(zl, lambda: zl.ebsp_predict_zipline_batch(torch.from_numpy(le).cuda(), torch.from_numpy(iv).cuda(), R))
            assert is_sliced
            same_as(got, oracle.zipline(oracle.predicted_rows(le, iv, R), "sweep", threads=16), f"{B} x {P} x {R} {kind}, {label}, {unit}")


@pytest.mark.parametrize("unit", [1, 1000])
@pytest.mark.parametrize("kind", ["one", "two", "almost one", "in step"])
@pytest.mark.parametrize("B,P,R", [(48, 1021, 1031), (640, 150, 523), (190, 257, 1024)])
def test_stored_rows_whose_waits_repeat(zl, oracle, B, P, R, kind, unit):
    rng = np.random.default_rng(P + R)
    if kind == "in step":
        ts = np.arange(R) * (100_000 * unit) + rng.integers(0, 20 * unit, size=(B, P, R)) + EPOCH
    else:
        iv = intervals_of(kind, rng, B, P) * unit
        off = (rng.random((B, P)) * 100_000).astype(np.int64) * unit
        ts = off[:, :, None] + np.arange(R) * iv[:, :, None] + EPOCH
    got, is_sliced = sliced(zl, lambda: zl.ebsp_zipline_batch(torch.from_numpy(ts).cuda()))
    assert is_sliced
    same_as(got, oracle.zipline(ts, "sweep", threads=16), f"{B} x {P} x {R} {kind}, {unit}")
    where = [1, 2, R // 8, R // 4, R // 2, R - 200, R - 2]                   # (the last entry stays: all rows of one length)
    for b, i in enumerate(where):
        ts[b, 7 * b, i] = ts[b, 7 * b, i - 1] - 1
    st = zl.ebsp_zipline_batch(torch.from_numpy(ts).cuda())[3].cpu().numpy()
    assert (st[:len(where)] == 1).all() and (st[len(where):] == 0).all(), st
