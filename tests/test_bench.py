"""The benchmark's byte model (no GPU): every kernel that a search may launch has one."""
import os
import re

import numpy as np
import pytest

import bench
from paper_2001_01347_amd import zipline

NOT_A_SEARCH = {"zl_copy_kernel", "zl_read_kernel", "zl_gridscan_kernel", "zl_gridscan_finish_kernel"}
NOTHING_TO_DO = {"zl_window_general_kernel", "zl_instance_general_kernel"}


def test_every_kernel_of_a_search_is_priced():
    for name in zipline.ebsp_zipline_kernel_names():
        if name in NOT_A_SEARCH:
            continue
        for predicted in (False, True):
            got = bench.algorithmic_bytes(name, 2, 100, 50, 20, 8, predicted)
            assert got == 0.0 if name in NOTHING_TO_DO else got > 0.0, name
    with pytest.raises(ValueError):
        bench.algorithmic_bytes("zl_unheard_of_kernel", 2, 100, 50, 20, 8)


def test_kernels_of_slices_are_named_and_priced():
    assert bench.named_by_what_ran({"zl_bounds_kernel": 1.0, "zl_window_kernel": 2.0}) == {"zl_bounds_kernel": 1.0, "zl_window_kernel": 2.0}
    assert bench.named_by_what_ran({"zl_cells_kernel": 1.0}) == {"zl_cells_kernel": 1.0}
    got = bench.named_by_what_ran({k: 1.0 for k in bench.OF_SLICES})
    assert set(got) == set(bench.OF_SLICES.values())
    for predicted, rows in ((False, 8.0 * 2 * 100 * 50), (True, 16.0 * 2 * 100)):
        assert bench.algorithmic_bytes("zl_slices_kernel", 2, 100, 50, 20, 8, predicted) == rows
        assert all(bench.algorithmic_bytes(k, 2, 100, 50, 20, 8, predicted) >= 0.0 for k in got)


def test_bytes_of_the_searches_in_one_launch():
    # 3 instances of 16 x 60; outputs: barrier, wait and an iteration count per worker
    out = 3 * (16 + 4 * 16)
    assert bench.algorithmic_bytes("zl_run_kernel", 3, 16, 60, 0, 0) == 8 * 3 * 16 * 60 + out
    assert bench.algorithmic_bytes("zl_run_kernel", 3, 16, 60, 0, 0, predicted=True) == 16 * 3 * 16 + out
    # a run of 8: the start times once, the intervals of every superstep
    assert 8 * bench.algorithmic_bytes("zl_run_kernel", 3, 16, 60, 0, 0, True, 8) == 8 * 3 * 16 + 8 * (8 * 3 * 16 + out)


def test_the_librarys_limits_of_the_value_cut():
    csrc = os.path.join(os.path.dirname(bench.__file__), "paper_2001_01347_amd", "csrc")
    text = "".join(open(os.path.join(csrc, f)).read() for f in ("zipline.hip", "zl_plan.h"))
    for name in ("CUT_MIN_WINDOWS", "CUT_ROWS", "CUT_STEPS"):
        assert int(re.search(rf"constexpr \w+ {name} = (\d+);", text).group(1)) == getattr(bench, name), name


def test_entries_behind_the_last_value_that_can_win_by_hand():
    # the first worker is through at 3, the second starts at 10: the best barrier by then waits 10 - 3 = 7, and every
    # later one longer, since the first worker already waits more; 1, 2, 3 and 10 are left
    t = np.array([[[1, 2, 3], [10, 20, 30]]])
    assert bench.searched_entries(t, True) == bench.searched_entries(t, False) == 4
    # the same workers predicted: (1, 2, 3) from 0 by 1, (10, 20, 30) from 0 by 10
    assert bench.searched_entries((np.array([[0, 0]]), np.array([[1, 10]]), 3), True) == 4
    # what is priced: 4 entries of 6, one window
    assert bench.algorithmic_bytes("zl_window_kernel", 1, 2, 3, 1, 1, searched=4.0) == 8 * 4 + 2 * 2 * 2 + 16


@pytest.mark.parametrize("P,R", [(2, 9), (5, 7), (30, 20)])
def test_no_entry_behind_it_is_a_best_barrier(P, R):
    rng = np.random.default_rng(P)
    kept = 0
    for k in range(40):
        t = np.cumsum(rng.integers(1, 30, size=(P, R)) * rng.integers(1, 9, size=(P, 1)), axis=1) + rng.integers(0, 90, size=(P, 1))
        last = lambda c: np.array([row[row <= c].max() for row in t])
        every = np.unique(t[t >= t[:, 0].max()])
        for summed, cost in ((True, lambda c: (c - last(c)).sum()), (False, lambda c: (c - last(c)).max())):
            C = bench.last_value_that_can_win(t[:, 0], t[:, -1], last, summed)
            best = min(cost(c) for c in every if c <= C)
            assert all(cost(c) > best for c in every if c > C)
            assert bench.searched_entries(t[None], summed) == (t <= C).sum()
            kept += (t <= C).sum()
    assert kept < 40 * 2 * P * R        # and it leaves something out
