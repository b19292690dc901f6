"""The benchmark's byte model (no GPU): every kernel that a search may launch has one."""
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


def test_bytes_of_the_searches_in_one_launch():
    # 3 instances of 16 x 60; outputs: barrier, wait and an iteration count per worker
    out = 3 * (16 + 4 * 16)
    assert bench.algorithmic_bytes("zl_run_kernel", 3, 16, 60, 0, 0) == 8 * 3 * 16 * 60 + out
    assert bench.algorithmic_bytes("zl_run_kernel", 3, 16, 60, 0, 0, predicted=True) == 16 * 3 * 16 + out
    # a run of 8: the start times once, the intervals of every superstep
    assert 8 * bench.algorithmic_bytes("zl_run_kernel", 3, 16, 60, 0, 0, True, 8) == 8 * 3 * 16 + 8 * (8 * 3 * 16 + out)
