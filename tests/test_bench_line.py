"""bench.py's roofline counts the operations of the kernel that ran (no GPU)."""
import bench
import paper_2203_15561_amd as ga

PROFILE = {"window_cells": 6400, "window_word_ops": 5000, "window_workgroups": 20, "n_pairs": 1000}


def test_window_kernel_operations():
    def ran(commit=40, workgroups=20, **kw):
        launch = ga.make_launch(ga.FORM_BATCHED, **kw)
        name, ops = bench.window_kernel(launch, dict(PROFILE, window_workgroups=workgroups), commit)
        return name.split()[0], ops

    # 100 columns of 64 cells, whatever the distances are
    assert ran() == ("k_windows_lane", 3400)
    assert ran(workers_per_cu=2, lpt_order=0) == ("k_windows_lane", 3400)
    assert ran(workgroups=1000) == ("k_pair_wave", None)
    # the row recurrence: two halves a word operation
    assert ran(commit=41) == ("k_windows", 10000)
    for field, value in (("table_bits", 32), ("hard_row", 24), ("hard_row", -1), ("search_per_cu", 4), ("hard_share", 25)):
        assert ran(**{field: value}) == ("k_windows", 10000), field
    assert ran(hard_share=-1, tb_prefetch=-1) == ("k_windows_lane", 3400)
