"""The kernels that take one pair per lane (csrc/lanes.h): under the CPU
emulation with its sanitizers at launches of few workgroups, so that a
workgroup takes several rounds of pairs, and on the GPU through the launch
fields that lead there."""
import numpy as np
import pytest

import paper_2203_15561_amd as ga
from tests.emu import run as emu
from tests.test_pair_paths import expected_of, pairs_of
from workloads import gen


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return emu.build(str(tmp_path_factory.mktemp("emu") / "emu_driver"))


def results(res, cig):
    assert (res["flags"] == 0).all()
    return [(int(r["edit_distance"]), c, int(r["ref_begin"]), int(r["ref_end"]), int(r["n_windows"]))
            for r, c in zip(res, cig)]


def rounds_of_pairs(n, seed):
    # reads of one window at most (W - O = 40 bases and less), so that a round of
    # pairs ends at its first barrier; some that fail, some without reads
    return pairs_of(n, seed, [30, 1, 40, 17, 39, 0, 25], [60, 1, 40, 90, 0, 33])


@pytest.mark.slow
@pytest.mark.parametrize("k", [64, 3])
def test_rounds_of_one_window_emulated(driver, k):
    # 200 pairs on two workgroups of 32 lanes: four rounds; and the other way round
    # (the second wavefront computes)
    ps = gen.from_lists("rounds", *rounds_of_pairs(200, 71), k)
    want = expected_of(ps)
    for turned_from in (1 << 30, 0):
        got = results(*emu.run(driver, ps, emu.LANES, pair_lanes=32, window_blocks=2, turned_from=turned_from))
        assert got == want


@pytest.mark.slow
@pytest.mark.parametrize("budget,ticks", [(1, 0), (0, 1)])
def test_serving_rounds_emulated(driver, budget, ticks):
    # one workgroup and more resident pairs than its 64 lanes, every turn one
    # window: each round ends at its first barrier
    reads, refs = pairs_of(150, 72, [30, 70, 100, 1, 45], [60, 120, 40])
    ps = gen.from_lists("rounds", reads, refs, 64)
    got = results(*emu.run(driver, ps, emu.SERVE_LANES, window_blocks=1, slots=140, admit_per_iteration=140,
                           window_budget=budget, ticks=ticks, search_chunk=64))
    assert got == expected_of(ps)


@pytest.mark.gpu
def test_rounds_of_one_window():
    # one workgroup a compute unit: 40,000 pairs are three rounds and more
    reads, refs = rounds_of_pairs(40_000, 73)
    ps = gen.from_lists("rounds", reads, refs, 64)
    want = expected_of(ps)
    with ga.Context(0) as ctx:
        for lpt in (1, 0):
            launch = ga.make_launch(ga.FORM_BATCHED, workers_per_cu=1, lpt_order=lpt)
            got = results(*ctx.align(reads, refs, 64, launch=launch))
            bad = [i for i in range(len(reads)) if got[i] != want[i]]
            assert not bad, (lpt, len(bad), bad[:5], got[bad[0]], want[bad[0]])
