"""The one-pair-per-lane path (csrc/lanes.h): its window on the CPU against a
textbook dynamic program, and the batched launch that takes it against the
oracle at the sizes where its launch, its blocks of columns and its short
windows have their edges."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2203_15561_amd as ga
from tests._helpers import rle
from workloads import gen

HERE = os.path.dirname(os.path.abspath(__file__))


def test_window_path_against_textbook(tmp_path):
    exe = str(tmp_path / "window_path_test")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                           os.path.join(HERE, "lanes", "window_path_test.cpp"), "-o", exe])
    out = subprocess.run([exe, "7", "40000"], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr


def pairs_of(n, seed, read_len, ref_len):
    """n pairs cycling over the given read and reference lengths, related at
    error rates of 0 to 40%, every seventh reference unrelated."""
    reads, refs = [], []
    for i in range(n):
        rng = gen.pair_rng(seed, i)
        m, t = read_len[i % len(read_len)], ref_len[(i // len(read_len)) % len(ref_len)]
        read = gen.random_bases(rng, m)
        ref = gen.random_bases(rng, t)
        if i % 7 and m and t:
            core = gen.mutate(rng, read, rng.uniform(0, 0.4), (1 / 3, 1 / 3, 1 / 3))[:t]
            at = int(rng.integers(0, t - len(core) + 1))
            ref[at:at + len(core)] = core
        reads.append(read)
        refs.append(ref)
    return reads, refs


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 2, 63, 65, 513, 1025])
@pytest.mark.parametrize("W,O,k", [(64, 24, 64), (64, 24, 9), (64, 32, 64), (64, 23, 64), (33, 9, 64),
                                   (40, 0, 40), (8, 7, 3)])
def test_batched_launch_at_its_edges(n, W, O, k):
    # 1 to 64 pairs per wavefront and a last wavefront that is not full; reads
    # and references around 0, 1, 40, 64 and 128 bases and around several search
    # parts; W - O of 40 and less (the lane path) and of 41 (the row tables)
    reads, refs = pairs_of(n, 900 + W + O, [150, 0, 1, 39, 40, 41, 63, 64, 65, 104, 129, 600],
                           [170, 64, 0, 1, 63, 65, 128, 129, 640, 1500])
    ps = gen.from_lists("edges", reads, refs, k, W, O)
    res_o, ops_o, _, _ = oracle.batch(ps)
    with ga.Context(0) as ctx:
        res, cig = ctx.align(reads, refs, k, W, O)
    assert (res["flags"] == 0).all()
    for i in range(n):
        sc = int(res_o["score"][i])
        want = (sc, rle(oracle.pair_ops(ps, res_o, ops_o, i)) if sc >= 0 else "",
                int(res_o["ref_begin"][i]) if sc >= 0 else 0, int(res_o["ref_end"][i]) if sc >= 0 else 0,
                int(res_o["n_windows"][i]))
        r = res[i]
        got = (int(r["edit_distance"]), cig[i], int(r["ref_begin"]), int(r["ref_end"]), int(r["n_windows"]))
        assert got == want, (i, len(reads[i]), len(refs[i]), got, want)


@pytest.mark.gpu
def test_one_read_against_a_long_reference():
    # more search parts than lanes of a wavefront: the parts' keys combine in
    # device memory
    rng = np.random.default_rng(11)
    ref = rng.integers(0, 4, 300_001).astype(np.uint8)
    reads, want = [], []
    for at in (0, 77_777, 299_950):
        reads.append(ref[at:at + 50].copy())
        want.append(at)
    with ga.Context(0) as ctx:
        for r, at in zip(reads, want):
            res, cig = ctx.align([r], [ref], 5)
            assert (int(res["edit_distance"][0]), int(res["ref_begin"][0]), cig[0]) == (0, at, "50=")


@pytest.mark.gpu
@pytest.mark.parametrize("longest", [1, 64, 65, 128, 256, 257, 512, 513, 1024])
def test_filter_at_its_edges(longest):
    # a lane per 64 read bases: reads up to each lane count's limit, shorter
    # ones whose last lanes have no rows, references around 0 and around blocks
    # of 32 columns, k from 0 to past the read length
    lens = sorted({m for m in (0, 1, 2, 40, 63, 64, 65, 127, 129, 255, 400, longest - 1, longest) if 0 <= m <= longest})
    reads, refs = pairs_of(90, 40 + longest, lens, [longest + 9, 0, 1, 31, 32, 33, 64, 65, longest + 60])
    with ga.Context(0) as ctx:
        for k in (0, 12, 63):
            dist, start = ctx.filter(reads, refs, k)
            for i in range(len(reads)):
                want = oracle.filter_pair(reads[i], refs[i], k)
                got = (int(dist[i]), int(start[i]))
                assert got == (want if want[0] >= 0 else (-1, 0)), (i, len(reads[i]), len(refs[i]), k, got, want)
