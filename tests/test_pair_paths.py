"""The paths that take one pair per lane (csrc/lanes.h) and one pair per
wavefront (csrc/wave_pair.h): a lane's window on the CPU against a textbook
dynamic program, the wavefront's kernel under the CPU emulation and both paths
on the GPU against the oracle at the sizes where their launches, their blocks
of columns, their bands of diagonals and their short windows have their
edges; and the filter at its edges."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2203_15561_amd as ga
from tests._helpers import rle
from tests.emu import run as emu
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


def expected_of(ps):
    res, ops, _, _ = oracle.batch(ps)
    return [(int(res["score"][i]), rle(oracle.pair_ops(ps, res, ops, i)) if res["score"][i] >= 0 else "",
             int(res["ref_begin"][i]) if res["score"][i] >= 0 else 0,
             int(res["ref_end"][i]) if res["score"][i] >= 0 else 0, int(res["n_windows"][i]))
            for i in range(ps.n_pairs)]


@pytest.mark.slow
def test_wavefront_kernel_emulated(tmp_path):
    # every overlap and cap, unrelated pairs (distances past the band of 64
    # diagonals, which take the full band), reads past their reference's end
    driver = emu.build(str(tmp_path / "emu_driver"))
    reads, refs = pairs_of(9, 31, [70, 1, 64, 103], [90, 0, 64, 20])
    for W, O, k in ((64, 24, 64), (64, 0, 64), (64, 63, 20), (33, 9, 7), (2, 1, 1)):
        ps = gen.from_lists("wave", reads, refs, k, W, O)
        res, cig = emu.run(driver, ps, 0, 16, 16, 16)
        got = [(int(r["edit_distance"]), c, int(r["ref_begin"]), int(r["ref_end"]), int(r["n_windows"]))
               for r, c in zip(res, cig)]
        assert (res["flags"] == 0).all() and got == expected_of(ps), (W, O, k)


@pytest.mark.gpu
@pytest.mark.parametrize("n,form", [(1, None), (65, None), (2047, None), (2048, ga.FORM_PLAIN),
                                    (2049, None), (4096, None), (4097, None), (33_001, None)])
@pytest.mark.parametrize("W,O,k", [(64, 24, 64), (64, 24, 9), (64, 32, 64), (64, 23, 64), (33, 9, 64),
                                   (40, 0, 40), (8, 7, 3)])
def test_batched_launch_at_its_edges(n, form, W, O, k):
    # up to 4,096 short pairs (2,048 where one reference makes them long on
    # average) one per wavefront, past that 8, 16 and 64 pairs per wavefront and
    # a last one that is not full; reads and references around 0, 1,
    # 40, 64 and 128 bases and around several search parts, unrelated pairs (deep
    # windows); W - O of 40 and less (the lane path) and of 41 (the row tables)
    reads, refs = pairs_of(n, 900 + W + O, [150, 0, 1, 39, 40, 41, 63, 64, 65, 104, 129, 600],
                           [170, 64, 0, 1, 63, 65, 128, 129, 640, 1500])
    if n == 2049:
        refs[5] = gen.random_bases(gen.pair_rng(901, n), 600 * n)
    ps = gen.from_lists("edges", reads, refs, k, W, O)
    want_all = expected_of(ps)
    with ga.Context(0) as ctx:
        res, cig = ctx.align(reads, refs, k, W, O, None if form is None else ga.make_launch(form))
    assert (res["flags"] == 0).all()
    for i in range(n):
        r = res[i]
        got = (int(r["edit_distance"]), cig[i], int(r["ref_begin"]), int(r["ref_end"]), int(r["n_windows"]))
        assert got == want_all[i], (i, len(reads[i]), len(refs[i]), got, want_all[i])


@pytest.mark.gpu
@pytest.mark.parametrize("shift", [0, 1, 4, 8, 13])
def test_packed_streams_at_any_address(shift):
    # the planes come from 8-byte loads of aligned streams and bytes otherwise, up
    # to the stream's last byte: the host form's results at every alignment
    import torch

    def stream(seqs):
        codes = np.concatenate(seqs)
        codes = np.concatenate([codes, np.zeros(-len(codes) % 4, np.uint8)]).reshape(-1, 4)
        packed = (codes << np.array([0, 2, 4, 6], np.uint8)).sum(axis=1).astype(np.uint8)
        t = torch.full((shift + len(packed),), 255, dtype=torch.uint8, device="cuda")
        t[shift:] = torch.from_numpy(packed).cuda()
        off = np.concatenate([[0], np.cumsum([len(q) for q in seqs])])
        return t[shift:], torch.from_numpy(off.astype(np.int64)).cuda()

    reads, refs = pairs_of(4100, 77, [70, 41, 64, 133], [90, 64, 150])
    with ga.Context(0) as ctx:
        want, _ = ctx.align(reads, refs, 64)
        (r, ro), (f, fo) = stream(reads), stream(refs)
        out, _ = ctx.align_dev(r, ro, f, fo, 64)
        torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(-1).view(ga.RESULT_DTYPE)
    for field in ("edit_distance", "ref_begin", "ref_end", "n_windows", "flags"):
        assert (got[field] == want[field]).all(), field


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
