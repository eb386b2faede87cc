"""The kernels that take one pair per lane (csrc/lanes.h): under the CPU
emulation with its sanitizers at launches of few workgroups, so that a
workgroup takes several rounds of pairs, and on the GPU through the launch
fields that lead there."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
import paper_2203_15561_amd as ga
from tests.emu import run as emu
from tests.test_pair_paths import expected_of, pairs_of
from workloads import gen


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return emu.build(str(tmp_path_factory.mktemp("emu") / "emu_driver"))


@pytest.fixture(scope="module")
def debug_driver(tmp_path_factory):
    return emu.build(str(tmp_path_factory.mktemp("emu") / "emu_driver_debug"), debug=True)


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
    # 200 pairs on two workgroups of 32 lanes: four rounds
    ps = gen.from_lists("rounds", *rounds_of_pairs(200, 71), k)
    want = expected_of(ps)
    for alone in (0, 1):
        got = results(*emu.run(driver, ps, emu.LANES, pair_lanes=32, window_blocks=2, alone=alone))
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


def long_references(n, seed, ref_len, at):
    """n pairs, every reference of pairs_of but those of `at`: of the given
    lengths, with the read in their last bases (or nowhere)."""
    reads, refs = pairs_of(n, seed, [50, 70, 0, 1], [90, 0, 64])
    for i, m in zip(at, ref_len):
        refs[i] = gen.random_bases(gen.pair_rng(seed + 1, i), m)
        reads[i] = gen.random_bases(gen.pair_rng(seed + 2, i), 55)
        if i % 3:
            refs[i][-60:-5] = reads[i]
    return reads, refs


@pytest.mark.slow
def test_long_references_emulated(driver):
    # references around a pair's own 1,024 columns and the chunks after them, next
    # to each other and apart, in both paths, and the same without a limit
    lengths = [1024, 1025, 2048, 2049, 2047, 3100, 4096, 5000]
    reads, refs = long_references(30, 81, lengths, [0, 4, 5, 6, 13, 20, 28, 29])
    reads[20] = reads[20][:0]
    for k in (64, 2):
        ps = gen.from_lists("long", reads, refs, k)
        want = expected_of(ps)
        for own in (1024, 0):
            assert results(*emu.run(driver, ps, 0, own_cols=own)) == want, (k, own)
            assert results(*emu.run(driver, ps, emu.LANES, pair_lanes=32, own_cols=own)) == want, (k, own)
        assert results(*emu.run(driver, ps, emu.LANES, pair_lanes=32, search_parts_log=1, own_cols=512)) == want, k


def mixed_batch(n, seed, longest=400):
    """Pairs of pairs_of around the windows' edges, every 16th read long."""
    reads, refs = pairs_of(n, seed, [150, 0, 39, 40, 41, 64, 65, 104, 81], [170, 64, 0, 129, 250, 90])
    for i in range(0, n, 16):
        rng = gen.pair_rng(seed + 1, i)
        reads[i] = gen.random_bases(rng, longest)
        refs[i] = gen.mutate(rng, reads[i], 0.1, (0.15, 0.5, 0.35)) if i % 48 else gen.random_bases(rng, longest)
    return reads, refs


@pytest.mark.slow
@pytest.mark.parametrize("W,O,k", [(64, 24, 64), (64, 24, 5), (33, 9, 64), (8, 7, 3)])
def test_batches_emulated(driver, debug_driver, W, O, k):
    # several rounds of full and part wavefronts, the longest pairs on wavefronts of
    # their own, several search parts a pair; the debug build's checks and its audit
    # that every pair is taken once
    ps = gen.from_lists("mixed", *mixed_batch(72, 51), k, W, O)
    want = expected_of(ps)
    for kw in (dict(pair_lanes=8, window_blocks=3, alone=1), dict(pair_lanes=64, long_pairs=5, long_bases=200),
               dict(pair_lanes=16, long_pairs=3, long_bases=200, search_parts_log=2)):
        for build in (driver, debug_driver):
            assert results(*emu.run(build, ps, emu.LANES, **kw)) == want, kw


@pytest.mark.slow
@pytest.mark.parametrize("slots,admit", [(3, 2), (20, 20), (60, 60)])
@pytest.mark.parametrize("budget,ticks", [(0, 40), (2, 0)])
def test_serving_emulated(driver, slots, admit, budget, ticks):
    # few resident pairs, a wavefront each (up to two a workgroup; with small windows
    # up to sixteen, one after the other), and more, a lane each; turns that end by
    # time and by windows
    reads, refs = mixed_batch(min(slots, 40) + 11, 52, 300)
    for k, W, O in ((64, 64, 24), (5, 16, 8), (8, 8, 3)):
        ps = gen.from_lists("serve", reads, refs, k, W, O)
        got = results(*emu.run(driver, ps, emu.SERVE_LANES, window_blocks=2, slots=slots, admit_per_iteration=admit,
                               window_budget=budget, ticks=ticks, search_chunk=64))
        assert got == expected_of(ps), (k, W, O)


@pytest.mark.gpu
def test_launch_fields_and_counters_of_lanes():
    # a batch too large for a wavefront a pair: the launch fields that keep it on
    # lanes, and the work counters against the oracle's
    reads, refs = mixed_batch(4600, 53, 3000)
    ps = gen.from_lists("mixed", reads, refs, 64)
    res_o, _, _, _ = oracle.batch(ps)
    want = expected_of(ps)
    with ga.Context(0) as ctx:
        for kw in ({}, dict(workers_per_cu=1), dict(lpt_order=0), dict(workers_per_cu=2, lpt_order=0)):
            ctx.profile(1)
            got = results(*ctx.align(reads, refs, 64, launch=ga.make_launch(ga.FORM_BATCHED, **kw)))
            p = ctx.profile_read()
            assert got == want, kw
            # two wavefronts a workgroup, not the row tables' resident grid
            assert 0 < p["window_workgroups"] <= 256 * (kw.get("workers_per_cu") or 4), kw
            for name, field in (("window_cells", "cells_window"), ("search_cells", "cells_search"), ("windows", "n_windows"),
                                ("window_word_ops", "word_ops"), ("table_words", "words_stored")):
                assert p[name] == int(res_o[field].sum()), (kw, name)
            ctx.profile(0)
            assert results(*ctx.align(reads, refs, 64, launch=ga.make_launch(ga.FORM_BATCHED, **kw))) == want, kw


CHILD = r"""
import paper_2203_15561_amd as ga
from paper_2203_15561_amd import capi
from tests.test_lane_kernels import mixed_batch, results, rounds_of_pairs
from tests.test_pair_paths import expected_of
from workloads import gen

assert capi.LIB_PATH.endswith("libgenasm_debug.so"), capi.LIB_PATH
with ga.Context(0) as ctx:
    for name, (reads, refs) in (("mixed", mixed_batch(4600, 54, 2000)), ("one window", rounds_of_pairs(17_000, 55))):
        want = expected_of(gen.from_lists(name, reads, refs, 64))
        for kw in ({}, dict(workers_per_cu=1), dict(lpt_order=0)):
            print("debug build:", name, kw, flush=True)
            assert results(*ctx.align(reads, refs, 64, launch=ga.make_launch(ga.FORM_BATCHED, **kw))) == want
print("all clean", flush=True)
"""


@pytest.mark.gpu
def test_debug_build_on_lanes():
    # every pair taken by exactly one lane or wavefront (flags are 0 in results())
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-u", "-c", CHILD], cwd=root, env=dict(os.environ, GENASM_LIB_VARIANT="debug"),
                       timeout=100, capture_output=True, text=True)
    assert r.returncode == 0 and "all clean" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("n", [3, 2000, 3000])
def test_long_references(n):
    # references of more than 131,072 columns (a wavefront's own) and of many times
    # the mean (a lane's parts): results, several calls, a captured call, and no
    # slower than the row tables' search, which cuts all references alike
    import torch

    lengths = [131_072, 131_073, 400_000, 132_000 if n == 3 else 1_500_000]
    at = [0, 1, 2] if n == 3 else [1, 2, n // 2, n - 1]
    reads, refs = long_references(n, 82, lengths[-len(at):], at)
    ps = gen.from_lists("long", reads, refs, 20)
    want = expected_of(ps)
    with ga.Context(0) as ctx:
        for _ in range(2):
            assert results(*ctx.align(reads, refs, 20)) == want
        r, f = torch.from_numpy(emu.pack2b(ps.reads)).cuda(), torch.from_numpy(emu.pack2b(ps.refs)).cuda()
        ro, fo = (torch.from_numpy(x.astype(np.int64)).cuda() for x in (ps.read_off, ps.ref_off))
        out, cig = ctx.align_dev(r, ro, f, fo, 20)
        nr, nf = len(ps.reads), len(ps.refs)

        def call(launch=None):
            ctx.align_dev(r, ro, f, fo, 20, launch=launch, out=out, cigar=cig, total_read_bases=nr, total_ref_bases=nf)

        def same():
            got = out.cpu().numpy().reshape(-1).view(ga.RESULT_DTYPE)
            return all((int(g["edit_distance"]), int(g["ref_begin"]), int(g["ref_end"])) == (w[0], w[2], w[3])
                       for g, w in zip(got, want))

        def ms(launch):
            times = []
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                call(launch)
                b.record()
                b.synchronize()
                times.append(a.elapsed_time(b))
            return min(times)

        assert same()
        for _ in range(2):
            out.zero_()
            ctx.align_dev(r, ro, f, fo, 20, out=out, cigar=cig, total_read_bases=nr, total_ref_bases=nf, noalloc=True)
            assert same()
        here, tables = ms(None), ms(ga.make_launch(ga.FORM_BATCHED, search_per_cu=4))
        assert here < 1.5 * tables, (here, tables)
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.align_dev(r, ro, f, fo, 20, out=out, cigar=cig, total_read_bases=nr, total_ref_bases=nf,
                          stream=stream.cuda_stream)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert same()
            call()
            torch.cuda.synchronize()
            assert same()
        del graph
        ctx.unpin()


@pytest.mark.gpu
def test_long_reference_first_seen_in_capture():
    # the slots for long references can't be allocated then: the same results without
    import torch

    reads, refs = long_references(500, 83, [300_000, 140_000], [7, 400])
    ps = gen.from_lists("long", reads, refs, 20)
    want = [(w[0], w[2], w[3]) for w in expected_of(ps)]
    r, f = torch.from_numpy(emu.pack2b(ps.reads)).cuda(), torch.from_numpy(emu.pack2b(ps.refs)).cuda()
    ro, fo = (torch.from_numpy(x.astype(np.int64)).cuda() for x in (ps.read_off, ps.ref_off))
    nr, nf = len(ps.reads), len(ps.refs)
    out = torch.zeros((500, 32), dtype=torch.uint8, device="cuda")
    cig = torch.zeros(nr + nf, dtype=torch.int32, device="cuda")
    with ga.Context(0) as ctx:
        ctx.align(reads[:3], refs[:3], 20)
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.align_dev(r, ro, f, fo, 20, out=out, cigar=cig, total_read_bases=nr, total_ref_bases=nf,
                          stream=stream.cuda_stream)
        for _ in range(2):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            got = out.cpu().numpy().reshape(-1).view(ga.RESULT_DTYPE)
            assert [(int(g["edit_distance"]), int(g["ref_begin"]), int(g["ref_end"])) for g in got] == want
        del graph
        ctx.unpin()


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


@pytest.mark.gpu
@pytest.mark.parametrize("W,O", [(8, 3), (2, 0), (9, 3)])
def test_serving_small_windows(W, O):
    # more resident pairs than wavefronts, and than eight times as many
    reads, refs = mixed_batch(10_000, 95, 700)
    ps = gen.from_lists("serve", reads, refs, W, W, O)
    want = expected_of(ps)
    with ga.Context(0) as ctx, ga.Server(ctx, W, W, O, cigar_runs=1, max_pending=10_001) as srv:
        for n in (1500, 10_000):
            rc, taken = srv.submit_batch(ga.pack(ps.reads), ps.read_off[:n + 1].astype(np.uint64), ga.pack(ps.refs),
                                         ps.ref_off[:n + 1].astype(np.uint64), np.arange(n, dtype=np.uint64))
            assert rc == 0 and taken == n
            done = 0
            while done < n:
                info, elems = srv.poll_arrays(timeout_ms=1000)
                for i in info:
                    r, at = i["result"], int(i["result"]["cigar_off"])
                    cigar = ga.decode_cigar(elems[at:at + int(r["cigar_len"])])
                    assert (int(r["edit_distance"]), cigar, int(r["ref_begin"]), int(r["ref_end"]),
                            int(r["n_windows"])) == want[int(i["tag"])], int(i["tag"])
                done += len(info)


@pytest.mark.gpu
@pytest.mark.parametrize("W,O,k", [(2, 1, 1), (2, 0, 2), (4, 2, 4), (8, 7, 3), (8, 3, 8), (16, 8, 16), (32, 31, 3)])
def test_small_windows_no_slower_than_row_tables(W, O, k):
    # 6,000 even pairs and 6,000 uneven ones: results and times against the row tables
    import torch

    def times(ctx, args, kw, launch):
        best = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ctx.align_dev(*args, launch=launch, **kw)
            b.record()
            b.synchronize()
            best.append(a.elapsed_time(b))
        return min(best)

    rng = np.random.default_rng(W * 100 + O)
    for spread in (0.0, 1.0):
        lens = np.clip(300 * np.exp(spread * rng.normal(0, 1, 6000)), 1, 2400).astype(int)
        ref_off = np.concatenate([[0], np.cumsum(lens + 20)])
        read_off = np.concatenate([[0], np.cumsum(lens)])
        refs = rng.integers(0, 4, ref_off[-1]).astype(np.uint8)
        reads = np.concatenate([refs[a + 10:a + 10 + m] for a, m in zip(ref_off, lens)])
        reads = np.where(rng.random(len(reads)) < 0.02, rng.integers(0, 4, len(reads)), reads).astype(np.uint8)
        args = [torch.from_numpy(x).cuda() for x in (emu.pack2b(reads), read_off, emu.pack2b(refs), ref_off)] + [k, W, O]
        outs = [torch.zeros((6000, 32), dtype=torch.uint8, device="cuda") for _ in range(2)]
        cigs = [torch.zeros(len(reads) + len(refs), dtype=torch.int32, device="cuda") for _ in range(2)]
        kws = [dict(out=o, cigar=c, total_read_bases=len(reads), total_ref_bases=len(refs)) for o, c in zip(outs, cigs)]
        with ga.Context(0) as ctx:
            here = times(ctx, args, kws[0], None)
            tables = times(ctx, args, kws[1], ga.make_launch(ga.FORM_BATCHED, search_per_cu=9))
        assert torch.equal(outs[0], outs[1]) and torch.equal(cigs[0], cigs[1])
        assert here < 1.1 * tables, (spread, here, tables)


@pytest.mark.gpu
def test_profile_of_every_path():
    # one pair per wavefront (plain, and a batch of few pairs), one pair per lane with
    # the longest pairs on wavefronts: every pair's cycles and clocks, the workgroups
    few = pairs_of(40, 91, [300, 700], [400, 800])
    many = pairs_of(4500, 92, [60, 90], [80, 110])
    for i in range(0, 4500, 300):  # longer than twice the mean
        many[0][i] = gen.random_bases(gen.pair_rng(93, i), 1200)
        many[1][i] = many[0][i].copy()
    with ga.Context(0) as ctx:
        ctx.profile(1)
        for (reads, refs), form, blocks in ((many, ga.FORM_BATCHED, None), (few, ga.FORM_BATCHED, 40),
                                            (few, ga.FORM_PLAIN, 0), (few, ga.FORM_UNIMPROVED, 0)):
            res, _ = ctx.align(reads, refs, 64, launch=ga.make_launch(form))
            p, w = ctx.profile_read(), ctx.profile_pairs()
            word = dict(zip(ctx.PROFILE_FIELDS, w.T))
            assert (word["windows"] == res["n_windows"]).all() and p["windows"] == int(res["n_windows"].sum())
            assert p["window_workgroups"] == blocks if blocks is not None else 0 < p["window_workgroups"] < 4500
            if form == ga.FORM_UNIMPROVED:
                continue
            ran = res["n_windows"] > 0
            for name in ("dc_cycles", "tb_cycles", "start_clock"):
                assert (word[name][ran] > 0).all(), (len(reads), form, name)
            assert (word["pair_cycles"][ran] >= word["dc_cycles"][ran]).all()
            assert (word["end_clock"][ran] >= word["start_clock"][ran]).all()
        # a call without profiling leaves the last profiled call's figures
        want = ctx.profile_read()
        ctx.profile(0)
        ctx.align(*many, 64)
        ctx.profile(1)
        assert ctx.profile_read()["window_workgroups"] == want["window_workgroups"]
