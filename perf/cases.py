"""The aligner's performance cases: the calls a program that uses it makes,
through the public entry points, from a handful of short reads to the largest
batches of long ones.

Inputs are synthetic and drawn on the GPU from the seed alone: i.i.d. bases,
a reference of flank + segment + flank per pair and a read that is the segment
with random substitutions, insertions and deletions (indel lengths geometric),
the recipe of workloads/gen.py in vectorised form. A decoy pair's reference is
unrelated to its read, as a mapper's wrong candidate location is.

A case's fields:
  path     align (device form), host (host-memory form), filter, serve
  pairs    reads per call (requests per pass for serve)
  bases    segment length; with `sigma` > 0 the median of a log-normal length
           (clipped to [100, 30,000])
  error    edit events per base; `spread` draws each read's rate from
           [error / 15, error] instead
  sub, ins the shares of substitutions and insertions (the rest: deletions)
  mean     mean length of an insertion or deletion
  flank    reference bases on either side of the segment
  decoy    share of decoy pairs
  k, W, O  error cap, window, overlap
  form     batched or plain launch of the device form
  pack     the call starts from ASCII bases in device memory (pack, then align)
"""
import math

import numpy as np
import torch

import paper_2203_15561_amd as ga

# substitution and insertion shares of short-read, long-read and even error models
SHORT_MIX = dict(sub=0.90, ins=0.05, mean=1.0)
LONG_MIX = dict(sub=0.15, ins=0.50, mean=1.0 / 0.7)
EVEN_MIX = dict(sub=1 / 3, ins=1 / 3, mean=1.0)
MIXES = {"short": SHORT_MIX, "long": LONG_MIX, "even": EVEN_MIX}


def _case(name, path, pairs, bases, error, mix, flank, k, *, sigma=0.0, spread=False, decoy=0.0,
          W=64, O=24, form="batched", pack=False):
    c = dict(path=path, pairs=pairs, bases=bases, sigma=sigma, error=error, spread=spread,
             flank=flank, decoy=decoy, k=k, W=W, O=O, form=form, pack=pack, **MIXES[mix])
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # an interactive or per-read call: a few short reads, all latency
        _case("align_4x150", "align", 4, 150, 0.01, "short", 20, 15),
        # a small batch of short reads (the 100 bp configuration)
        _case("align_1000x100", "align", 1000, 100, 0.05, "even", 10, 10),
        # a sequencer tile's worth of short reads (the 250 bp configuration)
        _case("align_100000x250", "align", 100_000, 250, 0.02, "short", 20, 15),
        # the headline batch: 10 kb reads at 10% error with decoy locations,
        # from ASCII bases in device memory
        _case("align_20000x10k", "align", 20_000, 10_000, 0.10, "long", 500, 64, decoy=0.3, pack=True),
        # reads of very different lengths in one batch
        _case("align_50000_uneven", "align", 50_000, 2000, 0.15, "long", 50, 64, sigma=1.0, spread=True),
        # a few very long reads: too few pairs to fill the chip
        _case("align_67x30k", "align", 67, 30_000, 0.10, "long", 500, 64),
        # the one-kernel launch form, used for small batches
        _case("plain_256x150", "align", 256, 150, 0.01, "short", 20, 15, form="plain"),
        # pre-alignment filter ahead of short-read alignment, some candidates wrong
        _case("filter_20000x250", "filter", 20_000, 250, 0.02, "short", 20, 15, decoy=0.3),
        # the filter near its longest reads
        _case("filter_4000x1000", "filter", 4000, 1000, 0.03, "even", 40, 50, decoy=0.3),
        # the synchronous host call: ASCII in, CIGAR text out
        _case("host_1000x1000", "host", 1000, 1000, 0.05, "long", 50, 64),
        # the serving loop: a burst of mixed requests (70% of 150 bp, 30% of 1-30 kb)
        _case("serve_1024_mixed", "serve", 1024, 30_000, 0.10, "long", 500, 64),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["short", "short", "long", "long", "uneven", "few", "plain", "filter", "host", "serve"])
    if kind == "short":
        bases = log(60, 400)
        return _case(None, "align", log(2, 100_000), bases, rng.uniform(0.005, 0.06),
                     rng.choice(["short", "even"]), rng.randint(0, 40), rng.choice([10, 15, 32]),
                     decoy=rng.choice([0.0, 0.1]), O=rng.choice([24, 24, 32]))
    if kind == "long":
        bases = log(1000, 20_000)
        return _case(None, "align", log(100, max(200, 150_000_000 // bases)), bases,
                     rng.uniform(0.03, 0.15), "long", rng.randint(20, 600), 64,
                     decoy=rng.choice([0.0, 0.3, 0.6]), O=rng.choice([24, 24, 32]), pack=rng.random() < 0.5)
    if kind == "uneven":
        return _case(None, "align", log(500, 50_000), log(400, 2000), rng.uniform(0.05, 0.15), "long",
                     rng.randint(20, 200), 64, sigma=rng.uniform(0.5, 1.0), spread=True)
    if kind == "few":
        return _case(None, "align", log(1, 300), log(5000, 30_000), rng.uniform(0.05, 0.15), "long",
                     rng.randint(50, 600), 64, decoy=rng.choice([0.0, 0.2]))
    if kind == "plain":
        return _case(None, "align", log(1, 2000), log(60, 400), rng.uniform(0.005, 0.05), "short",
                     rng.randint(5, 40), 15, form="plain")
    if kind == "filter":
        return _case(None, "filter", log(100, 20_000), log(50, 900), rng.uniform(0.01, 0.06),
                     rng.choice(["short", "even"]), rng.randint(5, 60), rng.choice([5, 15, 40, 60]),
                     decoy=rng.choice([0.0, 0.3, 0.6]))
    if kind == "host":
        bases = log(100, 5000)
        return _case(None, "host", log(10, max(20, 4_000_000 // bases)), bases, rng.uniform(0.01, 0.12),
                     "long", rng.randint(10, 100), 64)
    return _case(None, "serve", log(64, 1024), 30_000, rng.uniform(0.05, 0.12), "long", 500, 64)


# Inputs -----------------------------------------------------------------------

def _pairs(case, seed):
    """Base codes and offsets of the case's reads and references, on the GPU."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    n = case["pairs"]

    def rand(*shape):
        return torch.rand(*shape, device=dev, generator=g)

    def bases(count):
        return torch.randint(0, 4, (count,), device=dev, generator=g, dtype=torch.uint8)

    flank = torch.full((n,), case["flank"], device=dev, dtype=torch.int64)
    rate = torch.full((n,), case["error"], device=dev)
    if case["spread"]:
        rate = case["error"] * (1 + 14 * rand(n)) / 15
    sub, ins, mean = case["sub"], case["ins"], case["mean"]
    if case["path"] == "serve":
        short = rand(n) < 0.7
        length = (1000 + rand(n) * (case["bases"] - 999)).long()
        length = torch.where(short, torch.full_like(length, 150), length)
        flank = torch.where(short, torch.full_like(flank, 20), flank)
        rate = torch.where(short, torch.full_like(rate, 0.01), rate)
    elif case["sigma"] > 0:
        z = torch.randn(n, device=dev, generator=g)
        length = (case["bases"] * torch.exp(case["sigma"] * z)).round().long().clamp(100, 30_000)
    else:
        length = torch.full((n,), case["bases"], device=dev, dtype=torch.int64)
    decoy = rand(n) < case["decoy"]
    zero = torch.zeros(1, device=dev, dtype=torch.int64)
    ref_len = length + 2 * flank
    ref_off = torch.cat([zero, ref_len.cumsum(0)])
    refs = bases(int(ref_off[-1]))

    # blocks of pairs, so that the per-base arrays stay small
    reads, read_len = [], []
    total = int(length.sum())
    step = max(1, int(n * 32_000_000 // max(total, 1)))
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        seg_len = length[lo:hi]
        seg_off = torch.cat([zero, seg_len.cumsum(0)])
        count = int(seg_off[-1])
        pair = torch.repeat_interleave(torch.arange(hi - lo, device=dev), seg_len)
        at = torch.arange(count, device=dev)
        where = ref_off[lo:hi][pair] + flank[lo:hi][pair] + (at - seg_off[pair])
        seg = torch.where(decoy[lo:hi][pair], bases(count), refs[where])
        # one event per base at most: a substitution, an insertion before the
        # base, or a deletion from it on
        per = sub + (1 - sub) * mean
        event = rand(count) < (rate[lo:hi] / per)[pair]
        kind = rand(count)
        extent = torch.ones(count, device=dev, dtype=torch.int64)
        if mean > 1:
            extent += (torch.log(rand(count).clamp_min(1e-7)) / math.log(1 - 1 / mean)).floor().long().clamp(0, 30)
        is_sub = event & (kind < sub)
        is_ins = event & (kind >= sub) & (kind < sub + ins)
        is_del = event & (kind >= sub + ins)
        seg = torch.where(is_sub, (seg + torch.randint(1, 4, (count,), device=dev, generator=g, dtype=torch.uint8)) & 3, seg)
        reach = torch.cummax(torch.where(is_del, at + extent, zero), 0).values
        made = (at >= reach).long() + torch.where(is_ins, extent, zero)
        end = made.cumsum(0)
        out = torch.repeat_interleave(seg, made)
        # the last base of an insertion's run is the kept base; the ones before it are new
        pos = torch.arange(out.numel(), device=dev)
        last = torch.repeat_interleave(end - 1, made)
        out = torch.where(pos == last, out, bases(out.numel()))
        reads.append(out)
        total_end = torch.cat([zero, end])
        read_len.append(total_end[seg_off[1:]] - total_end[seg_off[:-1]])
    read_off = torch.cat([zero, torch.cat(read_len).cumsum(0)])
    return torch.cat(reads), read_off, refs, ref_off


def _packed(codes):
    pad = (-codes.numel()) % 4
    q = torch.cat([codes, torch.zeros(pad, dtype=torch.uint8, device=codes.device)]).view(-1, 4)
    return (q[:, 0] | (q[:, 1] << 2) | (q[:, 2] << 4) | (q[:, 3] << 6)).contiguous()


def _ascii(codes):
    return torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device=codes.device)[codes.long()]


def _mean_bases(case):
    if case["path"] == "serve":
        return 0.7 * 150 + 0.3 * (1000 + case["bases"]) / 2
    return case["bases"] * math.exp(case["sigma"] ** 2 / 2)


def _room(case):
    """Read bases (and reference bases) the program makes room for: its output
    buffers are allocated once for batches of this shape, whatever the reads
    turn out to be."""
    per = 1.7 if case["sigma"] > 0 else 1.25
    return int(case["pairs"] * (per * _mean_bases(case) + 2 * case["flank"] + 64)) + 4096


def prepare(case, seed):
    reads, read_off, refs, ref_off = _pairs(case, seed)
    n, dev, room = case["pairs"], reads.device, _room(case)
    st = dict(case=case, ctx=ga.Context(0), nr=int(read_off[-1]), nf=int(ref_off[-1]))
    if max(st["nr"], st["nf"]) > room and case["path"] != "serve":
        raise RuntimeError("more bases than the case makes room for")
    if case["path"] == "host":
        st.update(r=_ascii(reads).cpu().numpy().tobytes(), f=_ascii(refs).cpu().numpy().tobytes(),
                  ro=read_off.cpu().numpy().astype(np.uint64), fo=ref_off.cpu().numpy().astype(np.uint64),
                  text=np.zeros(room, dtype=np.uint8))
        return st
    if case["path"] == "serve":
        st.update(r=_packed(reads).cpu().numpy(), f=_packed(refs).cpu().numpy(),
                  ro=read_off.cpu().numpy().astype(np.uint64), fo=ref_off.cpu().numpy().astype(np.uint64),
                  tags=np.arange(n, dtype=np.uint64), runs=np.zeros((n, case["bases"]), dtype=np.uint32),
                  srv=ga.Server(st["ctx"], case["k"], case["W"], case["O"], cigar_runs=1, max_pending=n + 1))
        return st
    st.update(ro=read_off, fo=ref_off)
    if case["path"] == "filter":
        st.update(r=_packed(reads), f=_packed(refs), longest=int((read_off[1:] - read_off[:-1]).max()),
                  dist=torch.zeros(n, dtype=torch.int32, device=dev),
                  start=torch.zeros(n, dtype=torch.int32, device=dev))
        return st
    st.update(out=torch.zeros((n, 32), dtype=torch.uint8, device=dev),
              cigar=torch.zeros(2 * room, dtype=torch.int32, device=dev),
              launch=ga.make_launch(ga.FORM_PLAIN) if case["form"] == "plain" else None)
    if case["pack"]:
        st.update(ra=_ascii(reads), fa=_ascii(refs), bad=torch.zeros(1, dtype=torch.int32, device=dev),
                  r=torch.zeros(room // 4 + 1, dtype=torch.uint8, device=dev),
                  f=torch.zeros(room // 4 + 1, dtype=torch.uint8, device=dev))
    else:
        st.update(r=_packed(reads), f=_packed(refs))
    return st


def run(st):
    c, ctx = st["case"], st["ctx"]
    if c["path"] == "host":
        out, text = ctx.align_buffers(st["r"], st["ro"], st["f"], st["fo"], c["k"], c["W"], c["O"])
        st["text"][:len(text)] = np.frombuffer(text, dtype=np.uint8)
        return out.view(np.uint8), st["text"]
    if c["path"] == "serve":
        return _serve(st)
    if c["path"] == "filter":
        return ctx.filter_dev(st["r"], st["ro"], st["f"], st["fo"], c["k"], st["longest"],
                              dist=st["dist"], start=st["start"])
    if c["pack"]:
        ctx.pack_dev(st["ra"], st["r"], st["bad"])
        ctx.pack_dev(st["fa"], st["f"], st["bad"])
    out, cigar = ctx.align_dev(st["r"], st["ro"], st["f"], st["fo"], c["k"], c["W"], c["O"],
                               launch=st["launch"], out=st["out"], cigar=st["cigar"],
                               total_read_bases=st["nr"], total_ref_bases=st["nf"])
    return (out, cigar, st["r"], st["f"], st["bad"]) if c["pack"] else (out, cigar)


def _serve(st):
    """Submits the burst and takes every completion, by tag."""
    srv, n = st["srv"], st["case"]["pairs"]
    rc, taken = srv.submit_batch(st["r"], st["ro"], st["f"], st["fo"], st["tags"])
    if rc or taken != n:
        raise RuntimeError("serving: burst refused (%d, %d)" % (rc, taken))
    results, runs, done = np.zeros(n, dtype=ga.RESULT_DTYPE), st["runs"], 0
    while done < n:
        info, elems = srv.poll_arrays(timeout_ms=1000)
        tags = info["tag"].astype(np.int64)
        results[tags] = info["result"]
        first = info["result"]["cigar_off"].astype(np.int64)
        last = first + info["result"]["cigar_len"]
        for t, a, b in zip(tags.tolist(), first.tolist(), last.tolist()):
            runs[t, :b - a] = elems[a:b]
        done += len(tags)
    fields = {f: results[f] for f in ("edit_distance", "ref_begin", "ref_end", "n_windows", "cigar_len", "flags")}
    return fields, runs


# What a pass cannot do without --------------------------------------------------

def work(case):
    """Bytes: each packed base (ASCII where the call starts from it) and offset
    read once, each result and CIGAR run written once. Operations: the dynamic
    programming cells of the path at 64 cells per step of a bit-vector
    recurrence on vertical differences (17 operations on 64-bit words, the
    published form for approximate matching, so 34 of 32 bits)."""
    n = case["pairs"]
    m = _mean_bases(case)
    ref = m + 2 * case["flank"]
    per_base = 1.0 if case["path"] == "host" or case["pack"] else 0.25
    ops = 34 / 64
    if case["path"] == "filter":
        return {"bytes": n * ((m + ref) * per_base + 24), "flops": n * m * ref * ops}
    rate = case["error"] * (8 / 15 if case["spread"] else 1.0)
    runs = 2 * rate * m * (1 - case["decoy"]) + 0.9 * m * case["decoy"] + 1
    windows = max(1.0, m / (case["W"] - case["O"]))
    cells = windows * case["W"] * case["W"] + case["W"] * ref
    return {"bytes": n * ((m + ref) * per_base + 16 + 32 + 4 * runs), "flops": n * cells * ops}


def exact(case, seed):
    """The filter's distances and starts by the textbook dynamic program. The
    alignments have no such form (the windows' and ties' rules are the
    library's own, pinned by the tests' oracle)."""
    if case["path"] != "filter":
        return None
    reads, read_off, refs, ref_off = _pairs(case, seed)
    dev, n, k = reads.device, case["pairs"], case["k"]
    m, t = read_off[1:] - read_off[:-1], ref_off[1:] - ref_off[:-1]
    M, T = int(m.max()), int(t.max())
    # read bases from the last one back; column j of `d` is the distance of the
    # last j read bases to the best prefix of the reference from column i on
    j = torch.arange(M, device=dev)
    back = (read_off[1:, None] - 1 - j).clamp_min(0)
    read = torch.where(j < m[:, None], reads[back].long(), 9)
    ramp = torch.arange(M + 1, device=dev)
    d = ramp.repeat(n, 1)
    best, start = m.clone(), t.clone()
    for i in range(T - 1, -1, -1):
        live = i < t
        base = refs[(ref_off[:-1] + i).clamp_max(refs.numel() - 1)].long()
        new = d + 1
        new[:, 0] = 0
        new[:, 1:] = torch.minimum(new[:, 1:], d[:, :-1] + (read != base[:, None]))
        new = torch.cummin(new - ramp, 1).values + ramp
        d = torch.where(live[:, None], new, d)
        here = d.gather(1, m[:, None])[:, 0]
        hit = live & (here <= best)
        best, start = torch.where(hit, here, best), torch.where(hit, i, start)
    ok = best <= k
    return (torch.where(ok, best, -1), torch.where(ok, start, 0))
