"""The calls whose speed counts, as a user's program makes them.

One case per way the library is used: the whole path (suffix array, LCP array, overlaps) on the
smallest, an ordinary, the large and the repeat-heavy read set; many sets in one batched build;
jobs through the server; pattern lookup, few and many; the skew construction; the radix sort by
itself; overlaps on both strands; and reconstruction from two cuttings.  Sizes are those of the
repository's workloads (synth.py, bench.py) or lie between them.  Inputs are drawn on the GPU
from the seed alone with the generators' distributions: i.i.d. genomes (the repeat-heavy ones
with synth.repeat_genome's repeats), reads at uniform starts, substitutions.

Every output is a whole number (positions, ranks, lengths, read ids, sorted keys), so there is
nothing for exact() to say: the arrays are unique and have to be equal.
"""
from __future__ import annotations

import math
import time

import numpy as np
import torch

import paper_1404_3456_amd as pkg
from paper_1404_3456_amd import synth

_ASCII = (65, 67, 71, 84)  # A C G T
_SEP = 36                  # $


# ---- the cases ------------------------------------------------------------------------------

def listed():
    return [
        # a small set, error-free (plain-small-20k): launches and latency decide
        {"name": "path-small", "kind": "path", "genome": 20_000, "reads": 400, "lo": 200,
         "hi": 200, "err": 0.0, "min_len": 30, "repeats": False},
        # the middle of the serving sizes, one job by itself: ragged reads, 8x, odd length
        {"name": "path-job", "kind": "path", "genome": 70_711, "reads": 1191, "lo": 150,
         "hi": 800, "err": 0.005, "min_len": 40, "repeats": False},
        # a bacterial genome at 10x (plain-large-5M, the benchmark's step)
        {"name": "path-large", "kind": "path", "genome": 5_000_000, "reads": 100_000, "lo": 500,
         "hi": 500, "err": 0.005, "min_len": 40, "repeats": False},
        # repeats and tandem arrays (repeat-stress-40M): large groups in every round
        {"name": "path-repeats", "kind": "path", "genome": 40_000_000, "reads": 400_000,
         "lo": 1000, "hi": 1000, "err": 0.01, "min_len": 100, "repeats": True},
        # many independent sets in one build (a quarter of batched-256), with LCP and overlaps
        {"name": "batch-sets", "kind": "batch", "sets": 64, "g_lo": 10_000, "g_hi": 2_000_000,
         "lo": 100, "hi": 1000, "cov_lo": 5.0, "cov_hi": 20.0, "err": 0.005, "min_len": 40},
        # jobs of the serving stream through the job server: host texts in, results out
        {"name": "serve-jobs", "kind": "serve", "jobs": 32, "g_lo": 1_000, "g_hi": 5_000_000,
         "lo": 150, "hi": 800, "cov_lo": 8.0, "cov_hi": 8.0, "err": 0.005, "min_len": 40},
        # a million 40-base queries against the large text
        {"name": "lookup-many", "kind": "lookup", "genome": 5_000_000, "reads": 100_000,
         "read": 500, "patterns": 1_000_000, "p_lo": 40, "p_hi": 40},
        # a few ragged queries, empty ones among them, against a small text
        {"name": "lookup-few", "kind": "lookup", "genome": 20_000, "reads": 400, "read": 200,
         "patterns": 1001, "p_lo": 0, "p_hi": 80},
        # the skew construction on a fifth of the large workload
        {"name": "skew", "kind": "skew", "genome": 1_000_000, "reads": 20_000, "lo": 500,
         "hi": 500, "err": 0.005},
        # the radix sort alone: an odd number of pairs by 52 of 64 key bits
        {"name": "sort-pairs", "kind": "sort", "pairs": 20_000_003, "bit_lo": 0, "bit_hi": 52},
        # both strands: error-free reads of either strand, a fifth of the benchmark's
        {"name": "both-strands", "kind": "strands", "genome": 1_000_000, "reads": 20_000,
         "lo": 500, "hi": 500, "min_len": 40},
        # a sequence cut twice, put together again (index on the GPU, search on the host)
        {"name": "reconstruct", "kind": "reconstruct", "length": 5_000_000, "mean": 500,
         "gap": 32},
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi], odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["path", "path", "path", "batch", "serve", "lookup", "lookup", "skew",
                       "sort", "strands", "reconstruct"])
    if kind == "path":
        repeats = rng.random() < 0.25
        g = _log(rng, 100_000, 20_000_000) if repeats else _log(rng, 10_000, 10_000_000)
        hi = rng.randint(150, 1000)
        lo = hi if rng.random() < 0.4 else rng.randint(100, hi)
        cov = rng.uniform(4.0, 12.0)
        return {"kind": "path", "genome": g, "reads": max(2, int(cov * g * 2 / (lo + hi))),
                "lo": lo, "hi": hi, "err": rng.choice([0.0, 0.005, 0.01]),
                "min_len": rng.randint(30, 100), "repeats": repeats}
    if kind == "batch":
        return {"kind": "batch", "sets": rng.randint(2, 64), "g_lo": 10_000,
                "g_hi": _log(rng, 50_000, 2_000_000), "lo": 100, "hi": 1000, "cov_lo": 5.0,
                "cov_hi": rng.uniform(6.0, 20.0), "err": 0.005, "min_len": rng.randint(30, 60)}
    if kind == "serve":
        cov = rng.uniform(4.0, 8.0)
        return {"kind": "serve", "jobs": rng.randint(4, 48), "g_lo": 1_000,
                "g_hi": _log(rng, 20_000, 4_000_000), "lo": 150, "hi": rng.randint(200, 800),
                "cov_lo": cov, "cov_hi": cov, "err": 0.005, "min_len": rng.randint(30, 60)}
    if kind == "lookup":
        g = _log(rng, 10_000, 5_000_000)
        read = rng.randint(100, 1000)
        p_lo = rng.randint(0, 60)
        return {"kind": "lookup", "genome": g, "reads": max(2, 10 * g // read), "read": read,
                "patterns": _log(rng, 300, 1_000_000), "p_lo": p_lo,
                "p_hi": p_lo + rng.choice([0, 1, 40])}
    if kind == "sort":
        lo = rng.randint(0, 20)
        return {"kind": "sort", "pairs": _log(rng, 2_000, 50_000_000), "bit_lo": lo,
                "bit_hi": rng.randint(lo + 8, 64)}
    if kind == "reconstruct":
        return {"kind": "reconstruct", "length": _log(rng, 20_000, 5_000_000),
                "mean": rng.randint(200, 1000), "gap": 32}
    g = _log(rng, 10_000, 1_500_000)
    read = rng.randint(150, 800)
    c = {"kind": kind, "genome": g, "reads": max(2, int(rng.uniform(4.0, 12.0) * g / read)),
         "lo": read, "hi": read}
    c.update({"err": 0.005} if kind == "skew" else {"min_len": rng.randint(30, 60)})
    return c


# ---- inputs ---------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2_654_435 + 14_043_456)
    return g


def _genome(gen, g):
    return torch.randint(0, 4, (g,), generator=gen, device="cuda", dtype=torch.uint8)


def _randint(gen, lo, hi, k):
    """k whole numbers of [lo, hi]."""
    return torch.randint(lo, hi + 1, (k,), generator=gen, device="cuda", dtype=torch.int64)


def _lengths(gen, m, lo, hi, g):
    """m lengths spread evenly over [lo, hi], in random order: their sum is the case's."""
    lo, hi = min(lo, g), min(hi, g)
    even = lo + (hi - lo) * torch.arange(m, device="cuda") // max(m - 1, 1)
    return even[torch.randperm(m, generator=gen, device="cuda")]


def _starts(gen, lengths, g):
    u = torch.rand(lengths.numel(), generator=gen, device="cuda", dtype=torch.float64)
    return (u * (g - lengths + 1).double()).long()


def _text(gen, genome, starts, lengths, err=0.0, strands=None):
    """ASCII text of the reads genome[start : start + length], each closed by '$'; a strand of 1
    takes the reverse complement; every base is replaced with probability err."""
    step = lengths + 1
    ends = torch.cumsum(step, 0)
    n = int(ends[-1])
    rel = starts - (ends - step)
    if strands is not None:  # position k of the read is genome[start + length - 1 - k]
        rel = torch.where(strands == 1, starts + lengths - 1 + (ends - step), rel)
    idx = torch.repeat_interleave(rel, step, output_size=n)
    at = torch.arange(n, device="cuda")
    if strands is None:
        idx += at
    else:
        back = torch.repeat_interleave(strands, step, output_size=n)
        idx += at * (1 - 2 * back)
    del at
    codes = genome[idx.clamp_(0, genome.numel() - 1)]
    del idx
    if strands is not None:
        codes = torch.where(back == 1, 3 - codes, codes)
    if err > 0.0:
        hit = torch.rand(n, generator=gen, device="cuda") < err
        other = torch.randint(1, 4, (n,), generator=gen, device="cuda", dtype=torch.uint8)
        codes = (codes + hit * other) & 3
        del hit, other
    lut = torch.tensor(_ASCII, dtype=torch.uint8, device="cuda")
    text = torch.empty(n, dtype=torch.uint8, device="cuda")
    for a in range(0, n, 1 << 26):  # in pieces: the index of a gather takes 4 or 8 bytes a base
        b = min(n, a + (1 << 26))
        text[a:b] = lut[codes[a:b].int()]
    text[ends - 1] = _SEP
    return text


def _read_set(case, seed):
    gen = _gen(seed)
    g = case["genome"]
    if case.get("repeats"):
        scale = g / 40_000_000
        rng = np.random.Generator(np.random.PCG64(int(seed)))
        codes = synth.repeat_genome(rng, g, n_copies=max(1, round(50 * scale)),
                                    n_tandem=max(1, round(2000 * scale)))
        genome = torch.from_numpy(codes).cuda()
    else:
        genome = _genome(gen, g)
    lengths = _lengths(gen, case["reads"], case.get("lo", case.get("read")),
                       case.get("hi", case.get("read")), g)
    strands = None
    if case["kind"] == "strands":
        strands = _randint(gen, 0, 1, case["reads"])
    return _text(gen, genome, _starts(gen, lengths, g), lengths, case.get("err", 0.0), strands)


def _set_sizes(case, count):
    """(genome, reads, shortest, longest) of a case's sets: genome sizes log-uniform (the
    middle of each of `count` equal parts of the range), coverage uniform."""
    ratio = case["g_hi"] / case["g_lo"]
    sizes = []
    for i in range(count):
        g = int(round(case["g_lo"] * ratio ** ((i + 0.5) / count)))
        cov = case["cov_lo"] + (case["cov_hi"] - case["cov_lo"]) * ((i * 0.6180339887) % 1.0)
        lo, hi = min(case["lo"], g), min(case["hi"], g)
        sizes.append((g, max(1, int(cov * g * 2 / (lo + hi))), lo, hi))
    return sizes


def _sets(case, count, seed):
    """Texts of independent sets, in random order."""
    gen = _gen(seed)
    sizes = _set_sizes(case, count)
    texts = []
    for i in torch.randperm(count, generator=gen, device="cuda").tolist():
        g, m, lo, hi = sizes[i]
        lengths = _lengths(gen, m, lo, hi, g)
        texts.append(_text(gen, _genome(gen, g), _starts(gen, lengths, g), lengths, case["err"]))
    return texts


def _patterns(gen, text, case):
    """Half substrings of the text, a quarter read prefixes, a quarter random strings; those
    from the text end before the first separator they would cross."""
    k, n = case["patterns"], text.numel()
    lengths = _randint(gen, case["p_lo"], case["p_hi"], k)
    kind = torch.arange(k, device="cuda") & 3
    ends = torch.nonzero(text == _SEP).flatten()
    start = _randint(gen, 0, n - 1, k)
    which = _randint(gen, 0, ends.numel() - 1, k)
    first = torch.where(which > 0, ends[(which - 1).clamp(min=0)] + 1, torch.zeros_like(which))
    start = torch.where(kind == 2, first, start)
    room = ends[torch.searchsorted(ends, start)] - start
    lengths = torch.where(kind == 3, lengths, torch.minimum(lengths, room))
    off = torch.zeros(k + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(lengths, 0)
    total = int(off[-1])
    src = torch.repeat_interleave(start - off[:-1], lengths, output_size=total)
    src += torch.arange(total, device="cuda")
    buf = text[src.clamp_(0, n - 1)]
    lut = torch.tensor(_ASCII, dtype=torch.uint8, device="cuda")
    rand = lut[torch.randint(0, 4, (total,), generator=gen, device="cuda")]
    random_ones = torch.repeat_interleave(kind == 3, lengths, output_size=total)
    return torch.where(random_ones, rand, buf), off


def _two_cuttings(case, seed):
    """synth.two_cuttings on the GPU: one sequence, two sets of cuts on multiples of the gap,
    no cut shared, the fragments shuffled."""
    gen = _gen(seed)
    length, gap = case["length"], case["gap"]
    seq = _genome(gen, length)
    k = max(1, length // case["mean"] - 1)
    slots = (torch.randperm((length - 1) // gap, generator=gen, device="cuda") + 1) * gap
    k = min(k, slots.numel() // 2)
    starts, lengths = [], []
    for cuts in (slots[:k], slots[k:2 * k]):
        edge = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"),
                          torch.sort(cuts).values,
                          torch.full((1,), length, dtype=torch.int64, device="cuda")])
        starts.append(edge[:-1])
        lengths.append(edge[1:] - edge[:-1])
    starts, lengths = torch.cat(starts), torch.cat(lengths)
    mix = torch.randperm(starts.numel(), generator=gen, device="cuda")
    return _text(gen, seq, starts[mix], lengths[mix])


# ---- what a program holds, and one pass -----------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "min_len": case.get("min_len")}
    if kind in ("path", "batch", "serve", "strands"):
        s["room"] = _room(case)
    if kind in ("path", "skew", "strands"):
        s["text"] = _read_set(case, seed)
    elif kind == "batch":
        texts = _sets(case, case["sets"], seed)
        s["off"] = np.concatenate([[0], np.cumsum([t.numel() for t in texts])]).astype(np.int64)
        s["text"] = torch.cat(texts)
    elif kind == "serve":
        s["texts"] = [t.cpu().numpy() for t in _sets(case, case["jobs"], seed)]
        s["server"] = pkg.AsmServer(24 << 30, max_jobs_per_batch=64, workers=8)
    elif kind == "lookup":
        s["text"] = _read_set(case, seed)
        s["patterns"] = _patterns(_gen(seed + 1), s["text"], case)
        s["sa"], _ = pkg.sa_build(s["text"], isa=False)
    elif kind == "sort":
        gen = _gen(seed)
        n = case["pairs"]
        hi = torch.randint(0, 1 << 32, (n,), generator=gen, device="cuda", dtype=torch.int64)
        lo = torch.randint(0, 1 << 32, (n,), generator=gen, device="cuda", dtype=torch.int64)
        s["keys"] = (hi << 32) | lo
        s["vals"] = torch.arange(n, dtype=torch.int32, device="cuda")
        s["bits"] = (case["bit_lo"], case["bit_hi"])
    else:
        s["text"] = _two_cuttings(case, seed)
    return s


def _held(rows, room):
    """The overlap rows in a table of fixed size, as a program that reads a count's worth of
    them holds it; rows of -1 after the last."""
    table = torch.full((room, rows.shape[1]), -1, dtype=rows.dtype, device=rows.device)
    table[: rows.shape[0]] = rows
    return table


def _serve(s):
    server = s["server"]
    ids = [server.asm_submit(t, s["min_len"], borrow=True) for t in s["texts"]]
    got = [None] * len(ids)
    while None in got:
        waiting = False
        for k, jid in enumerate(ids):
            if got[k] is None:
                got[k] = server.asm_poll(jid)
                waiting = waiting or got[k] is None
        if waiting:
            time.sleep(0.0002)
    out = [torch.cat([r[key] for r in got]) for key in ("sa", "isa", "lcp", "ovl")]
    out[3] = _held(out[3], s["room"])
    torch.cuda.current_stream().synchronize()  # the copies are made: the arena may be reused
    for jid in ids:
        server.asm_release(jid)
    return out


def run(state):
    kind = state["kind"]
    if kind == "path":
        sa, isa, lcp, rows = pkg.sa_path(state["text"], state["min_len"])
        return sa, isa, lcp, _held(rows, state["room"])
    if kind == "batch":
        sa, isa, lcp = pkg.sa_build_batched(state["text"], state["off"], lcp=True)
        rows = pkg.sa_overlaps(state["text"], sa, isa, lcp, state["min_len"])
        return sa, isa, lcp, _held(rows, state["room"])
    if kind == "serve":
        return _serve(state)
    if kind == "lookup":
        return pkg.sa_lookup(state["text"], state["sa"], state["patterns"])
    if kind == "skew":
        return pkg.sa_build_dc3(state["text"])
    if kind == "sort":  # sorts in place: the program keeps its unsorted pairs and sorts a copy
        return pkg.sa_sort_pairs(state["keys"].clone(), state["vals"].clone(), *state["bits"])
    if kind == "strands":
        return _held(pkg.sa_overlaps_rc(state["text"], state["min_len"]), state["room"])
    found = pkg.sa_reconstruct(state["text"])
    if found is None:
        return np.zeros(0, dtype=np.uint8), np.zeros(0, dtype=np.int32)
    return np.frombuffer(found[0], dtype=np.uint8), np.asarray(found[1], dtype=np.int32)


def _reads(case):
    """(reads, characters) of a case's text or texts; a set of m reads of lengths even over
    [lo, hi] has m * (lo + hi) / 2 bases and m separators."""
    if case["kind"] in ("batch", "serve"):
        sizes = _set_sizes(case, case.get("sets", case.get("jobs")))
    else:
        lo, hi = case.get("lo", case.get("read")), case.get("hi", case.get("read"))
        sizes = [(case["genome"], case["reads"], min(lo, case["genome"]), min(hi, case["genome"]))]
    return sum(m for _, m, _, _ in sizes), sum(m * (0.5 * (lo + hi) + 1) for _, m, lo, hi in sizes)


def _room(case):
    """Rows of the overlap table: a read overlaps at most about as many others as cover its
    bases, on either strand, and repeats add to that."""
    if case["kind"] in ("batch", "serve"):
        cov = case["cov_hi"]
    else:
        cov = _reads(case)[1] / case["genome"]
    return int(_reads(case)[0] * (2.0 * cov + 4.0)) + 1024


def work(case):
    """The text read once; the arrays that come back written once.  Nothing here is a product
    of numbers, so there are no operations to count beside the bytes."""
    kind = case["kind"]
    if kind == "sort":
        return {"bytes": 24.0 * case["pairs"], "flops": 0}
    if kind == "reconstruct":  # fragments in; the sequence and the order out
        return {"bytes": 3.0 * case["length"] + 10.0 * case["length"] / case["mean"], "flops": 0}
    m, n = _reads(case)
    if kind == "lookup":  # text, suffix array, patterns and their offsets; two ends each
        mean = 0.5 * (case["p_lo"] + case["p_hi"])
        return {"bytes": 5.0 * n + case["patterns"] * (mean + 16.0), "flops": 0}
    if kind == "skew":  # SA and inverse
        return {"bytes": 9.0 * n, "flops": 0}
    if kind == "strands":  # only the rows come back, four words each
        return {"bytes": n + 16.0 * _room(case), "flops": 0}
    return {"bytes": 13.0 * n + 12.0 * _room(case), "flops": 0}


def exact(case, seed):
    """No output is a rounded number: see the head of this file."""
    return None
