"""The sample that tells a first round whether nearly all its runs are too long for the run sort:
texts of either kind above the size it is taken from, whose route the timing records show, and a
batch whose sets share what none of them repeats.  Every entry against the definition."""
import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import synth
from tests import checks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MIN_N = 1 << 23
LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def cover(n, times, read=150, err=0.003, seed=9970):
    t = synth.genome_reads(seed, max(read + 1, n // times), n // (read + 1) + 2, read, err=err)[:n].copy()
    t[-1] = synth.SEP
    return t


def text_of(kind, n):
    rng = np.random.default_rng([synth.SEED_BASE, 811])
    copies = np.resize(np.append(rng.choice(LETTERS, 500), np.uint8(synth.SEP)), n)
    text = {"10x": lambda: cover(n, 10), "60x": lambda: cover(n, 60), "400x": lambda: cover(n, 400),
            "error-free 400x": lambda: cover(n, 400, err=0.0), "copies": lambda: copies,
            "tenth copies": lambda: np.concatenate([cover(n - n // 10, 10), copies[: n // 10]]),
            "tandem": lambda: np.resize(np.append(np.resize(rng.choice(LETTERS, 7), 700), np.uint8(synth.SEP)), n),
            "homopolymer": lambda: np.resize(np.append(np.full(900, ord("C")), synth.SEP).astype(np.uint8), n),
            "short reads": lambda: cover(n, 400, read=9)}[kind]().copy()
    text[-1] = synth.SEP
    return text


def check(lib, text, off, whole_keys):
    n = text.size
    lib.sa_timing_reset()
    lib.sa_timing_enable(True)
    try:
        sa, isa, lcp = lib.sa_build_batched(torch.from_numpy(text).cuda(), off, lcp=True)
    finally:
        lib.sa_timing_enable(False)
    assert lib.sa_timing_items("first_runs") == (0 if whole_keys else n)
    sa, isa, lcp = sa.cpu().numpy(), isa.cpu().numpy(), lcp.cpu().numpy()
    assert np.array_equal(isa[sa], np.arange(n, dtype=np.int32))
    for lo, hi in zip(off[:-1], off[1:]):
        assert sa[lo:hi].min() == lo and sa[lo:hi].max() == hi - 1 and lcp[lo] == 0
        bad, first = oracle.check_all(text, sa, lcp, lo=int(lo) + 1, hi=int(hi))
        assert bad == 0, f"{bad} bad adjacent pairs, the first at {first}"
    return sa


@pytest.mark.parametrize("n", [MIN_N + 1, MIN_N + 70_001])
@pytest.mark.parametrize("kind, whole_keys", [("10x", False), ("60x", False), ("400x", True),
                                              ("error-free 400x", True), ("copies", True),
                                              ("tandem", True), ("homopolymer", True),
                                              ("tenth copies", False)])
def test_route_above_the_least_size(lib, kind, whole_keys, n):
    text = text_of(kind, n)
    sa = check(lib, text, np.array([0, n], dtype=np.int64), whole_keys)
    checks.assert_sa_basic(text, sa)


@pytest.mark.parametrize("kind", ["400x", "copies", "short reads"])
def test_no_sample_at_the_least_size(lib, kind):
    text = text_of(kind, MIN_N)
    checks.assert_sa_basic(text, check(lib, text, np.array([0, MIN_N], dtype=np.int64), False))


def test_short_reads_above_it(lib):
    """Most suffixes end before the top bases do and are not sampled."""
    n = MIN_N + 5
    text = text_of("short reads", n)
    sa, _ = lib.sa_build(torch.from_numpy(text).cuda())
    sa = sa.cpu().numpy()
    checks.assert_sa_basic(text, sa)
    assert oracle.check_all(text, sa, None)[0] == 0


@pytest.mark.parametrize("count, times, own", [(12, 400, True), (200, 2, False)])
def test_runs_end_with_their_set(lib, count, times, own):
    """Twelve sets of 400x each; or 200 sets of the same reads, which hardly repeat in a set."""
    size = MIN_N // count + 60
    one = cover(size, times, err=0.0)
    sets = [cover(size, times, seed=9980 + k) if own else one for k in range(count)]
    off = np.cumsum([0] + [s.size for s in sets]).astype(np.int64)
    check(lib, np.concatenate(sets), off, own)
