"""The first round's run sort in both of its shapes (tiles of 896 items up to 2^21 suffixes, of
1,408 above), with the LCP array the build makes itself: sizes at the edges of the tiles and of the
switch, texts above it with runs too long for LDS and with matches past the windows, past the scan
after them and past both.  Every entry against the definition (a permutation whose neighbours all
ascend, each with its common prefix).  At the workloads' full sizes the arrays are those of
sa_build and sa_lcp, which the full-size tests hold to the same."""
import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import synth
from tests import checks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SMALL, LARGE, LIMIT = 896, 1408, 128  # items a tile finishes; longest run it sorts
SWITCH = 1 << 21
ABOVE = (SWITCH // LARGE + 1) * LARGE
LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def check(lib, text):
    n = text.size
    sa, isa, lcp = lib.sa_build_batched(torch.from_numpy(text).cuda(), np.array([0, n], dtype=np.int64), lcp=True)
    sa, isa, lcp = sa.cpu().numpy(), isa.cpu().numpy(), lcp.cpu().numpy()
    checks.assert_sa_basic(text, sa)
    assert np.array_equal(isa[sa], np.arange(n, dtype=np.int32))
    bad, first = oracle.check_all(text, sa, lcp)
    assert bad == 0 and lcp[0] == 0, f"{bad} bad adjacent pairs, the first at {first}"


def reads(seed, n, cover=8, read=180):
    t = synth.genome_reads(seed, max(read + 1, n // cover), n // (read + 1) + 2, read, err=0.005)[:n].copy()
    t[-1] = synth.SEP
    return t


@pytest.mark.parametrize("n", [7 * SMALL - 1, 7 * SMALL, 7 * SMALL + 1, 7 * SMALL + LIMIT,
                               40 * SMALL + LIMIT + 1, SWITCH - 1, SWITCH, SWITCH + 1, ABOVE - 1, ABOVE,
                               ABOVE + 1, ABOVE + LIMIT])
def test_tile_and_switch_edges(lib, n):
    check(lib, reads(9900 + n % 89, n))


def with_extra(extra, size):
    """Reads of random genomes with the extra ones among them, in an order of their own."""
    rng = np.random.default_rng([synth.SEED_BASE, 807, len(extra), size])
    some = bytes(reads(9950, size)).split(b"$")[:-1]
    every = some + [e.encode() for e in extra]
    return synth.text_from_strings([every[i].decode() for i in rng.permutation(len(every))])


@pytest.mark.parametrize("size", [40_000, SWITCH + 20_000])
@pytest.mark.parametrize("kind", ["copies", "homopolymer", "empty", "beyond the windows",
                                  "beyond the scan", "both, many"])
def test_long_runs_and_matches(lib, kind, size):
    rng = np.random.default_rng([synth.SEED_BASE, 808, len(kind)])
    word = lambda k: rng.choice(LETTERS, k).tobytes().decode()  # noqa: E731
    a, b, c = word(300), word(1200), word(3500)  # windows reach about 490, the scan 2,048 more
    extra = {"copies": [a] * (LIMIT - 1) + [word(90)] * LIMIT + [word(200)] * (LIMIT + 1) + [word(60)] * 700,
             "homopolymer": ["A" * 900] * 9 + ["T" * 400] * 7,
             "empty": [""] * 600,
             "beyond the windows": [b + word(5) for _ in range(3)],
             "beyond the scan": [b, b + "A", c + "C", c + "G"],
             "both, many": [b] * 40 + [c] * 40 + ["AC" * 900] * 3}[kind]
    check(lib, with_extra(extra, size))


@pytest.mark.parametrize("workload", ["large_plain", "repeat_stress"])
def test_full_size_index_of_the_path(lib, workload):
    r = getattr(synth, workload)()
    t = torch.from_numpy(r.text).cuda()
    sa, isa, lcp, _ = lib.sa_path(t, r.min_len)
    sa2, isa2 = lib.sa_build(t)
    assert torch.equal(sa, sa2) and torch.equal(isa, isa2)
    assert torch.equal(lcp, lib.sa_lcp(t, sa2, isa2))


def test_full_size_batch(lib):
    sets = synth.batched_sets()
    off = np.concatenate([[0], np.cumsum([s.text.size for s in sets])]).astype(np.int64)
    t = torch.from_numpy(np.concatenate([s.text for s in sets])).cuda()
    sa, isa, lcp = lib.sa_build_batched(t, off, lcp=True)
    torch.cuda.empty_cache()
    assert torch.equal(lcp, lib.sa_lcp(t, sa, isa))
    sa2, isa2 = lib.sa_build_batched(t, off)
    assert torch.equal(sa, sa2) and torch.equal(isa, isa2)


def test_small_sets_in_concatenated_coordinates(lib):
    """Suffix arrays of a batch hold positions of the whole text; the inverse is of the whole."""
    parts = [reads(9960 + n, n, read=20) for n in (1, 22, 90, 130, 700, 5000)]
    off = np.cumsum([0] + [p.size for p in parts]).astype(np.int64)
    sa, isa, lcp = (x.cpu().numpy() for x in lib.sa_build_batched(
        torch.from_numpy(np.concatenate(parts)).cuda(), off, lcp=True))
    for k, p in enumerate(parts):
        want = oracle.suffix_array(p)
        assert np.array_equal(sa[off[k]:off[k + 1]] - off[k], want)
        assert np.array_equal(lcp[off[k]:off[k + 1]], oracle.lcp_array(p, want))
    assert np.array_equal(isa[sa], np.arange(off[-1]))
