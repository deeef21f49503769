"""The first round's run sort at the sizes where it can go wrong: texts on either side of its
threshold and of its tiles, runs of equal top key bits on either side of the longest it sorts in
LDS, groups that end inside, at and past the symbols its keys are extended by, and batches.
Exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TILE = 1408      # items a tile of the run sort finishes
LIMIT = 128      # longest run it sorts
MIN_N = 16384    # shorter texts sort whole keys by passes


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def check(lib, text, tuning=None):
    want = oracle.suffix_array(text)
    sa, isa = lib.sa_build(torch.from_numpy(text).cuda(), tuning=tuning)
    assert np.array_equal(sa.cpu().numpy(), want)
    inv = np.empty(text.size, dtype=np.int32)
    inv[want] = np.arange(text.size, dtype=np.int32)
    assert np.array_equal(isa.cpu().numpy(), inv)


def reads_of_size(seed, n, cover=8, read=180):
    """n characters of reads at `cover`x (the last read shorter), 0.5 % substitutions."""
    t = synth.genome_reads(seed, max(read + 1, n // cover), n // (read + 1) + 2, read, err=0.005)[:n].copy()
    t[-1] = synth.SEP
    return t


@pytest.mark.parametrize("n", [MIN_N - 1, MIN_N, MIN_N + 1, 10 * TILE - 1, 10 * TILE, 10 * TILE + 1,
                               11 * TILE + LIMIT, 300 * TILE + 63])
def test_text_sizes(lib, n):
    check(lib, reads_of_size(9000 + n % 97, n))


@pytest.mark.parametrize("copies", [31, 32, 33, 64, LIMIT - 1, LIMIT, LIMIT + 1, 192, 193, 400])
@pytest.mark.parametrize("read", [40, 89, 90, 91, 200])
def test_runs_and_groups_of_copies(lib, copies, read):
    """`copies` equal reads (groups of that size to the reads' ends) among others that are not
    repeated; reads of 89 to 91 bases end about where an extended key does."""
    rng = np.random.default_rng([synth.SEED_BASE, 801, copies, read])
    letters = np.frombuffer(b"ACGT", dtype=np.uint8)
    one = rng.choice(letters, read).tobytes().decode()
    rest = [rng.choice(letters, int(rng.integers(1, 300))).tobytes().decode() for _ in range(150)]
    reads = [one] * copies + rest
    reads = [reads[i] for i in rng.permutation(len(reads))]
    text = synth.text_from_strings(reads)
    while text.size < MIN_N:
        text = np.concatenate([text, synth.text_from_strings(rest)])
    check(lib, text)


@pytest.mark.parametrize("kind", ["homopolymer", "tandem", "empty", "two-letter", "mixed"])
@pytest.mark.parametrize("digit_bits", [0, 4, 8, 11])
def test_long_runs(lib, kind, digit_bits):
    rng = np.random.default_rng([synth.SEED_BASE, 802])
    letters = np.frombuffer(b"ACGT", dtype=np.uint8)
    some = [rng.choice(letters, int(rng.integers(50, 400))).tobytes().decode() for _ in range(120)]
    extra = {"homopolymer": ["A" * 700] * 9 + ["T" * 300] * 7,
             "tandem": ["ACG" * 150] * 40 + ["AC" * 90] * 25,
             "empty": [""] * 500,
             "two-letter": [rng.choice(letters[:2], 500).tobytes().decode() for _ in range(40)],
             "mixed": ["A" * 500] * 3 + [""] * 130 + [some[0]] * 200 + ["GT" * 200]}[kind]
    reads = some + extra
    text = synth.text_from_strings([reads[i] for i in rng.permutation(len(reads))])
    while text.size < MIN_N:
        text = np.concatenate([text, text])
    check(lib, text, tuning={"digit_bits": digit_bits} if digit_bits else None)


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("kind", ["plain", "repeats"])
def test_batches(lib, use_graph, kind):
    texts = [reads_of_size(9100 + k, n) for k, n in enumerate([40, 17_000, 5, TILE, 60_001, 3000])]
    if kind == "repeats":
        texts.append(synth.text_from_strings(["ACGT" * 100] * 60 + ["C" * 300] * 3))
    off = np.concatenate([[0], np.cumsum([t.size for t in texts])]).astype(np.int64)
    sa, isa, lcp = lib.sa_build_batched(torch.from_numpy(np.concatenate(texts)).cuda(), off,
                                        use_graph=use_graph, lcp=True)
    sa, lcp = sa.cpu().numpy(), lcp.cpu().numpy()
    for k, t in enumerate(texts):
        want = oracle.suffix_array(t)
        assert np.array_equal(sa[off[k]:off[k + 1]] - off[k], want)
        assert np.array_equal(lcp[off[k]:off[k + 1]], oracle.lcp_array(t, want))
    assert np.array_equal(isa.cpu().numpy()[sa], np.arange(off[-1]))


def lcp_of(lib, text):
    off = np.array([0, text.size], dtype=np.int64)
    sa, _, lcp = lib.sa_build_batched(torch.from_numpy(text).cuda(), off, lcp=True)
    return sa.cpu().numpy(), lcp.cpu().numpy()


@pytest.mark.parametrize("read", [24, 25, 80, 81, 82, 137, 138, 139, 481, 2400, 2600])
def test_lcp_of_the_build(lib, read):
    """The LCP array a build makes itself: pairs that share about as much as a key, a stage, a
    window and all windows hold, and more than the scan after them goes on for (then the
    array is Kasai's), in groups small and large."""
    rng = np.random.default_rng([synth.SEED_BASE, 803, read])
    letters = np.frombuffer(b"ACGT", dtype=np.uint8)
    base = rng.choice(letters, read)
    reads = []
    for copies, cut in ((3, 0), (40, 1), (150, 2)):  # copies that end differently
        for _ in range(copies if read < 1000 else min(copies, 12)):
            r = base.copy()
            if r.size > 30:
                r[int(rng.integers(20, r.size))] = letters[int(rng.integers(0, 4))]
            reads.append(r[: r.size - cut].tobytes().decode())
    reads += [rng.choice(letters, int(rng.integers(1, 300))).tobytes().decode() for _ in range(200)]
    text = synth.text_from_strings([reads[i] for i in rng.permutation(len(reads))])
    sa, lcp = lcp_of(lib, text)
    want = oracle.suffix_array(text)
    assert text.size >= MIN_N
    assert np.array_equal(sa, want)
    assert np.array_equal(lcp, oracle.lcp_array(text, want))


@pytest.mark.parametrize("kind", ["homopolymer", "tandem", "empty"])
def test_lcp_of_long_runs(lib, kind):
    reads = {"homopolymer": ["A" * 9000, "C" * 9000], "tandem": ["ACG" * 150] * 60, "empty": [""] * 17_000}[kind]
    text = synth.text_from_strings(reads + ["ACGT"])
    sa, lcp = lcp_of(lib, text)
    want = oracle.suffix_array(text)
    assert text.size >= MIN_N
    assert np.array_equal(sa, want)
    assert np.array_equal(lcp, oracle.lcp_array(text, want))


def test_path_in_a_smaller_workspace(lib):
    """sa_path in the workspace its documentation asks for, and in its own, gives the same."""
    text = reads_of_size(9300, 40_000)
    t = torch.from_numpy(text).cuda()
    ws = torch.empty(lib.sa_workspace_bytes(text.size, 0), dtype=torch.uint8, device="cuda")
    want = oracle.suffix_array(text)
    for got in (lib.sa_path(t, 30, ws=ws), lib.sa_path(t, 30)):
        assert np.array_equal(got[0].cpu().numpy(), want)
        assert np.array_equal(got[2].cpu().numpy(), oracle.lcp_array(text, want))
        assert np.array_equal(got[3].cpu().numpy(), oracle.overlaps(text, 30))
