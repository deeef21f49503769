"""Small texts take the first round by top bits too: sizes from one character to past one radix
tile, texts with runs shorter and longer than the run sort takes, by the single and the batched
build, against the oracle and against the passes over the whole key (a build with a tuning)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TUNING = {"digit_bits": 9, "block_threads": 512, "items_per_thread": 8}


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def texts(n):
    rng = np.random.default_rng(n)
    bases = np.frombuffer(b"ACGT", dtype=np.uint8)
    random = bases[rng.integers(0, 4, n)]
    random[rng.random(n) < 0.01] = ord("$")
    same = np.full(n, ord("A"), dtype=np.uint8)
    copies = np.tile(np.append(bases[rng.integers(0, 4, 99)], np.uint8(ord("$"))), n // 100 + 1)[:n].copy()
    pairs = np.tile(bases[rng.integers(0, 4, 7)], n // 7 + 1)[:n].copy()
    for t in (random, same, copies, pairs):
        t[-1] = ord("$")
        yield t


@pytest.mark.parametrize("n", [1, 2, 3, 31, 64, 129, 257, 895, 896, 897, 1025, 1409, 4097, 8193, 16_383, 16_384])
def test_small_builds(lib, n):
    for text in texts(n):
        t = torch.from_numpy(text).cuda()
        want = oracle.suffix_array(text)
        sa, isa = lib.sa_build(t)
        assert np.array_equal(sa.cpu().numpy(), want)
        assert np.array_equal(isa.cpu().numpy()[want], np.arange(n))
        tuned, _ = lib.sa_build(t, tuning=TUNING)
        assert torch.equal(tuned, sa)
        sa, isa, lcp = lib.sa_build_batched(t, np.array([0, n], dtype=np.int64), lcp=True)
        assert np.array_equal(sa.cpu().numpy(), want)
        assert np.array_equal(lcp.cpu().numpy(), oracle.lcp_array(text, want))


def test_small_batches(lib):
    parts = [t for n in (1, 5, 90, 130, 700) for t in texts(n)]
    off = np.cumsum([0] + [p.size for p in parts]).astype(np.int64)
    sa, isa, lcp = lib.sa_build_batched(torch.from_numpy(np.concatenate(parts)).cuda(), off, lcp=True)
    sa, lcp = sa.cpu().numpy(), lcp.cpu().numpy()
    for k, p in enumerate(parts):
        want = oracle.suffix_array(p)
        assert np.array_equal(sa[off[k]:off[k + 1]] - off[k], want) or np.array_equal(sa[off[k]:off[k + 1]], want)
        assert np.array_equal(lcp[off[k]:off[k + 1]], oracle.lcp_array(p, want))
