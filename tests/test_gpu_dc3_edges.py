"""The skew construction at the edges of its merge tiles (2,048 outputs) and of the groups of lanes
that look for a split: sizes around them, lists of which one ends early, with and without the
inverse.  Exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def texts(n):
    rng = np.random.default_rng(n)
    bases = np.frombuffer(b"ACGT", dtype=np.uint8)
    mixed = bases[rng.integers(0, 4, n)]
    mixed[rng.random(n) < 0.02] = ord("$")
    same = np.full(n, ord("A"), dtype=np.uint8)
    third = np.full(n, ord("C"), dtype=np.uint8)
    third[::3] = ord("T")  # the positions 0 mod 3 sort above all others
    first = np.full(n, ord("T"), dtype=np.uint8)
    first[::3] = ord("A")  # and below
    for t in (mixed, same, third, first):
        t[-1] = ord("$")
        yield t


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 17, 2047, 2048, 2049, 2050, 4095, 4097, 6145, 12_289])
def test_dc3_merge_edges(lib, n):
    for text in texts(n):
        t = torch.from_numpy(text).cuda()
        want = oracle.suffix_array(text)
        sa, isa = lib.sa_build_dc3(t)
        assert np.array_equal(sa.cpu().numpy(), want)
        assert np.array_equal(isa.cpu().numpy()[want], np.arange(n))
        sa, none = lib.sa_build_dc3(t, isa=False)
        assert none is None and np.array_equal(sa.cpu().numpy(), want)
