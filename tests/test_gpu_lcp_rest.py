"""Who finishes the LCP array of a build: entry by entry, or Kasai's scan where that is the shorter
way, on either side of the line for texts with and without long runs and on both sides of the
size at which the packed text leaves an XCD's L2."""
import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)
L2_CHARACTERS = (4 << 20) * 8 // 3


def reads(rng, n, read, cover):
    """Error-free reads of one genome; cover 0: copies of one read."""
    k = n // (read + 1) + 1
    genome = rng.choice(LETTERS, max(read, k * read // cover if cover else read))
    at = rng.integers(0, genome.size - read + 1, k)
    x = np.full((k, read + 1), synth.SEP, dtype=np.uint8)
    x[:, :read] = genome[at[:, None] + np.arange(read)]
    return x.reshape(-1)[:n]


@pytest.mark.parametrize("n, read, cover, scan", [
    (400_000, 650, 11, False), (400_000, 1000, 11, True),
    (L2_CHARACTERS, 800, 11, False), (L2_CHARACTERS, 1000, 5, True),
    (L2_CHARACTERS + 1, 700, 11, False), (L2_CHARACTERS + 1, 800, 11, True),
    (400_000, 200, 0, False), (400_000, 500, 0, True)])
def test_the_shorter_way(n, read, cover, scan):
    import paper_1404_3456_amd as lib
    lib.load()
    rng = np.random.default_rng([synth.SEED_BASE, 811, read])
    text = reads(rng, n, read, cover) if cover else \
        np.concatenate([reads(rng, n // 2, 300, 10), reads(rng, n - n // 2, read, 0)])
    text[-1] = synth.SEP
    t = torch.from_numpy(text).cuda()
    lib.sa_timing_reset()
    lib.sa_timing_enable(True)
    try:
        sa, isa, lcp = lib.sa_build_batched(t, np.array([0, n], dtype=np.int64), lcp=True)
    finally:
        lib.sa_timing_enable(False)
    assert [lib.sa_timing_get(k)[0] for k in ("lcp_rest", "kasai")] == ([0, 1] if scan else [1, 0])
    sa, lcp = sa.cpu().numpy(), lcp.cpu().numpy()
    assert np.array_equal(isa.cpu().numpy()[sa], np.arange(n, dtype=np.int32))
    bad, first = oracle.check_all(text, sa, lcp)
    assert bad == 0 and lcp[0] == 0, f"{bad} bad adjacent pairs, the first at {first}"
