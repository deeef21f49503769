"""The host's check of a text that is copied at submission: lengths at the edges of its 64-byte
vectors and of its 8-bit counts, a foreign byte at every kind of place, all separators.  And its
point: jobs submitted together find their way into shared batches."""
import time

import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LENGTHS = [1, 2, 63, 64, 65, 127, 128, 129, 64 * 255 - 1, 64 * 255, 64 * 255 + 1, 64 * 256 + 65, 64 * 511 + 3]


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def wait(srv, jid):
    end = time.time() + 60
    while True:
        r = srv.asm_poll(jid)
        if r is not None:
            return r
        assert time.time() < end
        time.sleep(0.0005)


def text_of(n, share):
    rng = np.random.default_rng([synth.SEED_BASE, 813, n])
    t = rng.choice(np.frombuffer(b"ACGT", dtype=np.uint8), n)
    t[rng.random(n) < share] = synth.SEP
    t[-1] = synth.SEP
    return t


@pytest.mark.parametrize("share", [0.02, 1.0])
def test_counts(lib, share):
    texts = [text_of(n, share) for n in LENGTHS]
    with lib.AsmServer(1 << 30, max_jobs_per_batch=4, workers=1) as srv:
        ids = [srv.asm_submit(t, 8) for t in texts]
        for t, j in zip(texts, ids):
            r = wait(srv, j)
            assert r["status"] == lib.SA_OK and r["m"] == int((t == synth.SEP).sum())
            assert np.array_equal(r["sa"].cpu().numpy(), oracle.suffix_array(t))


def test_foreign_bytes(lib):
    with lib.AsmServer(1 << 28, workers=1) as srv:
        for n in LENGTHS[1:]:
            for at in sorted({0, n - 2, min(n - 2, 62), min(n - 2, 63), min(n - 2, 64), min(n - 2, n // 2)}):
                for byte in (0, ord("N"), ord("a"), ord("@"), 255):
                    t = text_of(n, 0.02)
                    t[at] = byte
                    with pytest.raises(lib.SaasmError) as e:
                        srv.asm_submit(t, 8)
                    assert e.value.code == lib.SA_ERR_ALPHABET
        assert srv.asm_server_stats()["jobs_done"] == 0
