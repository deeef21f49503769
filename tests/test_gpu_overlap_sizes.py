"""sa_overlaps through the C interface in workspaces of every kind: too small for the reads, for
the candidates, exactly what it asked for, and roomy; texts at the edges of its tiles (words of
32 positions by 256, 256 reads, 1,024 candidates) and reads with more matches than a thread
keeps.  Exact against the oracle."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def call(lib, t, index, min_len, ws_bytes, cap):
    c = lib.load()
    sa, isa, lcp = index
    n = t.numel()
    P = lambda x: ctypes.c_void_p(x.data_ptr())  # noqa: E731
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    out = torch.empty((max(cap, 1), 3), dtype=torch.int32, device="cuda")
    k, need = ctypes.c_int64(-1), ctypes.c_int64(-1)
    rc = c.sa_overlaps(P(t), n, P(sa), P(isa), P(lcp), min_len, P(out), cap, ctypes.byref(k), P(ws),
                       ws_bytes, ctypes.byref(need), None)
    return rc, k.value, need.value, out


def every_workspace(lib, text, min_len):
    t = torch.from_numpy(text).cuda()
    sa, isa = lib.sa_build(t)
    index = (sa, isa, lib.sa_lcp(t, sa, isa))
    torch.cuda.synchronize()
    want = oracle.overlaps(text, min_len)
    rows = want.shape[0]
    n = text.size
    ws, seen = lib.sa_overlaps_ws_bytes(n, 1, 0), 0
    while True:  # from the least the call takes, by what it asks for
        rc, k, need, out = call(lib, t, index, min_len, ws, rows)
        if rc == lib.SA_OK:
            break
        assert rc == lib.SA_ERR_NOMEM and need > ws and seen < 3
        ws, seen = need, seen + 1
    assert k == rows and np.array_equal(out.cpu().numpy()[:k], want)
    roomy = lib.sa_workspace_bytes(n, 0) + (64 << 20)
    rc, k, _, out = call(lib, t, index, min_len, roomy, rows)
    assert rc == lib.SA_OK and k == rows and np.array_equal(out.cpu().numpy()[:k], want)
    if rows > 1:
        rc, k, _, _ = call(lib, t, index, min_len, roomy, rows - 1)
        assert rc == lib.SA_ERR_CAPACITY and k == rows
    return rows


@pytest.mark.parametrize("n", [31, 32, 33, 8191, 8192, 8193, 24_576, 100_003])
def test_text_edges(lib, n):
    t = synth.genome_reads(9500 + n, max(40, n // 6), n // 31 + 2, 30)[:n].copy()
    t[-1] = synth.SEP
    every_workspace(lib, t, 12)


@pytest.mark.parametrize("m", [255, 256, 257, 1025])
def test_read_edges(lib, m):
    assert every_workspace(lib, synth.genome_reads(9600 + m, 8 * m, m, 60), 20) > 0


@pytest.mark.parametrize("copies", [12, 13, 14, 60])
def test_many_matches_a_read(lib, copies):
    """`copies` equal reads match each other, tandem reads match at several lengths."""
    reads = ["ACGGTCATTGCA" * 4] * copies + ["AC" * 20, "CA" * 19 + "C", "ACAC" * 9] * 3
    assert every_workspace(lib, synth.text_from_strings(reads), 8) > copies


def test_many_empty_reads(lib):
    """More reads than a workspace's first split has room for."""
    rng = np.random.default_rng([synth.SEED_BASE, 804])
    reads = [""] * 30_000 + ["ACGTTGCA"[int(rng.integers(0, 4)):] for _ in range(300)]
    every_workspace(lib, synth.text_from_strings([reads[i] for i in rng.permutation(len(reads))]), 3)


@pytest.mark.parametrize("bad", [(), (0,), (2, 3), (0, 1, 2, 3, 4)])
def test_borrowed_jobs_checked_on_the_device(lib, bad):
    """Borrowed texts of odd lengths in one batch, some with a foreign byte at their first or
    last base: those (only) are refused, the others' results are their own."""
    import time
    texts = [synth.genome_reads(9700 + k, 300 + 17 * k, 20 + k, 41 + k) for k in range(5)]
    jobs = [t.copy() for t in texts]
    for k in bad:
        jobs[k][0 if k % 2 else jobs[k].size - 2] = ord("N")
    with lib.AsmServer(1 << 30, max_jobs_per_batch=8, workers=1) as srv:
        first = srv.asm_submit(texts[0], 15, borrow=True)  # the others queue up behind it
        ids = [srv.asm_submit(t, 15, borrow=True) for t in jobs]
        end = time.time() + 60
        while any(srv.asm_poll(j) is None for j in [first] + ids):
            assert time.time() < end
            time.sleep(0.001)
        assert srv.asm_poll(first)["status"] == lib.SA_OK
        for k, j in enumerate(ids):
            r = srv.asm_poll(j)
            if k in bad:
                assert r["status"] == lib.SA_ERR_ALPHABET
                continue
            want = oracle.suffix_array(texts[k])
            assert r["status"] == lib.SA_OK and r["m"] == int((texts[k] == synth.SEP).sum())
            assert np.array_equal(r["sa"].cpu().numpy(), want)
            assert np.array_equal(r["ovl"].cpu().numpy(), oracle.overlaps(texts[k], 15))
