"""sa_lookup through the C interface with and without room for samples of the suffix array: the
two routes against each other and against the oracle, at the edges of the sample array (one
sample, the 512 a workgroup holds, more than patterns ask for) and of a sample's 29 bases."""
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


def lookup(lib, t, sa, pats, samples, shift=0):
    c = lib.load()
    raw = b"".join(pats)
    buf = torch.zeros(len(raw) + shift + 1, dtype=torch.uint8, device="cuda")
    if raw:
        buf[shift:shift + len(raw)] = torch.from_numpy(np.frombuffer(raw, dtype=np.uint8).copy()).cuda()
    off = torch.from_numpy(np.cumsum([0] + [len(x) for x in pats])).cuda()
    need = lib.sa_lookup_ws_bytes(t.numel(), len(raw))
    ws = torch.empty(need - (0 if samples else 1), dtype=torch.uint8, device="cuda")
    out = torch.full((len(pats), 2), -7, dtype=torch.int32, device="cuda")
    P = lambda x, o=0: ctypes.c_void_p(x.data_ptr() + o)  # noqa: E731
    rc = c.sa_lookup(P(t), t.numel(), P(sa), P(buf, shift), P(off), len(raw), len(pats), P(out), P(ws),
                     ws.numel(), None)
    assert rc == lib.SA_OK
    return out.cpu().numpy().astype(np.int64)


def periodic(n):
    x = np.frombuffer((b"ACGTTT" * (n // 6 + 1))[: n - 1] + b"$", dtype=np.uint8).copy()
    x[n // 3] = ord("$")
    return x


TEXTS = {
    "one": np.frombuffer(b"$", dtype=np.uint8).copy(),
    "empty reads": np.frombuffer(b"$" * 33, dtype=np.uint8).copy(),
    "15": periodic(15), "16": periodic(16), "17": periodic(17),
    "same": np.frombuffer(b"A" * 3000 + b"$" + b"A" * 40 + b"$", dtype=np.uint8).copy(),
    "511 samples": periodic(16 * 511 - 1), "512 samples": periodic(16 * 512 - 1),
    "513 samples": periodic(16 * 513),
    "reads": synth.genome_reads(11, 9_000, 700, 100, err=0.01),
}


@pytest.mark.parametrize("name", sorted(TEXTS))
def test_lookup_routes_agree(lib, name):
    text = TEXTS[name]
    tb = bytes(text)
    t = torch.from_numpy(text).cuda()
    sa, _ = lib.sa_build(t)
    rng = np.random.default_rng(7)
    pats = [b"", b"A", b"T" * 29, b"T" * 30, b"A" * 28, b"A" * 29, b"A" * 30, b"A" * 60]
    for m in (1, 2, 3, 8, 27, 28, 29, 30, 31, 32, 33, 64):
        for _ in range(6):
            p = int(rng.integers(0, len(tb)))
            x = tb[p:p + m].split(b"$")[0]
            pats += [x, x[:-1] + b"T", x + b"A", b"A" + x]
    want = oracle.lookup(text, pats)
    for shift in (0, 3):
        assert np.array_equal(lookup(lib, t, sa, pats, True, shift), want)
        assert np.array_equal(lookup(lib, t, sa, pats, False, shift), want)


def test_lookup_samples_follow_the_patterns(lib):
    """More than four patterns per least sample: their number sets how many samples there are."""
    text = synth.genome_reads(12, 20_000, 2_000, 120, err=0.005)
    t = torch.from_numpy(text).cuda()
    sa, _ = lib.sa_build(t)
    pats = synth.lookup_patterns(text, 30_001, 5, 0, 50)
    a, b = lookup(lib, t, sa, pats, True), lookup(lib, t, sa, pats, False)
    assert np.array_equal(a, b)
    assert np.array_equal(a[:400], oracle.lookup(text, pats[:400]))
