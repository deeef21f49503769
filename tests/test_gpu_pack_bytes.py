"""Packing takes the text's bytes four at a time, at any alignment: every size around the words it
reads, every place of the end, and every byte value in every place of a word."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ALPHABET = np.frombuffer(b"ACGT$", dtype=np.uint8)


@pytest.fixture(scope="module")
def lib():
    import paper_1404_3456_amd as p
    p.load()
    return p


def at(text, shift):
    buf = torch.full((text.size + shift + 8,), ord("N"), dtype=torch.uint8, device="cuda")
    buf[shift:shift + text.size] = torch.from_numpy(text).cuda()
    return buf[shift:shift + text.size]


@pytest.mark.parametrize("shift", [0, 1, 2, 3, 8])
def test_pack_every_size_and_alignment(lib, shift):
    rng = np.random.default_rng(shift)
    for n in list(range(1, 70)) + [255, 256, 257, 8191, 8192, 8193, 8199]:
        text = ALPHABET[rng.integers(0, 5, n)]
        text[-1] = ord("$")
        packed, sepmask, read_end = lib.sa_pack(at(text, shift))
        sep = text == ord("$")
        code = np.where(sep, 0, np.searchsorted(np.frombuffer(b"ACGT", dtype=np.uint8), text)) & 3
        words = np.zeros(-(-n // 32) * 2, dtype=np.uint64)
        bits = np.zeros(-(-n // 32), dtype=np.uint64)
        i = np.arange(n)
        np.bitwise_or.at(words, i // 16, code.astype(np.uint64) << (30 - 2 * (i % 16)).astype(np.uint64))
        np.bitwise_or.at(bits, i // 32, sep.astype(np.uint64) << (31 - i % 32).astype(np.uint64))
        u32 = lambda x: x.cpu().numpy().view(np.uint32)  # noqa: E731
        assert np.array_equal(u32(packed)[: words.size], words.astype(np.uint32)), n
        assert np.array_equal(u32(sepmask)[: bits.size], bits.astype(np.uint32)), n
        assert np.array_equal(read_end.cpu().numpy(), np.flatnonzero(sep)), n


@pytest.mark.parametrize("n", [33, 70])
def test_pack_refuses_every_other_byte(lib, n):
    for c in range(256):
        text = np.full(n, ord("C"), dtype=np.uint8)
        text[-1] = ord("$")
        text[(c * 7) % (n - 1)] = c
        if c in b"ACGT$":
            lib.sa_pack(at(text, c & 3))
        else:
            with pytest.raises(lib.SaasmError) as e:
                lib.sa_pack(at(text, c & 3))
            assert e.value.code == lib.SA_ERR_ALPHABET
    text[(255 * 7) % (n - 1)] = text[-1] = ord("A")
    with pytest.raises(lib.SaasmError) as e:  # no separator at the end
        lib.sa_pack(at(text, 1))
    assert e.value.code == lib.SA_ERR_INVALID
