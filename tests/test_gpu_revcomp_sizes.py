"""The doubled text of both strands at sizes around the 16 characters a thread takes, with the text
at every alignment of a word; bytes outside the alphabet are copied as they are."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

COMPLEMENT = np.arange(256, dtype=np.uint8)
COMPLEMENT[np.frombuffer(b"ACGT", dtype=np.uint8)] = np.frombuffer(b"TGCA", dtype=np.uint8)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 18, 31, 32, 33, 34, 49, 4095, 4096, 4097, 70_001])
def test_revcomp_text(n):
    import paper_1404_3456_amd as lib
    rng = np.random.default_rng(n)
    for shift in range(4):
        text = np.frombuffer(b"ACGT$", dtype=np.uint8)[rng.integers(0, 5, n)]
        if shift == 3 and n > 40:
            text[5:-1] = rng.integers(0, 256, n - 6)
        text[-1] = ord("$")
        buf = torch.full((n + shift,), 7, dtype=torch.uint8, device="cuda")
        buf[shift:] = torch.from_numpy(text).cuda()
        out, m = lib.sa_revcomp_text(buf[shift:])
        want = np.concatenate([text, COMPLEMENT[text[:-1][::-1]], text[-1:]])
        assert m == int((text == ord("$")).sum())
        assert np.array_equal(out.cpu().numpy(), want)
