"""sa_reconstruct on arrays that are no suffix array and its inverse: refused, with nothing written;
and on fragments that start all over a sequence."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1404_3456_amd import _abi


def index(text):
    sa = oracle.suffix_array(text).astype(np.int32)
    isa = np.empty_like(sa)
    isa[sa] = np.arange(text.size, dtype=np.int32)
    return sa, isa, oracle.lcp_array(text, sa).astype(np.int32)


def cut_twice(seq, cuts_a, cuts_b):
    frags = [seq[i:j] for c in (cuts_a, cuts_b) for i, j in zip([0] + c, c + [len(seq)])]
    return np.frombuffer(b"".join(f + b"$" for f in frags), dtype=np.uint8).copy(), frags


def sequence(n, seed):
    return bytes(np.frombuffer(b"ACGT", dtype=np.uint8)[np.random.default_rng(seed).integers(0, 4, n)])


@pytest.mark.parametrize("seed", range(4))
def test_reconstructs_over_fragment_starts(seed):
    rng = np.random.default_rng(seed)
    seq = sequence(6000, seed)
    cuts = np.sort(rng.choice(np.arange(20, 5980), 60, replace=False))
    cuts = cuts[np.diff(cuts, prepend=-50) > 24].tolist()
    text, _ = cut_twice(seq, cuts[::2], cuts[1::2])
    found = _abi.sa_reconstruct_host(text, *index(text))
    assert found is not None and len(found[0]) == len(seq) and found[0] == seq


@pytest.mark.parametrize("spoil", ["sa low", "sa high", "isa low", "isa high", "swapped", "zeros"])
def test_refuses_arrays_that_are_not_inverse(spoil):
    seq = sequence(90_000, 9)
    text, frags = cut_twice(seq, list(range(500, 90_000, 997)), list(range(700, 90_000, 1009)))
    sa, isa, lcp = index(text)
    k = text.size // 3
    if spoil == "sa low":
        sa[k] = -5
    elif spoil == "sa high":
        sa[k] = text.size
    elif spoil == "isa low":
        isa[:] = -1
    elif spoil == "isa high":
        isa[:] = 2 ** 31 - 1
    elif spoil == "swapped":
        sa[[k, k + 1]] = sa[[k + 1, k]]
    else:
        sa[:] = 0
        lcp[:] = 2 ** 30
    order = np.full(len(frags), -7, dtype=np.int32)
    rs = np.full(text.size, 7, dtype=np.uint8)
    rs_len = ctypes.c_int64(-7)
    p = lambda x: x.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    rc = _abi.load().sa_reconstruct(p(text), text.size, p(sa), p(isa), p(lcp), p(order), p(rs), rs.size,
                                    ctypes.byref(rs_len), 10 ** 7)
    assert rc == _abi.SA_ERR_INVALID
    assert (order == -7).all() and (rs == 7).all() and rs_len.value == -7
