"""A text without its final separator is refused without being searched: nothing would end a
comparison of a long pattern there."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("samples", [False, True])
@pytest.mark.parametrize("n", [33, 5000])
def test_not_searched(n, samples):
    import paper_1404_3456_amd as lib
    c = lib.load()
    text = torch.full((n,), ord("A"), dtype=torch.uint8, device="cuda")
    sa = torch.arange(n - 1, -1, -1, dtype=torch.int32, device="cuda")
    lengths = np.array([1, 40, n + 100, 3 * n], dtype=np.int64)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)])).cuda()
    total = int(lengths.sum())
    pat = torch.full((total,), ord("A"), dtype=torch.uint8, device="cuda")
    lohi = torch.full((len(lengths), 2), -7, dtype=torch.int32, device="cuda")
    size = int(c.sa_lookup_ws_bytes(n, total)) - (0 if samples else 1)  # a byte less: no samples
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    P = lambda x: ctypes.c_void_p(x.data_ptr())  # noqa: E731
    rc = c.sa_lookup(P(text), n, P(sa), P(pat), P(off), total, len(lengths), P(lohi), P(ws), size, None)
    torch.cuda.synchronize()
    assert rc == lib.SA_ERR_INVALID
    assert bool((lohi == -7).all())
