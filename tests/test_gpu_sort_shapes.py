"""Sorts on either side of the numbers of items where the untuned tile changes, for the digits whose
numbers differ: stable and exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1 << 19, (1 << 19) + 1, 1 << 20, (1 << 20) + 1, 1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("digit_bits", [0, 11])
def test_sort_at_the_changes_of_shape(digit_bits, n):
    import paper_1404_3456_amd as lib
    lib.load()
    rng = np.random.default_rng(n + digit_bits)
    keys = rng.integers(0, 1 << 24, n, dtype=np.int64) << 20  # many equal keys
    k, v = torch.from_numpy(keys).cuda(), torch.arange(n, dtype=torch.int32, device="cuda")
    lib.sa_sort_pairs(k, v, 18, 45, tuning={"digit_bits": digit_bits} if digit_bits else None)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(v.cpu().numpy(), order) and np.array_equal(k.cpu().numpy(), keys[order])
