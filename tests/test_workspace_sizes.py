"""The one workspace of the path also holds the build that makes the LCP array itself, which is the
faster way to it: a batched build of the one text.  Host functions, without a GPU."""
import pytest

from paper_1404_3456_amd import _abi


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 16_384, 80_400, 1 << 26, 400_400_000, (1 << 31) - 3])
def test_path_workspace_holds_a_build_with_its_lcp(n):
    one = _abi.sa_build_batched_ws_bytes(n, 1)
    assert one >= _abi.sa_lcp_ws_bytes(n)
    assert _abi.sa_workspace_bytes(n, 1) >= one
