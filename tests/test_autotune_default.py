"""The untuned default is among what the autotuner measures, so its answer is no slower than no
tuning."""
from paper_1404_3456_amd import _abi, autotune


def test_the_default_is_a_candidate():
    assert (0, 0, 0) in autotune.TILE_CANDIDATES
    none, default = _abi.sa_build_ws_bytes(100_000), _abi.sa_build_ws_bytes(100_000, _abi.Tuning(0, 0, 0, 0))
    assert none == default
