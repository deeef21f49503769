"""The timing records of a build's first round: its run sort's units are the text's suffixes, once,
also where a run too long for LDS makes the build start over; and they are part of "keyruns"."""
import numpy as np
import pytest

from paper_1404_3456_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("copies, launches", [(20, 1), (400, 2)])
def test_first_run_sort_is_counted_once(copies, launches):
    import paper_1404_3456_amd as lib
    lib.load()
    rng = np.random.default_rng([synth.SEED_BASE, 809])
    word = lambda: rng.choice(list("ACGT"), 120).tobytes().decode().replace("\0", "")  # noqa: E731
    text = synth.text_from_strings([word()] * copies + [word() for _ in range(300)])
    t = torch.from_numpy(text).cuda()
    lib.sa_timing_reset()
    lib.sa_timing_enable(True)
    try:
        lib.sa_build(t)
    finally:
        lib.sa_timing_enable(False)
    got, ms, moved = lib.sa_timing_get("first_runs")
    assert got == launches and ms > 0
    assert lib.sa_timing_items("first_runs") == text.size
    assert moved == 24.0 * text.size
    assert lib.sa_timing_get("keyruns")[0] >= launches
    assert lib.sa_timing_items("keyruns") >= text.size
