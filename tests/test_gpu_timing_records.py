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


@pytest.mark.parametrize("copies, scan", [(0, False), (4, False), (30, False), (200, True)])
@pytest.mark.parametrize("use_graph", [False, True])
def test_who_finishes_the_lcp_array(copies, scan, use_graph):
    """Matches past the first round's windows are finished entry by entry while they are few and
    short, by Kasai's scan where that would be the longer way."""
    import oracle
    import paper_1404_3456_amd as lib
    lib.load()
    rng = np.random.default_rng([synth.SEED_BASE, 810])
    word = lambda k: rng.choice(np.frombuffer(b"ACGT", dtype=np.uint8), k).tobytes().decode()  # noqa: E731
    text = synth.text_from_strings([word(700)] * copies + [word(400) for _ in range(60)])
    t = torch.from_numpy(text).cuda()
    lib.sa_timing_reset()
    lib.sa_timing_enable(True)
    try:
        sa, _, lcp = lib.sa_build_batched(t, np.array([0, text.size], dtype=np.int64), lcp=True,
                                          use_graph=use_graph)
    finally:
        lib.sa_timing_enable(False)
    assert lib.sa_timing_get("kasai")[0] == (1 if scan else 0)
    assert lib.sa_timing_get("lcp_rest")[0] == (1 if copies and not scan else 0)
    want = oracle.suffix_array(text)
    assert np.array_equal(sa.cpu().numpy(), want)
    assert np.array_equal(lcp.cpu().numpy(), oracle.lcp_array(text, want))
