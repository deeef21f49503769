"""The pinned words a thread reads device results through go to other threads when it ends: a
program with a thread for every request holds no more of them than threads at once.  Threads that
take them over, at once and after a failed build, get their own results."""
import threading

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


def in_threads(calls):
    failed = []

    def guarded(f):
        try:
            f()
        except BaseException as e:  # shown by the caller's thread
            failed.append(e)

    threads = [threading.Thread(target=guarded, args=(f,)) for f in calls]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed[0]


def mappings():
    with open("/proc/self/maps") as f:
        return sum(1 for _ in f)


def test_ended_threads_leave_theirs(lib):
    text = torch.from_numpy(synth.text_from_strings(["ACGT", "GATT"])).cuda()
    sa, _ = lib.sa_build(text)
    calls = [lambda: lib.sa_lookup(text, sa, [b"A"]), lambda: lib.sa_build(text),
             lambda: lib.sa_build_dc3(text)]
    for f in calls:
        in_threads([f])
    before = mappings()
    for _ in range(50):
        for f in calls:
            in_threads([f])
    assert mappings() - before < 30  # one page a thread would be 150


def test_results_of_threads_at_once(lib):
    texts = [synth.genome_reads(9800 + k, 500 + 300 * k, 30 + 5 * k, 90) for k in range(8)]
    want = [oracle.suffix_array(t) for t in texts]
    bad = texts[0].copy()
    bad[7] = ord("N")

    def build(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            t = torch.from_numpy(texts[k]).cuda()
            for _ in range(5):
                sa, isa = lib.sa_build(t)
                assert np.array_equal(sa.cpu().numpy(), want[k])

    def fail():
        with pytest.raises(lib.SaasmError):
            lib.sa_build(torch.from_numpy(bad).cuda())

    for _ in range(3):
        in_threads([lambda k=k: build(k) for k in range(8)] + [fail, fail])
