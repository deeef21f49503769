"""A look-back's wait is bounded, so a tile must not do work of the input's length before it
publishes: no kernel that looks back walks LCP intervals or compares suffixes to their end.  Read
from the sources, without a GPU."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1404_3456_amd", "csrc")
UNBOUNDED = ("walk_read(", "cmp_suffix(")


def kernels():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\s*\(", text):
            body = text[m.end():text.index("\n}\n", m.end())]
            if "lookback_" in body:
                yield m.group(1), body


def test_the_kernels_are_found():
    assert {"k_ovl_reads", "k_ovl_rows", "k_onesweep", "k_rank_update"} <= {name for name, _ in kernels()}


@pytest.mark.parametrize("name, body", list(kernels()), ids=[n for n, _ in kernels()])
def test_work_before_publishing_is_bounded(name, body):
    for call in UNBOUNDED:
        assert call not in body, f"{name} looks back after {call}...)"
