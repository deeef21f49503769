"""The benchmark's per-kernel table, without a GPU: every kernel of a build has a key of its own
with a byte figure, and the first round's run sort is not averaged with the doubling rounds'."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def load_bench():
    sys.path.insert(0, ROOT)
    try:
        import bench
    finally:
        sys.path.remove(ROOT)
    return bench


class Timing:
    """What the library files for a build: two launches of 1 us under "keyruns" beside one of 3 ms
    that is under "first_runs" too."""
    got = {"first_runs": (1, 3.0, 2.4e9), "keyruns": (3, 3.002, 2.4e9 + 480.0)}
    items = {"first_runs": 1e8, "keyruns": 1e8 + 20.0}

    def sa_timing_get(self, key):
        return self.got.get(key, (0, 0.0, 0.0))

    def sa_timing_items(self, key):
        return self.items.get(key, 0.0)


def test_run_sorts_apart():
    bench = load_bench()
    table = bench.kernel_table(Timing(), bench.BUILD_KEYS, 1)
    assert table["first_runs"]["avg_us"] == 3000.0 and table["first_runs"]["units_per_step"] == 10 ** 8
    assert table["keyruns"]["launches_per_step"] == 2.0 and table["keyruns"]["units_per_step"] == 20
    assert table["keyruns"]["avg_us"] == 1.0
    assert sum(e["units_per_step"] for e in table.values()) == 10 ** 8 + 20  # counted once


def test_no_doubling_round():
    bench = load_bench()
    t = Timing()
    t.got = {"first_runs": (2, 6.0, 4.8e9), "keyruns": (2, 6.01, 4.8e9)}
    t.items = {"first_runs": 2e8, "keyruns": 2e8}
    assert "keyruns" not in bench.kernel_table(t, bench.KEYS, 2)


def test_build_keys():
    bench = load_bench()
    assert {"first_extract", "first_runs"} <= set(bench.BUILD_KEYS) <= set(bench.KEYS)
    assert all(bench.SURVEY_BYTES[k] > 0 for k in bench.BUILD_KEYS)


def test_traffic_records_are_of_one_workload_and_its_sources(tmp_path):
    import hashlib
    import json
    from types import SimpleNamespace
    bench = load_bench()
    csrc = os.path.join(ROOT, "paper_1404_3456_amd", "csrc")
    files = ("first_round.hip", "text.hpp", "device.hpp", "internal.hpp")
    h = hashlib.sha256(b"".join(open(os.path.join(csrc, f), "rb").read() for f in files)).hexdigest()
    record = {"bytes_per_launch": 7, "source_sha256": h, "workload": "plain-large-5M"}
    args = SimpleNamespace(traffic_dir=str(tmp_path), workload="plain-large-5M", sa_algo="doubling")
    path = tmp_path / "first_runs_traffic.json"
    path.write_text(json.dumps(record))
    assert bench.traffic_for(args, "first_runs", None) == 7
    args.workload = "repeat-stress-40M"
    assert bench.traffic_for(args, "first_runs", None) is None
    args.workload = "plain-large-5M"
    path.write_text(json.dumps({**record, "source_sha256": "0"}))
    assert bench.traffic_for(args, "first_runs", None) is None
