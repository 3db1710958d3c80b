"""The benchmark's stored counter passes and its count of multiplied operations,
without a GPU: a pass holds only for the sources it was taken on, all of those
that choose, launch and are the call's kernels."""
import os

import bench

CSRC = "paper_2405_04463_amd/csrc/"


def test_a_pass_names_every_source_of_its_call():
    for stored in bench.CALL_TRAFFIC.values():
        assert {os.path.basename(f) for f in stored["sources"]} == {
            "pair_dot.hip", "rot_dot.hip", "dot.hip", "plan.h", "launch.h", "api.cpp", "device.h"}
        assert all(os.path.exists(os.path.join(bench.ROOT, f)) for f in stored["sources"])


def test_a_pass_holds_only_for_its_sources(monkeypatch):
    t = bench.call_traffic(1984, 300_000, 0)
    # pairs: the sums read the database tile whole, the other two products half of it each
    assert t is None or t >= 2 * 300_000 * 102_400
    for f in bench.CALL_TRAFFIC[0]["sources"]:
        changed = dict(bench.CALL_TRAFFIC[0], sources=dict(bench.CALL_TRAFFIC[0]["sources"], **{f: "0" * 64}))
        monkeypatch.setitem(bench.CALL_TRAFFIC, 0, changed)
        assert bench.call_traffic(1984, 300_000, 0) is None, f
        monkeypatch.undo()
    assert bench.call_traffic(1984, 300_001, 0) is None and bench.call_traffic(1984, 300_000, 1) is None


def test_no_result_reports_the_record_of_another_kernel():
    src = open(os.path.join(bench.ROOT, "bench.py")).read()
    assert "one_pass_kernel_traffic" not in src
    assert src.count("DOT_TRAFFIC") == 2        # the record and the default of the function that reads one


def test_multiplied_operations():
    rot = list(range(-15, 16))
    assert bench.multiplied_share(rot, 0) == 24 / 31
    assert bench.multiplied_share(rot[:27], 0) == 24 / 27
    assert bench.multiplied_share(rot[:26], 0) == bench.multiplied_share(rot, 4) == 1
    assert bench.multiplied_share(rot[::-1], 0) == 1
