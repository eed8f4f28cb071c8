"""CPU checks of the bytes that bench.py charges to the particles: the records as the kernels' header
lays them out, read once a move and written once a survivor, without a cell index."""
import os
import re

import pytest

from test_bench_host import ROOT, _bench


def test_record_bytes_are_the_headers():
    src = open(os.path.join(ROOT, "paper_2007_13091_amd", "csrc", "device_common.hpp")).read()
    size = {"double": 8, "float": 4, "uint64_t": 8}

    def of(struct):
        body = re.search(r"struct alignas\(\d+\) " + struct + r" \{(.*?)\};", src, re.S).group(1)
        return sum(size[t] * int(n or 1) for t, n in re.findall(r"^\s*(\w+) \w+(?:\[(\d+)\])?;", body, re.M))

    b = _bench()
    assert b.RECORD_BYTES == {"double": of("PRec"), "float": of("PRec32") + 4}  # (the FP32 form's mass lies beside)


@pytest.mark.parametrize("rtype,rec", [("double", 64), ("float", 36)])
def test_a_dropped_particle_is_read_and_not_written(rtype, rec):
    b = _bench()
    moves, alive = 1e6, 7e5
    _, kr = b.kernel_roofline({"stream": 0.02, "gather": 0.01}, moves, {"n_alive": alive, "n_collided": 3e5}, rtype,
                              {"stream": "k_stream", "gather": "k_gather"}, "none")
    kr = b.charge_transport_alone(kr, rtype, moves, alive)
    n = rec * 1700000
    assert kr["stream"]["algorithmic_bytes_per_launch"] == n
    assert kr["stream"]["achieved"] == round(n / 0.02e-3 / 1e9, 1)
    assert kr["stream"]["frac"] == round(n / 0.02e-3 / 1e9 / 8000.0, 4)
    assert kr["gather"]["achieved"] is None and kr["gather"]["kernel_avg_ms"] == 0.01
    ws = b.whole_step(1.0, moves, 1000, rtype, survivors=alive)
    assert ws["algorithmic_bytes_per_step"] == n + 1000 * b.BYTES_PER_CELL[("hex", rtype, 0)]


def test_measured_traffic_is_that_of_the_timed_group(monkeypatch):
    b = _bench()
    held = {"k_stream<float, 256, true, 1>": 5, "k_track<float, false, 1, 8>": 7}
    monkeypatch.setattr(b, "measured_traffic", lambda k, w: held.get(k) if w == "here" else None)
    names = {"stream": "k_stream<float, 256, true, 1>", "gather": "k_gather"}
    for workload, want in (("here", 12), ("elsewhere", None)):
        _, kr = b.kernel_roofline({"stream": 1.0, "gather": 1.0}, 10, {"n_alive": 9, "n_collided": 1}, "float", names, workload)
        kr = b.charge_transport_alone(kr, "float", 10, 9, b.track_name("float", sparse=True), workload)
        assert kr["stream"]["traffic"] == want and kr["stream"]["kernel"].endswith("+ k_track<float, false, 1, 8>")
    src = open(os.path.join(ROOT, "paper_2007_13091_amd", "csrc", "kernels.hip")).read()
    assert "kListCellsSparse = 8, kListCellsDense = 2" in src
    assert "k_track<R, KE, MESH, kListCellsSparse><<<" in src
