"""CPU check of the bench's output: with every leg run and 64 instances' errors at hand it prints one
JSON line short enough for a record of 8,000 characters, the headline value to every digit."""
import json
import sys

import pytest

from test_bench_host import _bench

X = 12345678901.234567 / 7.0  # a float of full length


def _roof(kernel):
    return {"bound": "hbm", "achieved": 4058.6, "peak": 8000.0, "unit": "GB/s", "frac": 0.5073, "traffic": 123456789012,
            "kernel": kernel, "kernel_avg_ms": 17.8035, "algorithmic_bytes_per_launch": 72257469824}


def _whole():
    return {"bound": "hbm", "achieved": 2791.3, "peak": 8000.0, "unit": "GB/s", "frac": 0.3489,
            "algorithmic_bytes_per_step": 72994881488}


def _err():
    return {q: {"L1": 8.279356297214774e-07, "Linf": 0.0020164927864305656} for q in ("rho", "U", "T")}


def _batch(*_a, **_k):
    kernels = {"stream": _roof("k_stream<float, 128, true, 2>"), "gather": _roof("k_gather_sparse<float, 1, false>")}
    worst = {q: 4.2143349174107074e-05 for q in ("rho", "U", "T")}
    b = {"value": X, "ms_per_step": X / 1e9, "cell_steps_per_s": X / 17, "particles_per_step": 828153306, "steps": 20,
         "timed_after_step": 105, "launch_config": {"stream_bs": 128, "stream_ilp": 2, "sample_wpb": 4, "flux_bs": 64},
         "dominant": "stream", "kernels": kernels, "whole_step": _whole(),
         "flux": dict(_roof("k_flux<float, 64>"), bytes_per_face=144, faces=10074636, timed="the warm-up steps"),
         "graph_replay_ms_per_step": 26.6465, "cells": 2793226, "instances": 64,
         "fp64_plain_one_by_one": {"value": X / 3, "unit": "particle moves/s", "cell_steps_per_s": X / 29, "ms_per_step": X / 5e8,
                                   "kernel_ms_per_step_sum": {"stream": 23.4567, "gather": 9.8765}, "whole_step": _whole(),
                                   "kernels": {q: _roof("x") for q in ("stream", "gather")}},
         "speedup_vs_fp64_plain_one_by_one": 1.9876543210987,
         "stated_error": {"protocol": "p" * 330, "worst_over_instances_L1": worst, "worst_over_instances_Linf": worst,
                          "decision_flips": 1234,
                          "per_instance": [{"instance": k, "cells": 59319, "n_ref": 493, "mu_ref": 0.8458282596175564,
                                            "step": 126, **_err()} for k in range(64)]}}
    return b, [1]


def _cavity(*_a, **_k):
    return {"value": X, "unit": "particle moves/s", "ms_per_step": 0.8536301499994181, "cell_steps_per_s": X / 401,
            "particles_per_step": 14016418, "steps": 20, "timed_after_step": 1005, "dominant": "stream",
            "kernels": {"stream": _roof("k_stream<double, 256, false, 1>"), "gather": _roof("k_gather<double, 1, false>")},
            "whole_step": _whole()}


def _gks(*_a):
    slots = ("prim_dt", "cell_prep", "scan_sample", "flux", "sample", "stream", "stream_wall", "count", "scan_buckets",
             "scatter", "gather", "finalize")
    return {"workload": "w" * 87, "cell_steps_per_s": X / 21, "ms_per_step": X / 3e10, "steps": 20, "particles_per_step": 0,
            "capacity": 65536, "kernel_ms_per_step": {k: 0.0143 for k in slots}, "flux_roofline": _roof("k_flux<double, 128>")}


def _avg(*_a):
    return {"workload": "w" * 69, "ms_per_step": X / 2e9, "ms_per_step_without": X / 3e9, "steps_averaged": 25,
            "last_relative_change": 0.0038482448838895243, "averaging_kernels_ms": 0.0095,
            "roofline": dict(_whole(), bytes_per_cell=128, cells=32768)}


def _cpu(_sample):
    return {"value": X / 200, "unit": "particle moves/s", "cores": 16, "kind": "oracle", "build": "b" * 82, "cpu_model": "AMD EPYC",
            "cell_steps_per_s": X / 1e4, "single_core": {"value": X / 700, "cores": 1, "seconds": 13.15, "cell_steps_per_s": X / 1e5},
            "sample": "s" * 330}


@pytest.fixture
def bench(monkeypatch):
    b = _bench()
    for name, f in (("batched_run", _batch), ("cavity_leg", _cavity), ("gks_side", _gks), ("averaging_side", _avg),
                    ("cpu_baseline", _cpu)):
        monkeypatch.setattr(b, name, f)
    return b


def test_one_short_line_with_the_headline(bench, monkeypatch, capsys):
    monkeypatch.setattr(sys, "argv", ["bench.py"])
    bench.main()
    text = capsys.readouterr().out
    assert text.count("\n") == 1 and len(text) < 8000, len(text)
    d = json.loads(text)
    assert d["value"] == X and d["ms_per_step"] == X / 1e9 and d["n_gpus"] == 1 and d["steps"] == 20
    assert d["roofline"]["peak"] == 8000.0 and d["roofline"]["unit"] == "GB/s"
    assert d["stated_error"]["worst_over_instances_L1"]["T"] == pytest.approx(4.21433e-5, rel=1e-5)
    # every leg is there
    assert d["cavity32"]["fp32_form"]["ms_per_step"] == pytest.approx(0.85363, rel=1e-5)
    assert d["gks_limit"]["ms_per_step"] > 0 and d["time_averaging"]["steps_averaged"] == 25
    assert d["cpu_baseline"]["unit"] == "particle moves/s"


def test_the_full_record_keeps_every_instance(bench, monkeypatch, capsys, tmp_path):
    path = tmp_path / "full.json"
    monkeypatch.setattr(sys, "argv", ["bench.py", "--full", str(path)])
    bench.main()
    assert capsys.readouterr().out.count("\n") == 1
    d = json.loads(path.read_text())
    assert len(d["stated_error"]["per_instance"]) == 64 and d["cavity32"]["fp64_plain"]["value"] == X
