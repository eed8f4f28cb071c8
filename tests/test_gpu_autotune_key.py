"""The autotuner's cache answers only for the kernels that were timed: a line that another build's
kernels left, or one of a workload that takes other kernels on the same mesh, is a miss."""
import json

import pytest

from paper_2007_13091_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _solver(n_ref):
    from paper_2007_13091_amd.ugkwp import Solver

    w = wl.closed_box(n=(4, 3, 2), n_ref=n_ref)
    s = Solver(w.mesh, w.params, capacity=100000)
    s.init_state(w.W0)
    return w, s


def test_a_line_without_the_kernels_version_misses(tmp_path):
    import torch

    w, s = _solver(60)
    nc = w.mesh.n_cells
    faces = (6 * nc + len(w.mesh.bface_bc)) // 2
    arch = torch.cuda.get_device_properties(0).gcnArchName
    key = f"{arch} prec=0 K=0 inst=1 cells={nc} faces={faces} cap=100000 modes=00"
    cache = tmp_path / "tune.jsonl"
    cache.write_text(json.dumps({"key": key, "launch": [512, 2, 8, 64]}) + "\n")
    _, hit = s.autotune(steps_per_trial=1, cache=cache)
    assert not hit and s.step(0)["step"] == 26
    # the appended line is this workload's, and a hit from now on
    lines = [json.loads(ln) for ln in cache.read_text().splitlines()]
    assert len(lines) == 2 and lines[1]["key"].endswith(key[len(arch):]) and lines[1]["key"] != key
    assert _solver(60)[1].autotune(steps_per_trial=1, cache=cache) == (tuple(lines[1]["launch"]), True)


def test_another_particle_number_that_takes_other_kernels_misses(tmp_path):
    cache = tmp_path / "tune.jsonl"
    assert not _solver(60)[1].autotune(steps_per_trial=1, cache=cache)[1]
    assert not _solver(1000)[1].autotune(steps_per_trial=1, cache=cache)[1]
    assert _solver(1000)[1].autotune(steps_per_trial=1, cache=cache)[1]
