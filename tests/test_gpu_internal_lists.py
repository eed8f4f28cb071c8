"""Internal degrees of freedom (K = 2) where the kernels over the lists and buckets take eight cells
per wave (16,384 cells or more, few particles each) and the sampling too (32,768 cells): against
the oracle at the bar of tests/parity.py, with diffuse walls, where a particle's internal energy
is drawn anew on its way; the FP32 form by its one-step error (rounding only: far below the
difference between two seeds)."""
import pytest

from paper_2007_13091_amd import workloads as wl
from test_gpu_fp32 import _runs
from test_gpu_parity import run_pair

pytestmark = pytest.mark.gpu


def _case(name):
    kw = dict(kn=0.2, bc=wl.BC_DIFFUSE, perturb=0.1, gamma=1.4)
    if name == "17576-boxes":
        return wl.closed_box(n=(26, 26, 26), n_ref=16, **kw)
    if name == "16464-tets":
        return wl.closed_box(n=(14, 14, 14), n_ref=16, tets=True, jitter=0.1, **kw)
    return wl.closed_box(n=(33, 32, 32), n_ref=16, **kw)  # "33792-boxes"


@pytest.mark.parametrize("name", ["17576-boxes", "16464-tets", "33792-boxes"])
def test_diatomic_many_cells_against_the_oracle(name):
    s, _ = run_pair(_case(name), 2, name=name, sampling=1)
    assert s.step(0)["wall_hits"] > 0


@pytest.mark.parametrize("name", ["17576-boxes", "16464-tets", "33792-boxes"])
def test_diatomic_many_cells_fp32_error(name):
    w = _case(name)
    w.params.sampling = 1
    row = _runs(w, 1, 1)[0]
    for q in ("rho", "U", "T"):
        assert row["fp32_vs_oracle"][q]["L1"] <= 0.05 * row["noise_floor"][q]["L1"], (q, row)
