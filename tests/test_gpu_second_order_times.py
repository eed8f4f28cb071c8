"""The second order's kernels are chosen by the number of faces so that a smaller mesh is not the slower
one: its gradients and fluxes take no longer (beyond the timing's scatter) than a larger mesh's."""
import numpy as np
import pytest

from paper_2007_13091_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _flux_us(n, precision):
    from paper_2007_13091_amd.ugkwp import Solver

    w = wl.closed_box(n=(n, n, n), n_ref=50, bc=wl.BC_DIFFUSE, perturb=0.05)
    w.params.recon, w.params.gks_steps = 2, 1 << 30
    s = Solver(w.mesh, w.params, precision=precision, capacity=65536)
    s.init_state(w.W0)
    s.step(5)
    s.profile(True, slots=["flux"])
    best = np.inf
    for _ in range(8):
        s.profile_read()
        s.step(8)
        ms, k = s.profile_read()["flux"]
        best = min(best, 1e3 * ms / k)
    s.close()
    return best


@pytest.mark.parametrize("precision", [0, 1])
def test_fewer_faces_do_not_take_longer(precision):
    large = _flux_us(22, precision)  # 33,396 faces
    for n in (14, 15, 16, 18, 19):  # 8,820 to 21,660 faces, on both sides of the limit
        us = _flux_us(n, precision)
        print(f"[gpu-second-order] {n}^3 boxes: {us:.1f} us, 22^3 boxes {large:.1f}", flush=True)
        assert us < 1.15 * large
