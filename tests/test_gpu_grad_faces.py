"""Second order on tetrahedra by the gradient kernel of four faces a cell (every cell of the batch a
tetrahedron) and by that of six (a batch with boxes): the same bits, on one block of cells with
idle lanes and on several, with every kind of boundary, both limiters and both forms."""
import numpy as np
import pytest

from paper_2007_13091_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _tets(name):
    if name == "6-cells":
        return wl.closed_box(n=(1, 1, 1), n_ref=60, kn=0.2, tets=True)
    if name == "walls":
        return wl.closed_box(n=(4, 3, 3), n_ref=40, kn=0.1, bc=wl.BC_DIFFUSE, tets=True, jitter=0.15)
    return wl.free_stream_box(n=(4, 3, 3), U=(0.8, 0.3, 0.1), n_ref=40, kn=0.3, tets=True, jitter=0.15,
                              walls={"zlo": wl.BC(wl.BC_DIFFUSE, Tw=1.0), "zhi": wl.BC(wl.BC_SPECULAR)})


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("recon", [1, 2])
@pytest.mark.parametrize("name", ["6-cells", "walls", "far-field"])
def test_four_and_six_faces_a_cell_give_the_same_bits(name, recon, precision):
    from paper_2007_13091_amd.ugkwp import Solver

    w, box = _tets(name), wl.closed_box(n=(4, 4, 4), n_ref=20)
    for q in (w, box):
        q.params.recon, q.params.sampling = recon, 1
    a = Solver(w.mesh, w.params, precision=precision)
    a.init_state(w.W0)
    b = Solver([w.mesh, box.mesh], [w.params, box.params], precision=precision)
    b.init_state(np.concatenate([w.W0, box.W0]))
    lo, hi = b.instance_cells(0)
    for n in range(4):
        print(f"[gpu-grad-faces] {name} recon {recon} precision {precision} step {n}", flush=True)
        a.step(1)
        b.step(1)
        for k in (0, 1):
            np.testing.assert_array_equal(b.moments(k)[lo:hi], a.moments(k))
