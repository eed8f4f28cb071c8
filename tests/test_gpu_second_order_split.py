"""Second order on few faces and on many: the two kernels give the same bits.

A mesh of few faces shares each group of faces among three waves, a larger one does not.  A
batch is one mesh to the kernels, so instances alone (few faces) and in one batch (many) take the
two paths; without particles they are bitwise equal, and the batch with particles is the
oracle's at the bar of tests/parity.py.  Faces of every kind: inner,
specular, diffuse, free stream, of boxes and of tetrahedra; both limiters; the Shakhov energy term;
internal degrees of freedom; a first-order instance among the others.
"""
import numpy as np
import pytest

from paper_2007_13091_amd import workloads as wl
from test_gpu_batch import _run_batch

pytestmark = pytest.mark.gpu

MOST_SPLIT = 64 * 1024 // 3  # faces


def _instances(name):
    def one(k):
        if name == "boxes":
            w = wl.free_stream_box(n=(9, 8, 9), U=(0.8, 0.4, -0.3), T=1.2, n_ref=120, kn=0.1, perturb=0.2,
                                   walls={"zlo": wl.BC(wl.BC_DIFFUSE, Tw=1.0), "zhi": wl.BC(wl.BC_SPECULAR)})
            w.params.prandtl = 2.0 / 3.0
        else:
            w = wl.closed_box(n=(6, 5, 4), n_ref=120, kn=0.3, bc=wl.BC_DIFFUSE, gamma=1.4, tets=True)
        w.params.recon = (1, 2, 0)[k % 3] if k < 3 else 2
        if name == "boxes":
            w.params.sampling = 2 if w.params.recon else 3
        w.params.seed = 100 + k
        return w

    m = one(0).mesh
    nf = (int(np.where(m.cell_type == 8, 6, 4).sum()) + m.bface_nodes.shape[0]) // 2
    assert nf < MOST_SPLIT
    return [one(k) for k in range(MOST_SPLIT // nf + 2)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["boxes", "tets"])
def test_wave_only_steps_alone_and_in_a_batch_are_bitwise_equal(name, precision):
    from paper_2007_13091_amd.ugkwp import Solver

    ws, steps = _instances(name), 4
    for w in ws:
        w.params.gks_steps = steps  # no particles, whose numbers a batch gives out in common
    b = Solver([w.mesh for w in ws], [w.params for w in ws], precision=precision)
    b.init_state(np.concatenate([w.W0 for w in ws]))
    b.step(steps)
    Wb = b.moments(0)
    first = np.cumsum([0] + [w.mesh.n_cells for w in ws])
    for k in (0, 1, 2, len(ws) - 1):
        w = ws[k]
        print(f"[gpu-second-order] {name} {precision} instance {k}", flush=True)
        s = Solver(w.mesh, w.params, precision=precision)
        s.init_state(w.W0)
        s.step(steps)
        np.testing.assert_array_equal(s.moments(0), Wb[first[k]:first[k + 1]])


@pytest.mark.parametrize("name", ["boxes", "tets"])
def test_many_faces_with_particles_match_the_oracle(name):
    _run_batch(_instances(name), 3, name=f"many-faces {name}")
