"""A refused initial state names its first bad cell and leaves the state before as it was.

The field is checked on the device, 256 cells a block: bad cells at the edges of the blocks, one
and several, of every kind that is refused.
"""
import numpy as np
import pytest

from paper_2007_13091_amd import workloads as wl

pytestmark = pytest.mark.gpu

_BAD = {"density": (0, 0.0), "negative density": (0, -1.0), "nan density": (0, np.nan), "infinite density": (0, np.inf),
        "temperature": (4, 0.0), "nan energy": (4, np.nan), "infinite energy": (4, np.inf)}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cells", [(0,), (255,), (256, 300), (511, 512), (599,)])
def test_refused_field_leaves_the_state_before(cells, precision):
    from paper_2007_13091_amd.ugkwp import E_NONPHYS, Solver, UgkwpError

    w = wl.sod(nx=150, ny=2, nz=2, n_ref=30, kn=0.05)
    w.params.sampling = 1
    assert w.mesh.n_cells == 600
    ref, s = (Solver(w.mesh, w.params, precision=precision) for _ in range(2))
    for q in (ref, s):
        q.init_state(w.W0)
        q.step(3)
    for k, (name, (column, value)) in enumerate(_BAD.items()):
        print(f"[gpu-init] {cells} {precision} {name}", flush=True)
        W = w.W0.copy()
        for c in cells:
            W[c, column] = value
        with pytest.raises(UgkwpError, match=rf"init_state: cell {cells[0]} has") as e:
            s.init_state(W)
        assert e.value.status == E_NONPHYS
        if k % 3 == 0:
            assert s.step(1) == ref.step(1)
            np.testing.assert_array_equal(s.moments(0), ref.moments(0))
            np.testing.assert_array_equal(s.moments(1), ref.moments(1))
    # and one that is taken starts a run like the first
    for q in (ref, s):
        q.init_state(w.W0)
    fresh = Solver(w.mesh, w.params, precision=precision)
    fresh.init_state(w.W0)
    assert s.step(2) == ref.step(2) == fresh.step(2)
    np.testing.assert_array_equal(s.moments(0), fresh.moments(0))
    np.testing.assert_array_equal(s.moments(0), ref.moments(0))
