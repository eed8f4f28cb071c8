"""The particle buffers' layout: regions with empty ends, arrivals behind them, lists of leavers.

* At the tightest capacity that a run fits, the arrivals and new particles run past the end of
  the buffer into the empty slots of the cells' regions; the run must be the one with room to
  spare, bit for bit, and one slot less must be refused.
* Buckets of every path (64 and fewer arrivals, more, more than the sort's local memory; few
  cells per wave and many) against the oracle, at the bar of tests/parity.py.
"""
import numpy as np
import pytest

import oracle
from paper_2007_13091_amd import workloads as wl
from parity import compare_fields, compare_particles, compare_stats
from test_gpu_batch import _run_batch
from test_gpu_parity import run_pair

pytestmark = pytest.mark.gpu


def _solver(w, precision, capacity=0):
    from paper_2007_13091_amd.ugkwp import Solver

    s = Solver(w.mesh, w.params, precision=precision, capacity=capacity)
    s.init_state(w.W0)
    return s


def _case(name):
    if name == "boxes":
        w = wl.sod(nx=11, ny=3, nz=2, n_ref=70, kn=0.05)
        w.params.sampling = 1
        return w
    if name == "tets-inflow":
        return wl.free_stream_box(n=(4, 3, 3), U=(2.5, 0.4, -0.3), T=1.2, n_ref=60, kn=0.1, perturb=0.2, tets=True,
                                  jitter=0.15, walls={"zlo": wl.BC(wl.BC_DIFFUSE, Tw=1.0)})
    if name == "diatomic-walls":
        return wl.closed_box(n=(5, 4, 3), n_ref=50, kn=0.3, bc=wl.BC_DIFFUSE, gamma=1.4)
    w = wl.cavity(n=5, n_ref=60)
    w.params.recon, w.params.sampling, w.params.prandtl = 2, 2, 2.0 / 3.0
    return w


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("case", ["boxes", "tets-inflow", "diatomic-walls", "shakhov"])
def test_tightest_capacity_gives_the_same_run(case, precision):
    from paper_2007_13091_amd.ugkwp import E_CAPACITY, UgkwpError

    w = _case(case)
    roomy = _solver(w, precision, capacity=200 * w.mesh.n_cells + 65536)
    most, steps = 0, []
    for _ in range(7):
        st = roomy.step(1)
        most = max(most, st["n_moved"])
        steps.append((st, roomy.moments(0), roomy.moments(1), roomy.particles()))
    tight = _solver(w, precision, capacity=most)
    for n, (st, W, Wp, p) in enumerate(steps):
        print(f"[gpu-layout] {case} {precision} step {n}: {st['n_moved']} of {most}", flush=True)
        assert tight.step(1) == st
        np.testing.assert_array_equal(tight.moments(0), W)
        np.testing.assert_array_equal(tight.moments(1), Wp)
        q = tight.particles()
        for k in p:
            np.testing.assert_array_equal(q[k], p[k], err_msg=f"step {n} {k}")
    short = _solver(w, precision, capacity=most - 1)
    with pytest.raises(UgkwpError) as e:
        for _ in steps:
            short.step(1)
    assert e.value.status == E_CAPACITY


@pytest.mark.parametrize("name", ["few-cells-many-particles", "many-cells-few-particles", "many-tets"])
def test_buckets_of_every_length(name):
    if name == "few-cells-many-particles":
        # hundreds of arrivals per cell; the masses of the sampled particles are left out: they come from
        # rho - rho^p, and the rounding of the oracle's running sum of 3000 masses is itself above the bar
        w = wl.closed_box(n=(3, 2, 1), n_ref=3000, kn=0.5, perturb=0.1)
        s, o = _solver(w, 0), oracle.Oracle(w.mesh, w.params)
        o.set_state(w.W0)
        vol, _, _ = o.geometry()
        for n in range(3):
            st = s.step(1)
            o.step()
            compare_stats(st, o.stats(), what=f"{name} step {n}")
            Wo, Po, _ = o.state()
            compare_fields(s.moments(0), Wo, s.moments(1) * vol[:, None], Po, vol, what=f"{name} step {n}")
            pg, po = s.particles(), o.particles()
            compare_particles(dict(pg, m=np.ones_like(pg["m"])), dict(po, m=np.ones_like(po["m"])), vscale=3.0,
                              what=f"{name} step {n}")
    elif name == "many-cells-few-particles":  # 16,400 cells: many cells per wave
        run_pair(wl.sod(nx=4100, ny=2, nz=2, n_ref=12, kn=1e-3), 2, name=name, sampling=1)
    else:  # 16,464 tetrahedra
        run_pair(wl.closed_box(n=(14, 14, 14), n_ref=14, kn=0.2, tets=True, jitter=0.1, perturb=0.1), 2, name=name, sampling=1)


@pytest.mark.parametrize("U", [0.0, 0.99, 1.01, 2.99, 3.01, 4.0])
def test_inflow_speeds_on_both_sides_of_the_root_finders_rule(U):
    """Faces with a = U.n / sigma in [-U, U]: the iteration above -3, the plain bisections below."""
    run_pair(wl.free_stream_box(n=(3, 2, 2), U=(U, 0.0, 0.0), n_ref=20, kn=0.5, perturb=0.1), 2, vscale=3.0 + U,
             name=f"inflow U={U}")


@pytest.mark.parametrize("name", ["4096-cells", "4100-cells", "486-far-field-faces", "65-instances"])
def test_prefixes_on_both_sides_of_their_tiles(name):
    """8,192 buckets and a few more (one launch, two); more far-field faces than a block counts;
    more instances than have several words for their time step each."""
    if name == "65-instances":
        _run_batch(wl.small_batch(65), 2, name=name)
    elif name == "486-far-field-faces":
        run_pair(wl.free_stream_box(n=(9, 9, 9), U=(0.6, 0.2, 0.0), n_ref=12, kn=0.5, perturb=0.1), 2, name=name)
    else:
        run_pair(wl.sod(nx=int(name[:4]) // 4, ny=2, nz=2, n_ref=12, kn=1e-3), 2, name=name, sampling=1)
