"""Face intersections of the tracker (Newton with a contraction bound, the
wavefront search of what it leaves open) against the oracle's Bezier clipping:
mild and strong curvature, short paths and paths over a quarter of an element,
fewer segments than a wavefront has lanes and a ragged last wavefront.

Bar: elements, statuses and wall hits equal, the same number of crossings,
positions and velocities within the FP64 parity bound 1e-10."""
import numpy as np
import pytest

import oracle as O
from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(mesh, n):
    if mesh == "box4":
        return W.curved_box(cells=4, N=5, n_particles=n, seed=71)
    return W.config4(n_particles=n, cells=(48, 6, 48), seed=72)


@pytest.mark.parametrize("mesh,n,factor", [("box4", 1, 20.0), ("box4", 65, 20.0), ("box4", 2000, 20.0),
                                           ("passage", 65, 3.0), ("passage", 2000, 3.0)])
def test_crossings_equal_the_oracles(mesh, n, factor):
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = _workload(mesh, n)
    v = w.v * factor
    o = O.Oracle(w.mesh, w.N, w.U)
    o.push(w.x, v, w.d, w.elem_hint)
    o.step(w.dt, 3, rk=w.rk, drag=w.drag)
    ro, so = o.read(), o.stats()
    g = FlexiPart(w.mesh, w.N, n)
    g.set_fluid_state(w.U)
    g.push(w.x, v, w.d, w.elem_hint)
    g.step(w.dt, 3, rk=w.rk, drag=w.drag)
    rg, sg = g.read(), g.stats()
    for k in ("status", "elem", "hits"):
        np.testing.assert_array_equal(rg[k], ro[k])
    for k in ("crossings", "wall_hits", "lost"):
        assert sg[k] == so[k], k
    act = ro["status"] == 0
    assert np.abs(rg["x"] - ro["x"])[act].max(initial=0) <= 1e-10
    assert np.abs(rg["v"] - ro["v"])[act].max(initial=0) <= 1e-10 * max(1.0, factor)
