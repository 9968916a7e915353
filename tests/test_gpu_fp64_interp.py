"""The FP64 element kernel's matrix-core interpolation against the per-lane
kernel (no sort: every particle per lane), at the edges of its tiles of 16
particles and 32 particles per task, for every polynomial degree.

Bar: the same bits (the products round like the per-lane kernel's chain of
fused multiply-adds)."""
import numpy as np
import pytest

from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 3, 5, 7])
@pytest.mark.parametrize("n", [1, 16, 17, 33, 300])
def test_same_bits_as_per_lane(N, n):
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if N == 1:
        w = W.config1(n_particles=n, cells=2)
        w.N, w.U = 1, W.uniform_state(w.mesh.n_elem, 1, (0.3, -0.2, 0.1))
    else:
        w = W.curved_box(cells=2, N=N, n_particles=n, seed=61)
    out = []
    for sort in (1, 0):
        g = FlexiPart(w.mesh, w.N, n)
        g.set_fluid_state(w.U)
        g.push(w.x, w.v * 2.0, w.d, w.elem_hint)
        g.step(w.dt, 3, rk=w.rk, drag=w.drag, sort_every=sort)
        out.append(g.read())
    for k in out[0]:
        np.testing.assert_array_equal(out[0][k], out[1][k])
