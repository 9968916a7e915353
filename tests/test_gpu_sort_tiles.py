"""The counting sort at the edges of its scan tiles (4096 buckets: the elements
and one for the particles that left): 4095 elements fill one tile, 4096 take a
second one, 8191 and 8192 two and three.

Bar: sorting changes nothing in FP64 (bitwise)."""
import numpy as np
import pytest

from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu


def _box(cells):
    periods = [[float(cells[0]), 0.0, 0.0], [0.0, 0.0, 0.0], [0.0, 0.0, 0.0]]

    def node_map(I1, I2, I3, M):
        shp = np.broadcast_shapes(I1.shape, I2.shape, I3.shape)
        return np.stack([np.broadcast_to(I, shp).astype(np.float64) for I in (I1, I2, I3)], -1)
    X, ne, nf, bc, shift, _ = W.structured_mesh(cells, 1, node_map, (True, False, False), wall_bc=W.BC_OPEN,
                                                periods=periods)
    return W.Mesh(1, X, ne, nf, bc, shift, 1.0, cells)


@pytest.mark.parametrize("cells", [(13, 15, 21), (16, 16, 16), (1, 1, 8191), (32, 16, 16)])
def test_sorting_changes_nothing(cells):
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mesh = _box(cells)
    n, E = 6000, mesh.n_elem
    rng = np.random.default_rng(E)
    c = np.array(cells)
    x = rng.uniform(0.0, 1.0, (n, 3)) * c
    x[:200] = c - rng.uniform(0.0, 1.0, (200, 3))      # the last element, by an open corner
    e = np.minimum(np.floor(x).astype(int), c - 1)
    hint = (e[:, 0] + cells[0] * (e[:, 1] + cells[1] * e[:, 2])).astype(np.int32)
    v = rng.normal(size=(n, 3)) * 2000.0
    U = W.uniform_state(E, 1, (0.3, -0.2, 0.1))
    out = []
    for sort in (1, 0, -1):
        g = FlexiPart(mesh, 1, n)
        g.set_fluid_state(U)
        g.push(x, v, np.full(n, 1e-2), hint)
        g.step(1e-4, 3, rk=1, drag=1, sort_every=sort)
        out.append(g.read())
    left = (out[0]["status"] == 1).sum()
    assert 20 < left < n // 2 and (hint == E - 1).sum() >= 200
    for other in out[1:]:
        for k in out[0]:
            np.testing.assert_array_equal(out[0][k], other[k])
