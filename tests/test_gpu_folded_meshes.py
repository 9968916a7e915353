"""Tracking on meshes with faces that Newton's search does not serve, against the
oracle: many of them (all segments clipped: the annular passage meshed far too
coarsely), and a few (only the segments that meet one are clipped: one element
edge compressed 2.5 times in a box of 3 x 2 x 9 elements), particles that meet
the faces and others that do not, reflections, sorted or not.

Bar: elements, statuses, wall hits and crossings equal; positions within the
FP64 parity bound 1e-10 times the faces' stretch, 2.5, where a few faces are
compressed, and 1e-10 times 125, the ratio of second derivative to smallest
tangent, on the passage."""
import numpy as np
import pytest

import oracle as O
from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu

N_GEO, SQUEEZE = 4, 0.6


def _squeezed_box(n, seed):
    """Unit cells; the edge y = 1, x in [1, 2] of the middle slice squeezed."""
    cells = (3, 2, 9)

    def node_map(I1, I2, I3, M):
        shp = np.broadcast_shapes(I1.shape, I2.shape, I3.shape)
        out = np.empty(shp + (3,))
        x, y, z = (np.broadcast_to(I / N_GEO, shp) for I in (I1, I2, I3))
        # mild curvature away from the walls
        out[..., 0] = x + 0.02 * np.sin(np.pi * x / 3) * np.sin(np.pi * y / 2) * np.sin(np.pi * z / 9)
        out[..., 1] = y
        out[..., 2] = z
        return out
    X, ne, nf, bc, shift, _ = W.structured_mesh(cells, N_GEO, node_map, (False, False, False))
    ng, m = N_GEO + 1, N_GEO // 2
    X = X.reshape(-1, ng, ng, ng, 3)
    b = 1 + 3 * (0 + 2 * 4)
    X[b, m, -1, m, 0] -= SQUEEZE / 12.0
    X[b + 3, m, 0, m, 0] -= SQUEEZE / 12.0
    mesh = W.Mesh(N_GEO, X.reshape(len(X), -1, 3), ne, nf, bc, shift, 1.0, cells)
    rng = np.random.default_rng(seed)
    o = O.Oracle(mesh, 3, W.uniform_state(mesh.n_elem, 3, (0.0, 0.0, 0.0)))
    half = n // 2                       # half of them near the squeezed edge, moving across it
    hint = rng.integers(mesh.n_elem, size=n)
    hint[:half] = np.where(rng.random(half) < 0.5, b, b + 3)
    xi = rng.uniform(-0.98, 0.98, (n, 3))
    xi[:half] = rng.uniform([-0.4, 0.8, -0.6], [0.98, 0.98, 0.6], (half, 3))
    up = hint[:half] == b + 3
    xi[:half, 1] *= np.where(up, -1.0, 1.0)
    x = np.array([o.map(int(e), a)[0] for e, a in zip(hint, xi)])
    v = rng.normal(size=(n, 3)) * 120.0
    v[:half, 1] = np.where(up, -1.0, 1.0) * rng.uniform(50.0, 400.0, half)
    return mesh, x, v, np.full(n, 1e-5), hint.astype(np.int32)


def _compare(mesh, N, U, x, v, d, hint, dt, tol, **opt):
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    o = O.Oracle(mesh, N, U)
    o.push(x, v, d, hint)
    o.step(dt, 2, rk=1, drag=2)
    ro, so = o.read(), o.stats()
    g = FlexiPart(mesh, N, len(x))
    g.set_fluid_state(U)
    g.push(x, v, d, hint)
    g.step(dt, 2, rk=1, drag=2, **opt)
    rg, sg = g.read(), g.stats()
    for k in ("status", "elem", "hits"):
        np.testing.assert_array_equal(rg[k], ro[k])
    for k in ("crossings", "wall_hits", "lost"):
        assert sg[k] == so[k], k
    assert np.abs(rg["x"] - ro["x"]).max() <= tol
    return so


@pytest.mark.parametrize("sort", [0, 1, -1])
@pytest.mark.parametrize("n", [1, 64, 3000])
def test_a_few_folded_faces(n, sort):
    mesh, x, v, d, hint = _squeezed_box(n, 5 + n)
    so = _compare(mesh, 3, W.uniform_state(mesh.n_elem, 3, (0.0, 0.0, 0.0)), x, v, d, hint, 1e-3, 2.5e-10,
                  sort_every=sort)
    if n >= 64:
        assert so["crossings"] > n // 8
    if n >= 3000:
        assert so["wall_hits"] > 100


@pytest.mark.parametrize("cells,n", [(8, 1), (12, 500), (16, 2000), (24, 500)])
def test_many_folded_faces(cells, n):
    w = W.config4(n_particles=n, cells=(cells, 4, cells), seed=90 + cells)
    so = _compare(w.mesh, w.N, w.U, w.x, w.v * 10.0, w.d, w.elem_hint, w.dt, 1.25e-8)
    if n >= 500:
        assert so["crossings"] > n // 8


def test_folded_faces_do_not_hold_up_a_step():
    """500 fast particles on the 8 x 4 x 8 passage: tracking takes 10 ms of a
    step by clipping and took 100 ms where Newton's search was left to split
    those faces into parts; the bar lies between, the best of five steps."""
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = W.config4(n_particles=500, cells=(8, 4, 8))
    g = FlexiPart(w.mesh, w.N, 500)
    g.set_fluid_state(w.U)
    g.push(w.x, w.v * 10.0, w.d, w.elem_hint)
    g.set_timing(True)
    best = 1e300
    for _ in range(5):
        g.step(w.dt, 1, rk=1, drag=w.drag)
        best = min(best, g.timing()["track"][1])
    print("tracking of a step: %.2f ms" % best)
    assert best < 35.0
