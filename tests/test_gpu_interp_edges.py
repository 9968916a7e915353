"""The FP64 element kernel's matrix-core interpolation at the edges of its tiles
(16 particles) and tasks (32 particles, 64 for geometry degree 6): exact counts
in one element, and in a second one that shares its wavefront, with a state that
differs from node to node, for every compiled pair of degrees.

Bar: the bits of the per-lane kernel (no sort)."""
import numpy as np
import pytest

import oracle as O
from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu


def _state(E, N, seed):
    rng = np.random.default_rng(seed)
    U = np.empty((E, 5, (N + 1) ** 3))
    U[:, 0] = W.RHO_F * rng.uniform(0.8, 1.2, U[:, 0].shape)
    U[:, 1:4] = rng.uniform(-1.0, 1.0, U[:, 1:4].shape)
    U[:, 4] = W.P0 / (W.KAPPA - 1.0)
    return U


def _mesh(ng):
    return W.config1(n_particles=1, cells=2).mesh if ng == 1 else W.sine_mesh(2, ng)


@pytest.mark.parametrize("N,ng,counts", [
    (N, ng, c) for N, ng in ((1, 1), (3, 1), (3, 4), (5, 4), (7, 4)) for c in ((15, 0), (16, 17), (31, 1), (32, 33), (65, 16))
] + [(5, 6, c) for c in ((31, 32), (33, 0), (48, 49), (64, 63), (65, 1), (129, 80))])
def test_same_bits_as_per_lane(N, ng, counts):
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mesh = _mesh(ng)
    U = _state(mesh.n_elem, N, 10 * N + ng)
    o = O.Oracle(mesh, N, U)
    rng = np.random.default_rng(sum(counts) + 7 * N)
    hint = np.array([2] * counts[0] + [5] * counts[1], np.int32)
    x = np.array([o.map(int(e), rng.uniform(-0.9, 0.9, 3))[0] for e in hint])
    v = rng.normal(size=x.shape)
    d = np.full(len(x), 1e-4)
    out = []
    for sort in (1, 0):
        g = FlexiPart(mesh, N, len(x))
        g.set_fluid_state(U)
        g.push(x, v, d, hint)
        g.step(1e-4, 2, rk=1, drag=1, sort_every=sort)
        out.append(g.read())
    assert (out[0]["status"] == 0).all()
    for k in out[0]:
        np.testing.assert_array_equal(out[0][k], out[1][k])
