"""The counting sort's scan with the element tasks (tiles of 4096 buckets) and
the queue counters that every step leaves cleared.

Bar: sorting changes nothing in FP64 (bitwise), with bucket counts below, at and
above one tile, one particle, and particles that left through an open boundary;
a captured step replayed equals the same steps called one by one (bitwise)."""
import numpy as np
import pytest

from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("cells,n", [(2, 1), (15, 4000), (16, 4097), (17, 300)])
def test_sorting_changes_nothing(cells, n):
    _gpu()
    from paper_2211_05458_amd.lib import FlexiPart
    w = W.curved_box(cells=cells, N=3, n_particles=n, seed=31, wall_bc=W.BC_OPEN)
    out = []
    for sort in (1, 0, -1):
        g = FlexiPart(w.mesh, w.N, n)
        g.set_fluid_state(w.U)
        g.push(w.x, w.v * 10.0, w.d, w.elem_hint)
        g.step(w.dt, 4, rk=w.rk, drag=w.drag, sort_every=sort)
        out.append(g.read())
    for other in out[1:]:
        for k in out[0]:
            np.testing.assert_array_equal(out[0][k], other[k])


@pytest.mark.parametrize("rk", [0, 1])
def test_captured_step_replays(rk):
    torch = _gpu()
    from paper_2211_05458_amd.lib import FlexiPart
    n = 3000
    w = W.curved_box(cells=6, N=3, n_particles=n, seed=32)
    _, nb = FlexiPart.particle_block_layout(n)
    stream = torch.cuda.Stream()

    def start():
        g = FlexiPart(w.mesh, w.N, n)
        g.set_fluid_state(w.U)
        g.bind_particles(torch.zeros(nb, dtype=torch.uint8, device="cuda"), n)
        g.push(w.x, w.v * 10.0, w.d, w.elem_hint)
        g.step(w.dt, 1, rk=rk, drag=w.drag)
        return g
    with torch.cuda.stream(stream):
        a, b = start(), start()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            a.step(w.dt, 1, rk=rk, drag=w.drag)
        for _ in range(3):
            graph.replay()
            b.step(w.dt, 1, rk=rk, drag=w.drag)
            stream.synchronize()
            torch.cuda.synchronize()
        # replayed steps leave the host's note that the positions moved as the capture set it
        ra, rb = a.read(), b.read()
    for k in ra:
        np.testing.assert_array_equal(ra[k], rb[k])
