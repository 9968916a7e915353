"""Element tasks of another size than the last sort was for: the shape
source sorts where the steps do not, steps with and without the extra forces
take turns between two sorts, the fluid state changes precision, a captured step
is replayed between sorts for the other size.

Bar: from 2^18 particles on every stage runs the element kernel, below it the
stages whose tasks fit do; the FP64 states are bitwise those of steps that never
sort (per lane)."""
import numpy as np
import pytest

from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu

GRAVITY = (0.0, 0.0, -9.81)
MANY = 1 << 18


def _make(w, n):
    import torch
    from paper_2211_05458_amd.lib import FlexiPart
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = FlexiPart(w.mesh, w.N, n)
    g.set_fluid_state(w.U)
    g.push(w.x, w.v, w.d, w.elem_hint)
    g.set_timing(True)
    return g, torch


@pytest.mark.parametrize("cells,n", [(2, MANY - 1), (2, MANY), (6, MANY + 1), (17, MANY)])
def test_steps_on_the_sources_sort(cells, n):
    w = W.curved_box(cells=cells, N=3, n_particles=n, seed=51)
    a, torch = _make(w, n)
    b, _ = _make(w, n)
    S = torch.zeros((a.E, 4, a.n3), dtype=torch.float64, device="cuda")
    for _ in range(3):
        a.deposit(S, drag=w.drag, kind=1, radius=0.2 * w.mesh.h)
        a.step(w.dt, 1, rk=w.rk, drag=w.drag, sort_every=0)
        b.step(w.dt, 1, rk=w.rk, drag=w.drag, sort_every=0)
    stages = 3 * (5 if w.rk == 0 else 3)
    assert a.timing()["stage_elem"][0] == (stages if n >= MANY else 0)
    assert b.timing()["stage_elem"][0] == 0
    ra, rb = a.read(), b.read()
    for k in ra:
        np.testing.assert_array_equal(ra[k], rb[k])


@pytest.mark.parametrize("cells,n", [(1, MANY), (6, 4000), (6, MANY + 1), (17, MANY)])
def test_forces_on_and_off_between_sorts(cells, n):
    w = W.curved_box(cells=cells, N=3, n_particles=n, seed=52)
    a, _ = _make(w, n)
    b, _ = _make(w, n)
    for k in range(4):
        for g, sort in ((a, 4), (b, 0)):
            g.step(w.dt, 1, rk=w.rk, drag=w.drag, sort_every=sort, forces=15 * (k % 2), gravity=GRAVITY)
    t, stages = a.timing(), 4 * (5 if w.rk == 0 else 3)
    assert t["stage_elem"][0] == (stages if n >= MANY else stages // 2) and a.stats()["sorts"] == 1
    ra, rb = a.read(), b.read()
    for k in ra:
        np.testing.assert_array_equal(ra[k], rb[k])


def test_state_changes_precision_between_sorts():
    n = MANY
    w = W.curved_box(cells=5, N=5, n_particles=n, seed=53)
    g, torch = _make(w, n)
    for k in range(4):
        g.set_fluid_state(w.U.astype(np.float32) if k % 2 else w.U)
        g.step(w.dt, 1, rk=w.rk, drag=w.drag, precision=k % 2, sort_every=4, forces=15 * (k // 2), gravity=GRAVITY)
    assert g.timing()["stage_elem"][0] == 4 * (5 if w.rk == 0 else 3)
    st = g.stats()
    assert st["lost"] == 0 and st["sorts"] == 1


@pytest.mark.parametrize("forces", [0, 15])
def test_captured_step_after_a_sort_for_other_tasks(forces):
    """A captured step that does not sort runs on the last sort's tasks.  Between
    its replays steps with the other setting of the extra forces sort."""
    import torch
    n = 4000                                  # about 62 particles an element: tasks of 32 and of 64 differ
    w = W.curved_box(cells=4, N=3, n_particles=n, seed=54)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_05458_amd.lib import FlexiPart
    _, nb = FlexiPart.particle_block_layout(n)
    stream = torch.cuda.Stream()

    def step(g, f, sort):
        g.step(w.dt, 1, rk=w.rk, drag=w.drag, forces=f, gravity=GRAVITY, sort_every=sort)

    def start():
        g = FlexiPart(w.mesh, w.N, n)
        g.set_fluid_state(w.U)
        g.bind_particles(torch.zeros(nb, dtype=torch.uint8, device="cuda"), n)
        g.push(w.x, w.v * 10.0, w.d, w.elem_hint)
        step(g, forces, 1)
        return g
    with torch.cuda.stream(stream):
        a, b = start(), start()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            step(a, forces, 0)
        for _ in range(3):
            graph.replay()
            step(b, forces, 0)
            stream.synchronize()
            torch.cuda.synchronize()
            step(a, 15 - forces, 1)
            step(b, 15 - forces, 1)
            stream.synchronize()
        graph.replay()
        step(b, forces, 0)
        torch.cuda.synchronize()
        ra, rb = a.read(), b.read()
    for k in ra:
        np.testing.assert_array_equal(ra[k], rb[k])
