"""A step that ends early, on an error that another library's call left behind in
the runtime: the next push and steps are as on a fresh handle (the stages' queue
counters, which each stage leaves cleared for the next, start from zero).

Bar: bitwise equal."""
import ctypes

import numpy as np
import pytest

from paper_2211_05458_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rk", [0, 1])
@pytest.mark.parametrize("sort", [0, 1, -1])
def test_steps_after_a_failed_step(rk, sort):
    import torch
    from paper_2211_05458_amd import lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hip = ctypes.CDLL("libamdhip64.so")
    n = 2000
    w = W.curved_box(cells=4, N=3, n_particles=n, seed=81)

    def make():
        g = lib.FlexiPart(w.mesh, w.N, n)
        g.set_fluid_state(w.U)
        g.push(w.x, w.v * 10.0, w.d, w.elem_hint)
        return g

    a, b = make(), make()
    torch.cuda.synchronize()
    assert hip.hipSetDevice(9999) != 0          # leaves its error behind
    with pytest.raises(lib.FPError):
        a.step(w.dt, 1, rk=rk, drag=w.drag, sort_every=sort)
    hip.hipGetLastError()
    torch.cuda.synchronize()
    a.push(w.x, w.v * 10.0, w.d, w.elem_hint)
    for g in (a, b):
        g.reset_stats()
        for k in range(3):      # the two schemes in turn: five stages and three
            g.step(w.dt, 1, rk=(rk + k) % 2, drag=w.drag, sort_every=sort)
    sa, sb = a.stats(), b.stats()
    ra, rb = a.read(), b.read()
    for k in ra:
        np.testing.assert_array_equal(ra[k], rb[k])
    for k in ("crossings", "wall_hits", "lost"):
        assert sa[k] == sb[k], k
