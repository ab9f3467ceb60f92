"""Host-dt steps leave the new state's CFL rate pending for a caller that asks
for every dt and take none otherwise: in any order of questions and steps the
time step is that of a mesh given the same state, bit for bit."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu

MESHES = [((130,), None, None), ((70, 44), None, None), ((24, 20, 18), None, None), ((32, 32, 32), (2, 2, 2), None),
          ((32, 32, 32), (2, 2, 2), [3])]
# q: hydro_cfl_dt, s: a step of a dt brought along, a: two device steps
ORDERS = ["ssqsqsq", "qssq", "qsa", "sa", "qsqssaqsq"]


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


@pytest.mark.parametrize("n,blocks,refined,streams",
                         [(*m, False) for m in MESHES] + [(*m, True) for m in MESHES if m[1] and not m[2]])
@pytest.mark.parametrize("order", ORDERS)
def test_dt_after_any_order(H, n, blocks, refined, order, streams):
    say("host steps", n, blocks, refined, order, streams)
    c = wl.turbulence_3d(n=n, mach=0.6, seed=11)

    def mesh():
        return H.Hydro(c.n, c.gamma, c.cfl, blocks=blocks, refined=refined)

    h, fresh = mesh(), mesh()
    W = c.W
    if refined is not None:
        W = np.ascontiguousarray(np.broadcast_to(c.W[:, :16, :16, :16], h.shape))
    h.set_primitive(W)
    fresh.set_primitive(W)
    dt = 0.2 * fresh.cfl_dt()
    for i, op in enumerate(order):
        if streams and i == len(order) // 2:
            h.set_block_streams(True)
        if op == "s":
            h.step(dt)
            continue
        fresh.set_state(h.get_state())
        if op == "q":
            assert h.cfl_dt() == fresh.cfl_dt()
        else:
            h.step_auto(2)
            fresh.step_auto(2)
            assert np.array_equal(h.get_state(), fresh.get_state())
    fresh.set_state(h.get_state())
    assert h.cfl_dt() == fresh.cfl_dt()
    assert h.steps_done() == sum({"s": 1, "a": 2}.get(op, 0) for op in order)
    h.close()
    fresh.close()
