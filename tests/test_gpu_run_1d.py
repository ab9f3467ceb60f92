"""A 1-D mesh of up to 1024 cells advances many steps in one launch of one
work-group: the same state, time and step count bit for bit as the two stage
launches a step that larger meshes take (reached by stage timing), at the
edges of waves and of the range, for every boundary rule, and with a run
limit that falls inside the launch."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu

PER, FREE, OUT, REF = 0, 1, 2, 3


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


def advance(H, c, bc, precision, integrator, by_stage, calls):
    h = H.Hydro(c.n, c.gamma, c.cfl, precision=precision, bc=bc, integrator=integrator)
    h.set_primitive(c.W)
    if by_stage:
        h.profile(1)
    out = []
    for steps, t_end in calls:
        h.step_auto(steps, t_end)
        out.append((h.get_state(), h.time(), h.steps_done(), h.cfl_dt()))
    h.close()
    return out


@pytest.mark.parametrize("n,bc", [(2, (PER, PER)), (3, (FREE, REF)), (63, (OUT, OUT)), (64, (PER, PER)),
                                  (257, (REF, OUT)), (1024, (PER, PER)), (1025, (FREE, FREE))])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("integrator", [0, 1])
def test_one_launch_equals_stage_launches(H, n, bc, precision, integrator):
    rng = np.random.default_rng(n)
    c = wl.sod_1d(n)
    c.W[0] *= 1.0 + 0.1 * rng.random(c.W[0].shape)
    c.W[1] += 0.3 * rng.standard_normal(c.W[1].shape)
    say("run 1-D", n, bc, precision, integrator)
    # three steps; to an end time that cuts a step short; past it (no steps)
    t = advance(H, c, (bc,), precision, integrator, True, [(3, 0.0), (2, 0.0)])
    t_end = 0.5 * (t[0][1] + t[1][1])
    calls = [(3, 0.0), (7, t_end), (2, t_end), (1, 0.0)]
    a = advance(H, c, (bc,), precision, integrator, True, calls)
    b = advance(H, c, (bc,), precision, integrator, False, calls)
    assert a[1][1] == t_end and a[2][2] == a[1][2]
    for (U, t, s, dt), (V, tv, sv, dv) in zip(a, b):
        assert np.isfinite(U).all() and np.array_equal(U, V) and (t, s, dt) == (tv, sv, dv)


def test_nonphysical_state_is_reported(H):
    c = wl.sod_1d(100)
    c.W[2, 0, 0, 40] = -1.0
    h = H.Hydro(c.n, c.gamma, c.cfl, bc=c.bc)
    h.set_primitive(c.W)
    h.step_auto(2)
    with pytest.raises(H.HydroError) as e:
        h.time()
    assert e.value.status == H.E_NONPHYSICAL
    h.close()
