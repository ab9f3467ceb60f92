"""A state written through its device address (a source term added between
steps) has the time step of the state as written: as a mesh that was given
that state, bit for bit."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu

MESHES = [((96,), None, None), ((70, 44), None, None), ((24, 20, 18), None, None), ((32, 32, 32), (2, 2, 2), None),
          ((32, 32, 32), (2, 2, 2), [3])]


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


def _write(h, v):
    """Slower flow and half the internal energy, so a larger time step: a rate
    left from before could not hide under the new one."""
    import torch
    with torch.cuda.stream(h.stream):
        v.mul_(0.5)
        c = 1 if v.ndim == 5 else 0
        v.select(c, 0).mul_(2.0)


@pytest.mark.parametrize("n,blocks,refined,after",
                         [(*m, a) for m in MESHES for a in ("cfl_dt", "step_auto", "batch")
                          if a != "batch" or not m[1]])
@pytest.mark.parametrize("before", ["set", "step", "kept"])
def test_dt_of_the_written_state(H, n, blocks, refined, before, after):
    import torch
    say("state written", n, blocks, refined, before, after)
    c = wl.turbulence_3d(n=n, mach=0.6, seed=9)
    s = torch.cuda.Stream()

    def mesh():
        return H.Hydro(c.n, c.gamma, c.cfl, stream=s, blocks=blocks, refined=refined)

    h, ref = mesh(), mesh()
    W = c.W
    if refined is not None:
        W = np.ascontiguousarray(np.broadcast_to(c.W[:, :16, :16, :16], h.shape))
    h.set_primitive(W)
    v = h.state_view() if before == "kept" else None  # kept over the steps
    if before != "set":
        for _ in range(3):
            h.step(0.3 * h.cfl_dt())
    _write(h, h.state_view() if v is None else v)
    ref.set_state(h.get_state())
    if after == "cfl_dt":
        assert h.cfl_dt() == ref.cfl_dt()
        h.step(0.5 * ref.cfl_dt())
        ref.step(0.5 * ref.cfl_dt())
        assert h.cfl_dt() == ref.cfl_dt()
    elif after == "step_auto":
        h.step_auto(2)
        ref.step_auto(2)
    else:
        b = H.Batch([h], use_graph=False)
        b.step(2)
        s.synchronize()
        b.close()
        ref.step_auto(2)
    assert np.array_equal(h.get_state(), ref.get_state())
    h.close()
    ref.close()
